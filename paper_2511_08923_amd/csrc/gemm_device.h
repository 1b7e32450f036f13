// Device code shared by the bf16 GEMM kernels: buffer descriptors, the split-K ranges, and the row choice of the fused
// vocabulary reduction.
#pragma once
#include "tidar_internal.h"

namespace {

constexpr int SPLIT_UNIT = 512;           // k elements
constexpr int OOB = 0x7ffffff0;           // byte offset beyond any buffer: the load returns zeros

__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void *base, size_t bytes) {
    // raw buffer (stride 0), 32-bit data format; num_records in bytes
    return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, (int)(bytes > 0x7fffffe0ull ? 0x7fffffe0ull : bytes),
                                             0x00020000);
}
__device__ inline bf16x8 buf_load(__amdgpu_buffer_rsrc_t r, int byte_off) {
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, byte_off, 0, 0));
}

struct SplitRange {
    int q0, q1;   // k steps [q0, q1)
};
__device__ inline SplitRange split_range(int K, int splits, int split) {
    const int units = (K + SPLIT_UNIT - 1) / SPLIT_UNIT;
    const int per = (units + splits - 1) / splits;
    SplitRange r;
    r.q0 = split * per * (SPLIT_UNIT / 32);
    r.q1 = min(K >> 5, (split + 1) * per * (SPLIT_UNIT / 32));
    return r;
}

// What the fused vocabulary reduction does with output row `row`: perturb its values before the maximum is formed
// (key, inv_t when noisy) and/or also write its logits to the compact buffer (sel >= 0: row index there).
struct RowChoice {
    bool noisy;
    uint64_t key;
    float inv_t;
    int sel;
};
__device__ inline RowChoice row_choice(const ChooseArgs &ch, int row, int M) {
    RowChoice rc;
    rc.noisy = false;
    rc.key = 0;
    rc.inv_t = 1.f;
    rc.sel = -1;
    if (ch.n_choose <= 0 || row >= M) return rc;
    const int b = row / ch.Rh, o = row - b * ch.Rh;
    if (o < ch.n_choose) {
        if (ch.sample) {
            rc.noisy = true;                // causal rows are label shifted: they predict the position after theirs
            rc.key = noise_key(ch.seed, ch.seq_base + b, ch.pos_rows[(size_t)b * ch.pos_stride + ch.pos_row0 + o] + 1);
            rc.inv_t = ch.inv_t;
        }
        if (ch.sel_logits) rc.sel = b * 2 * ch.n_choose + o;
    } else if (ch.sel_logits) {
        const int m = o - ch.n_choose;
        if (m % ch.mix_stride == 0 && m / ch.mix_stride < ch.n_choose) rc.sel = b * 2 * ch.n_choose + ch.n_choose + m / ch.mix_stride;
    }
    return rc;
}

}  // namespace
