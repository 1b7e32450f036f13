// Device code shared by the bf16 GEMM kernels: buffer descriptors, the split-K ranges, and the row choice of the fused
// vocabulary reduction.
#pragma once
#include <atomic>

#include "tidar_internal.h"

namespace {

// LDS above 64 KiB has to be granted per kernel, on every device the kernel is launched on; `granted` is the launcher's own
// (several threads may be the first: the grant is the same).
constexpr int kLdsDevices = 64;
inline void grant_lds(const void *kernel, int bytes, std::atomic<bool> (&granted)[kLdsDevices]) {
    int dev = -1;
    (void)hipGetDevice(&dev);
    const bool known = dev >= 0 && dev < kLdsDevices;
    if (known && granted[dev].load(std::memory_order_relaxed)) return;
    (void)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (known) granted[dev].store(true, std::memory_order_relaxed);
}

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
// the same, non-temporal: for weights that one workgroup reads once
__device__ inline bf16x8 buf_load_once(__amdgpu_buffer_rsrc_t r, int byte_off) {
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, byte_off, 0, 2));
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

// out^T tiles: lane l holds activation row l % 16 and weight columns 4 * (l / 16) .. +3 of each 16 x 16 tile.
// Two neighbouring column tiles make the 128 bytes a row has in a 32-column tile of the output; half of the lanes
// trade one tile's values so that eight lanes store one whole row.
template <bool ROWMAJOR>
__device__ inline void store_pair(const f32x4 &t0, const f32x4 &t1, float *__restrict__ o, int row0, int col0, int M, int N,
                                  int lane) {
    const int n = lane & 15, g = lane >> 4;
    const bool low = n < 8;
    f32x4 first, second;                          // rows row0 + n % 8 and row0 + 8 + n % 8
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float give = low ? t1[e] : t0[e];
        const float got = __builtin_bit_cast(
            float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, give), 0x128, 0xf, 0xf, true));   // row_ror:8
        first[e] = low ? t0[e] : got;
        second[e] = low ? got : t1[e];
    }
    const int col = col0 + (low ? 0 : 16) + 4 * g;
    if (col >= N) return;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int row = row0 + 8 * h + (n & 7);
        if (row < M) *(f32x4 *)(o + (ROWMAJOR ? (size_t)row * N + col : pt_index(col, row, M))) = h ? second : first;
    }
}

// Epilogue of a wave that holds MTA row tiles (from row tile r0 of the workgroup's pass on) by NT column tiles
// (from tile0 on) of 32x32x16 accumulators.  NW waves per workgroup; ct_here: row tiles of the pass that exist; smem: at least NW * 32 * 36
// floats nobody reads any more (with NT == 1 and GEMM_EPI_ARGMAX all waves of the workgroup have to come here).
template <int MTA, int NT, int NW>
__device__ inline void large_epilogue(const f32x16 (&acc)[MTA][NT], float *__restrict__ out, unsigned char *gemm_smem,
                                      int epi, int split, int M, int N, int mt_base, int ct_here, int tile0, int r0,
                                      int wave, int lane, const ChooseArgs &ch) {
    const int t32 = (N + 31) >> 5, m_tiles = (M + 31) >> 5;
    // The weight fragment is the MFMA's first operand, so the accumulator holds the output tile
    // transposed: lane l owns activation row l%32 of the row tile, and its register e is column
    // 8*(e/4) + 4*(l/32) + e%4 of the 32-column tile: four consecutive registers are four consecutive columns of
    // one row.
    const int lq = lane & 31, lh = lane >> 5;
    if (epi == GEMM_EPI_SWIGLU) {
        // columns 0-15 of a tile are gate, 16-31 up, of the same 16 features (tile T = features 16T..16T+15 =
        // exactly one k step of the next GEMM's A-fragment layout), so gate and up of a feature sit in the same
        // lane, 8 registers apart: h = silu(gate) * up needs no shuffle.  A lane then holds features 4*(l/32)+0..3
        // and 8+4*(l/32)+0..3 of its row; the fragment wants 8*(l/32)+0..7.  One half-wave swap fixes that: the
        // upper lanes hand their features 4-7 to the lower lanes and take the lower lanes' 8-11.
        bf16_t *ho = reinterpret_cast<bf16_t *>(out);
        typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int mt = 0; mt < MTA; ++mt) {
            const int tile_r = r0 + mt;
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                unsigned pk[4];
#pragma unroll
                for (int i = 0; i < 8; i += 2) {
                    float h2[2];
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const float g = acc[mt][j][i + t], u = acc[mt][j][i + t + 8];
                        h2[t] = g * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g)) * u;
                    }
                    bf16x2 b;
                    b[0] = (bf16_t)h2[0];
                    b[1] = (bf16_t)h2[1];
                    pk[i >> 1] = __builtin_bit_cast(unsigned, b);
                }
                // pk[0..1]: features 4*lh + 0..3; pk[2..3]: features 8 + 4*lh + 0..3
                const auto s0 = __builtin_amdgcn_permlane32_swap(pk[0], pk[2], false, false);
                const auto s1 = __builtin_amdgcn_permlane32_swap(pk[1], pk[3], false, false);
                typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
                const u32x4 piece = {s0[0], s1[0], s0[1], s1[1]};
                if (tile_r < ct_here && tile0 + j < t32)
                    *(u32x4 *)(ho + (((size_t)(tile0 + j) * m_tiles + mt_base + tile_r) * 64 + lane) * 8) = piece;
            }
        }
        return;
    }
    if (epi == GEMM_EPI_ARGMAX) {
        // a lane walks its 16 columns of each of the wave's tiles in rising order (strict > keeps the lowest column
        // of a tie), then the two half-waves, which hold the same rows, are folded.  A column group is 64 columns:
        // the wave's two tiles, or (NT = 1) the tiles of two neighbouring waves, folded through LDS.
        const int G = (t32 + 1) >> 1;
        float *pmax = out;
        int *pidx = (int *)(out + (size_t)G * M);
        float bests[MTA];
        int bis[MTA];
#pragma unroll
        for (int mt = 0; mt < MTA; ++mt) {
            const int tile_r = r0 + mt;
            float best = -INFINITY;
            int bi = tile0 * 32 + 4 * lh;
            bests[mt] = best;
            bis[mt] = bi;
            if (tile_r >= ct_here) continue;      // wave-uniform
            const RowChoice rc = row_choice(ch, (mt_base + tile_r) * 32 + lq, M);
            if (__any(rc.noisy || rc.sel >= 0)) {     // a tile that holds rows a token is taken from (wave-uniform)
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int col = (tile0 + j) * 32 + 8 * (e >> 2) + 4 * lh + (e & 3);
                        float v = acc[mt][j][e];
                        if (rc.sel >= 0 && col < N) ch.sel_logits[(size_t)rc.sel * N + col] = v;
                        if (rc.noisy) v = perturbed_logit(v, rc.inv_t, rc.key, (uint32_t)col);
                        if (col < N && v > best) {
                            best = v;
                            bi = col;
                        }
                    }
            } else {
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int col = (tile0 + j) * 32 + 8 * (e >> 2) + 4 * lh + (e & 3);
                        const float v = acc[mt][j][e];
                        if (col < N && v > best) {
                            best = v;
                            bi = col;
                        }
                    }
            }
            const float ob = __shfl_xor(best, 32);
            const int oi = __shfl_xor(bi, 32);
            if (ob > best || (ob == best && oi < bi)) {
                best = ob;
                bi = oi;
            }
            bests[mt] = best;
            bis[mt] = bi;
        }
        if constexpr (NT == 1) {
            // the odd wave of a pair hands its result to the even one (the staging buffers are free by now)
            float *rb = reinterpret_cast<float *>(gemm_smem);
            int *ri = reinterpret_cast<int *>(gemm_smem) + NW * MTA * 32;
            if (lh == 0) {
#pragma unroll
                for (int mt = 0; mt < MTA; ++mt) {
                    rb[(wave * MTA + mt) * 32 + lq] = bests[mt];
                    ri[(wave * MTA + mt) * 32 + lq] = bis[mt];
                }
            }
            __syncthreads();
            if (wave & 1) return;
#pragma unroll
            for (int mt = 0; mt < MTA; ++mt) {
                const float ob = rb[((wave + 1) * MTA + mt) * 32 + lq];
                const int oi = ri[((wave + 1) * MTA + mt) * 32 + lq];
                if (ob > bests[mt] || (ob == bests[mt] && oi < bis[mt])) {
                    bests[mt] = ob;
                    bis[mt] = oi;
                }
            }
        }
#pragma unroll
        for (int mt = 0; mt < MTA; ++mt) {
            const int tile_r = r0 + mt;
            const int row = (mt_base + tile_r) * 32 + lq;
            if (tile_r < ct_here && lh == 0 && row < M && tile0 < t32) {
                pmax[(size_t)(tile0 >> 1) * M + row] = bests[mt];
                pidx[(size_t)(tile0 >> 1) * M + row] = bis[mt];
            }
        }
        return;
    }
    // Partial sums and logits: a lane's four consecutive columns are 16 bytes, but neighbouring lanes are
    // neighbouring rows, 128 bytes apart in the tiled layout.  Each tile is therefore turned through a per-wave
    // LDS patch (16-byte writes, 16-byte reads; the staging buffers are free after the last barrier) so that eight
    // lanes together store one whole row of the tile (128 bytes) and a store instruction covers 1 KiB in one run.
    float *scr = reinterpret_cast<float *>(gemm_smem) + wave * (32 * 36);
    float *o = out + (size_t)split * pt_split_stride(M, N);
#pragma unroll
    for (int mt = 0; mt < MTA; ++mt) {
        const int tile_r = r0 + mt;
        if (tile_r >= ct_here) continue;          // also drops the repeated tile (wave-uniform)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *(f32x4 *)(scr + lq * 36 + 8 * g + 4 * lh) = (f32x4){acc[mt][j][4 * g], acc[mt][j][4 * g + 1],
                                                                     acc[mt][j][4 * g + 2], acc[mt][j][4 * g + 3]};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int idx = lane + 64 * i;
                const int r = idx >> 3, c4 = idx & 7;
                const f32x4 v = *(const f32x4 *)(scr + r * 36 + 4 * c4);
                const int row = (mt_base + tile_r) * 32 + r;
                const int col = (tile0 + j) * 32 + 4 * c4;
                if (row < M && col < N) {
                    const size_t oi = (epi == GEMM_EPI_ROWMAJOR) ? (size_t)row * N + col : pt_index(col, row, M);
                    *(f32x4 *)(o + oi) = v;
                }
            }
        }
    }
}

}  // namespace
