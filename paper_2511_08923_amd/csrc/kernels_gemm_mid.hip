// bf16 GEMM of the narrower products of 33 to 480 rows (the narrowest: to 768): out = A[M][K] x W[N][K]^T, fp32
// accumulation, same operand layouts as kernels_gemm.hip.
//
// A workgroup has no barrier and no LDS in its loop: its four waves, one per SIMD, split K between them (k steps in
// turn) and each accumulates the whole tile of RT x CT 32 x 32 blocks, taking both operands from memory straight into
// a register ring of D k steps.  Every fragment is loaded once per workgroup ((RT + CT) KiB per RT * CT MFMAs) and no
// wave waits for another; the four sums meet in LDS at the end, in wave order, where the epilogue reads them in the
// order it stores them.  What bounds it is the time a compute unit's loads are under way: about 58 GB/s per unit with
// weights from HBM (the same loop on weights that stay in L2 takes 60 instead of 81 us at 272 x 24576 x 4096, on
// activations that stay in L1 no less), so it serves the products that leave compute units idle otherwise;
// the accumulators, held four times, leave no registers for a deeper ring.
#include <type_traits>

#include "gemm_device.h"

namespace {

constexpr int PIECE = 528;                        // 16-byte pieces of 32 rows, padded: reads of a row's 8 pieces are conflict-free
constexpr int phase_of(int tiles) { return tiles < 8 ? tiles : 8; }      // tiles reduced at a time: 4 waves x 4.1 KiB each

template <int RT, int CT, int D, bool SWIGLU>
__global__ __launch_bounds__(256) void gemm_bf16_mid_kernel(const bf16_t *__restrict__ a, const bf16_t *__restrict__ w,
                                                            float *__restrict__ out, int M, int N, int K, int splits,
                                                            int n_pass, int n_tall) {
    static_assert(D * (RT + CT) <= 60, "the loads in flight are counted in six bits");
    constexpr int PHASE = phase_of(RT * CT);
    extern __shared__ __attribute__((aligned(16))) unsigned char mid_smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t32 = (N + 31) >> 5, m_tiles = (M + 31) >> 5;
    // Workgroup i of a launch runs on XCD i % 8: the row passes of a column block and split follow each other on one
    // XCD (the second read of the weights is an L2 hit), and with 2, 4 or 8 splits an XCD sees one share of K only
    const int j8 = blockIdx.x >> 3, unit = (j8 / n_pass) * 8 + (blockIdx.x & 7);
    const int bz = j8 % n_pass, split = unit % splits, tile0 = (unit / splits) * CT;
    if (tile0 >= t32) return;
    const int mt_base = bz * (RT - 1) + min(bz, n_tall), ct_here = bz < n_tall ? RT : RT - 1;
    const SplitRange sr = split_range(K, splits, split);
    const int q1 = sr.q1 * 2, qw = sr.q0 * 2 + wave;               // k steps of 16; this wave's: qw, qw + 4, ...
    const int n = max((q1 - sr.q0 * 2 + 3) >> 2, 0);
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(a, (size_t)(K >> 4) * m_tiles * 1024);
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(w, (size_t)t32 * 32 * K * 2);
    int w_off[CT];
#pragma unroll
    for (int j = 0; j < CT; ++j) w_off[j] = tile0 + j < t32 ? lane * 16 : OOB;
    auto ld = [&](__amdgpu_buffer_rsrc_t r, int off, int tiles, int tile, int s) __attribute__((always_inline)) {
        const int q = qw + 4 * s;
        return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, q < q1 ? off : OOB,
                                                                                q < q1 ? (q * tiles + tile) * 1024 : 0, 0));
    };
    f32x16 acc[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    bf16x8 af[D][RT], wf[D][CT];
    auto k_loop = [&](auto ra_tag) __attribute__((always_inline)) {
        constexpr int RA = decltype(ra_tag)::value;
#pragma unroll
        for (int s = 0; s < D; ++s) {              // in the order of the loop's reloads
#pragma unroll
            for (int i = 0; i < RA; ++i) af[s][i] = ld(ra, lane * 16, m_tiles, mt_base + i, s);
#pragma unroll
            for (int j = 0; j < CT; ++j) wf[s][j] = ld(rw, w_off[j], t32, tile0 + j, s);
            __builtin_amdgcn_sched_barrier(0);
        }
        for (int s0 = 0; s0 < n; s0 += D) {
#pragma unroll
            for (int s = 0; s < D; ++s) {
#pragma unroll
                for (int i = 0; i < RA; ++i) {
#pragma unroll
                    for (int j = 0; j < CT; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[s][j], af[s][i], acc[i][j], 0, 0, 0);
                    af[s][i] = ld(ra, lane * 16, m_tiles, mt_base + i, s0 + s + D);
                    __builtin_amdgcn_sched_barrier(0);       // every reload right behind the last use of its slot
                }
#pragma unroll
                for (int j = 0; j < CT; ++j) wf[s][j] = ld(rw, w_off[j], t32, tile0 + j, s0 + s + D);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    if (RT == 1 || ct_here == RT) k_loop(std::integral_constant<int, RT>());
    else k_loop(std::integral_constant<int, RT == 1 ? 1 : RT - 1>());

    // ---- the four waves' sums.  acc is out^T: lane l holds activation row l % 32, its registers 4g .. 4g+3 are the
    // columns 4 * (2g + l/32) .. +3 of the tile: piece 2g + l/32 of that row
    const int lq = lane & 31, lh = lane >> 5;
#pragma unroll
    for (int p0 = 0; p0 < RT * CT; p0 += PHASE) {
        constexpr int TILES = RT * CT;
        if (p0) __syncthreads();
#pragma unroll
        for (int t = 0; t < PHASE; ++t) {
            if (p0 + t >= TILES) break;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x16 &v = acc[(p0 + t) / CT][(p0 + t) % CT];
                *(f32x4 *)(mid_smem + ((wave * PHASE + t) * 8 + 2 * g + lh) * PIECE + lq * 16) =
                    (f32x4){v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
            }
        }
        __syncthreads();
        for (int t = wave; t < min(PHASE, TILES - p0); t += 4) {
            const int i = (p0 + t) / CT, j = (p0 + t) % CT;
            if (i >= ct_here || tile0 + j >= t32) continue;
            auto piece = [&](int c4, int r) {
                const unsigned char *s = mid_smem + (t * 8 + c4) * PIECE + r * 16;
                f32x4 v = *(const f32x4 *)s;
#pragma unroll
                for (int x = 1; x < 4; ++x) v += *(const f32x4 *)(s + x * (PHASE * 8 * PIECE));
                return v;
            };
            if constexpr (SWIGLU) {
                // columns 0-15 gate, 16-31 up of the same 16 features: lane (half, row) makes features 8 * half .. +7 of
                // its row, its 16 bytes of the next GEMM's A fragment
                bf16x8 h;
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    const f32x4 gt = piece(2 * lh + x, lq), up = piece(4 + 2 * lh + x, lq);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        h[4 * x + e] = (bf16_t)(gt[e] * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * gt[e])) * up[e]);
                }
                *(bf16x8 *)(reinterpret_cast<bf16_t *>(out) + (((size_t)(tile0 + j) * m_tiles + mt_base + i) * 64 + lane) * 8) = h;
            } else {
                float *o = out + (size_t)split * pt_split_stride(M, N);
#pragma unroll
                for (int x = 0; x < 4; ++x) {      // eight lanes store the 128 bytes of a row
                    const int r = (lane >> 3) + 8 * x, c4 = lane & 7;
                    const int row = (mt_base + i) * 32 + r, col = (tile0 + j) * 32 + 4 * c4;
                    const f32x4 v = piece(c4, r);
                    if (row < M && col < N) *(f32x4 *)(o + pt_index(col, row, M)) = v;
                }
            }
        }
    }
}

template <int RT, int CT, int D, bool SWIGLU>
void launch_mid(const bf16_t *a, const bf16_t *w, float *out, int M, int N, int K, const GemmPlan &p, hipStream_t st) {
    constexpr int REDUCE_LDS = 4 * phase_of(RT * CT) * 8 * PIECE;
    const int units = ((N + 31) / 32 + CT - 1) / CT * p.splits, n_tall = (M + 31) / 32 - p.m_chunks * (RT - 1);
    static std::atomic<bool> granted[kLdsDevices];
    grant_lds((const void *)gemm_bf16_mid_kernel<RT, CT, D, SWIGLU>, REDUCE_LDS, granted);
    gemm_bf16_mid_kernel<RT, CT, D, SWIGLU><<<dim3((units + 7) / 8 * 8 * p.m_chunks), 256, REDUCE_LDS, st>>>(
        a, w, out, M, N, K, p.splits, p.m_chunks, n_tall);
}

// ring depth in k steps: as many registers as the accumulators leave, four or eight (the waves' shares of K are usually
// multiples of eight steps)
template <bool SWIGLU>
void launch_mid_rows(const bf16_t *a, const bf16_t *w, float *out, int M, int N, int K, const GemmPlan &p, hipStream_t st) {
    if (p.mt == 1) launch_mid<1, 2, 8, SWIGLU>(a, w, out, M, N, K, p, st);
    else if (p.mt == 2) launch_mid<2, 2, 8, SWIGLU>(a, w, out, M, N, K, p, st);
    else if (p.mt == 3) launch_mid<3, 2, 8, SWIGLU>(a, w, out, M, N, K, p, st);
    else if (p.mt == 4) launch_mid<4, 2, 8, SWIGLU>(a, w, out, M, N, K, p, st);
    else if (p.mt == 5) launch_mid<5, 2, 8, SWIGLU>(a, w, out, M, N, K, p, st);
    else if (p.mt == 6) launch_mid<6, 2, 4, SWIGLU>(a, w, out, M, N, K, p, st);
    else if (p.mt == 7) launch_mid<7, 2, 4, SWIGLU>(a, w, out, M, N, K, p, st);
    else launch_mid<8, 2, 4, SWIGLU>(a, w, out, M, N, K, p, st);
}

}  // namespace

// Partial sums in the tiled layout, or (one split) SwiGLU of the interleaved gate/up matrix.
void launch_gemm_bf16_mid(const bf16_t *a, const bf16_t *w, float *out, int M, int N, int K, const GemmPlan &p, bool swiglu,
                          hipStream_t st) {
    if (swiglu) launch_mid_rows<true>(a, w, out, M, N, K, p, st);
    else launch_mid_rows<false>(a, w, out, M, N, K, p, st);
}
