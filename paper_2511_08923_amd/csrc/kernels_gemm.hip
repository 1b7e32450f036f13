// Skinny bf16 GEMM of the decode step: out = A[M][K] (bf16) x W[N][K]^T (bf16), fp32 accumulation.
//
// M is the step's row count (1 .. 272 at batch 1; more rows run as row passes, 481 and more in kernels_gemm_rows.hip,
// the narrower products of 33 .. 480 - the narrowest to 768 - in kernels_gemm_mid.hip, the widest and those of many short
// shares of K up to 480 rows in kernels_gemm_tall.hip, the LM head of 33 .. 160 rows over some 65400 columns and more, where its last
// round of workgroups is nearly full to 256 or 288, in a form of kernels_gemm_rows.hip), N and K are model dimensions: every weight byte
// is used once per step, so the kernel is a weight streamer with MFMA attached.
//   * W lives in HBM as the register image of the 32x32x16 MFMA B operand
//     ([k step of 16][32-column tile][lane][8]); a wave's load of one fragment is one fully coalesced 1 KiB read
//     that goes straight to VGPRs through a ring many k steps deep (up to 32 rows: into an LDS ring that the
//     workgroup's waves share).  The k step is the outer index so that the workgroups, which all advance through K at
//     the same pace, read one
//     contiguous front of the matrix.
//   * A lives in memory as the register image of the MFMA A operand (see ActLayout): the slice a workgroup
//     needs for a chunk of K is one contiguous block and its LDS image reads back conflict-free.
//   * every load is a raw buffer load: out-of-range tiles, rows and k steps are steered to an out-of-bounds
//     offset, which the hardware answers with zeros and no memory traffic.  The steady-state loop therefore
//     has no branches, and the compiler can keep exact in-flight counts (vmcnt(n), not vmcnt(0)) on the ring;
//     sched_barrier pins each reload right behind the MFMAs that free its slot.
//   * M <= 32: 16x16x32 MFMA (fewer pad rows), both operands through LDS (gemm_bf16_few_kernel).  M > 32: 32x32x16 MFMA
//     (half the operand reads of 16x16x32 per product; a bare loop with few accumulators measured 2.2 vs 1.2 PFLOP/s),
//     A staged through LDS once per workgroup and prefetched into
//     registers ahead of the MFMAs; 4 waves either as a 2 x 2 grid over 128 columns (two row halves x two
//     64-column groups: launches without a row split), or side by side, every wave over all row tiles of the pass
//     (no weight fragment is then loaded by two waves): eight waves over 256 columns for single-split grids, four over
//     128 columns for the two-pass launches of 33-480 rows, one column tile per wave (no padded tile slots; twice the LDS fragment
//     reads per MFMA, which the LDS has room for).  The weight fragment is the MFMA's first operand, so the
//     accumulators hold the output transposed (lane = row): every epilogue starts from that.
//   * split-K works in units of 512 k, row passes are workgroups of their own; up to 480 rows the split count
//     and the order of a row's sum depend on (N, K) and the row class (M <= 4 with the producer folded in, M <= 32, more)
//     only, so the partial-sum grouping of a
//     row does not depend on how many rows travel with it (from 481 rows on both also follow the number of 256-row
//     multiples; which of the kernels with one order serves a row count is the plan's).  Splits fill about half the CUs, two row passes the other half: a split
//     costs an M x N partial sum written and read again, a row pass only a second read of W from L2.
//   * output: [split][32-column tile][row][32] fp32 partial sums (summed in fixed order by the consumer), or
//     row-major logits, or - fused epilogues - bf16 SwiGLU products in the next GEMM's A-fragment layout, or
//     per-column-group (maximum, column) pairs for the greedy vocabulary reduction.
// 16x16x32: A lane l = row l%16, k slots 8*(l/16)..+7; B lane l = column l%16, same k slots; D lane l register i
// = row 4*(l/16)+i, column l%16.   32x32x16: A lane l = row l%32, k slots 8*(l/32)..+7; B lane l = column l%32;
// D lane l register i = row 8*(i/4) + 4*(l/32) + i%4, column l%32.
#include "gemm_device.h"
#include "lds_dma.h"

namespace {

template <int MTW, int NT>
__device__ inline void store_tiles(const f32x4 (&acc)[MTW][NT], float *out, int split, int M, int N, int tile0,
                                   int n_tiles, int mt0, int lane, int out_row_major, const ChooseArgs &ch) {
    if (out_row_major == GEMM_EPI_ARGMAX) {
        // lane l holds rows 4*(l/16)+i of a 16-row tile and column l%16 of each of its NT 16-column tiles: the
        // larger of its columns per row, then the 16 lanes of a row group are folded (ties: lowest column)
        const int G = ((N >> 4) + 1) >> 1;
        float *pmax = out;
        int *pidx = (int *)(out + (size_t)G * M);
#pragma unroll
        for (int mt = 0; mt < MTW; ++mt) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float best = -INFINITY;
                int bi = (tile0 << 4) + (lane & 15);
                const int row_i = (mt0 + mt) * 16 + (lane >> 4) * 4 + i;
                const RowChoice rc = row_choice(ch, row_i, M);
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    float v = acc[mt][j][i];
                    const int col = ((tile0 + j) << 4) + (lane & 15);
                    if (rc.sel >= 0 && tile0 + j < n_tiles) ch.sel_logits[(size_t)rc.sel * N + col] = v;
                    if (rc.noisy) v = perturbed_logit(v, rc.inv_t, rc.key, (uint32_t)col);
                    if (tile0 + j < n_tiles && v > best) {
                        best = v;
                        bi = ((tile0 + j) << 4) + (lane & 15);
                    }
                }
#pragma unroll
                for (int o = 1; o < 16; o <<= 1) {
                    const float ob = __shfl_xor(best, o);
                    const int oi = __shfl_xor(bi, o);
                    if (ob > best || (ob == best && oi < bi)) {
                        best = ob;
                        bi = oi;
                    }
                }
                const int row = (mt0 + mt) * 16 + (lane >> 4) * 4 + i;
                if ((lane & 15) == 0 && row < M) {
                    pmax[(size_t)(tile0 >> 1) * M + row] = best;
                    pidx[(size_t)(tile0 >> 1) * M + row] = bi;
                }
            }
        }
        return;
    }
    if (NT == 2 && out_row_major == GEMM_EPI_SWIGLU) {
        // the wave's two 16-column tiles are gate and up of the same 16 features (tile0 is even): a lane holds both
        // values of (row, feature), so h = silu(gate) * up needs no data movement; it is stored as bf16 in the
        // A-fragment layout of the next GEMM
        bf16_t *ho = reinterpret_cast<bf16_t *>(out);
        const ActLayout lay = act_layout(M);
        if (tile0 + 1 < n_tiles) {
#pragma unroll
            for (int mt = 0; mt < MTW; ++mt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int row = (mt0 + mt) * 16 + (lane >> 4) * 4 + i;
                    const float g = acc[mt][0][i], u = acc[mt][NT - 1][i];
                    // a division, as in swiglu_kernel: v_rcp_f32 flushes silu below g = -87.3 and is an ulp off above
                    const float h = g / (1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g)) * u;
                    if (row < M) ho[af_index(row, (tile0 >> 1) * 16 + (lane & 15), lay)] = (bf16_t)h;
                }
        }
        return;
    }
    float *o = out + (size_t)split * pt_split_stride(M, N);
#pragma unroll
    for (int mt = 0; mt < MTW; ++mt) {
        const int row0 = (mt0 + mt) * 16 + (lane >> 4) * 4;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int tile = tile0 + j;
            if (tile >= n_tiles) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = row0 + i;
                if (row < M) {
                    size_t idx = out_row_major == GEMM_EPI_ROWMAJOR ? (size_t)row * N + tile * 16 + (lane & 15)
                                               : pt_index(tile * 16 + (lane & 15), row, M);
                    o[idx] = acc[mt][j][i];
                }
            }
        }
    }
}

// ------------------------------------------------------------------ M <= 4: one row tile, the GEMM's producer folded in
// The A operand is built by the workgroup itself (see FuseArgs) into LDS as plain bf16 rows of its share of K; a
// lane's fragment is then one 16-byte LDS read (lanes of rows that do not exist take zeros).  W streams through a register
// ring, whose first loads are in flight while the prologue runs; its loads are non-temporal, as nobody reads them again (together
// with those of gemm_bf16_few_kernel 8B one-token step 3626 -> 3527 us; these alone, one-token step of 1 / 2 / 3 / 4 sequences, 1.5B 1620 ->
// 1584, 1829 -> 1817, 2076 -> 2045, 2284 -> 2242, 8B with eight layers 977 -> 946 to 1103 -> 1079, in grids of 36 to 192 workgroups; eight and ten layers of d_model 1024 and d_ff 4096
// and 2816, grids of 16 to 64, 372 -> 378 and 489 -> 498 at one sequence, 419 -> 420 and 542 -> 552 at two).
template <int FUSE>
__global__ __launch_bounds__(256) void gemm_bf16_small_fused_kernel(FuseArgs f, const bf16_t *__restrict__ w,
                                                                    float *__restrict__ out, int M, int N, int K,
                                                                    int splits, int epi) {
    constexpr int NT = 2, PFK = 16, MT = 1;
    extern __shared__ __attribute__((aligned(16))) unsigned char fused_smem[];
    bf16_t *lds_a = reinterpret_cast<bf16_t *>(fused_smem);           // [M][kr]
    __shared__ float red[4][kFuseMaxRows];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n_tiles = N >> 4;
    const SplitRange sr = split_range(K, splits, blockIdx.y);
    const int k0 = sr.q0 * 32, kr = max(sr.q1 - sr.q0, 0) * 32;
    const int tile0 = (blockIdx.x * 4 + wave) * NT;
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(w, (size_t)((N + 31) / 32) * 32 * K * 2);
    const int t32 = (N + 31) >> 5;
    const int n = lane & 15, g = lane >> 4;
    int w_off[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j)
        w_off[j] = (tile0 + j < n_tiles)
                       ? ((((g >> 1) * t32 + ((tile0 + j) >> 1)) * 64) + (g & 1) * 32 + ((tile0 + j) & 1) * 16 + n) * 16
                       : OOB;
    const int w_step = 2 * t32 * 1024;
    auto ld_w = [&](int j, int q) {
        return buf_load_once(rw, (q < sr.q1 && w_off[j] != OOB) ? w_off[j] + q * w_step : OOB);
    };
    // Loads return in order: the ring's first loads (for a short share of K: all of the workgroup's weights) are
    // issued *behind* the prologue's loads, which come from L2 and the memory-side cache and are back long before
    // the weights; the prologue's arithmetic then runs while the weights stream in.
    bf16x8 wbuf[PFK][NT];
    auto fill_ring = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < PFK; ++s)
#pragma unroll
            for (int j = 0; j < NT; ++j) wbuf[s][j] = ld_w(j, sr.q0 + s);
        __builtin_amdgcn_sched_barrier(0);
    };

    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
    if (FUSE == GEMM_FUSE_NORM) {
        // thread t holds columns 4 (t + 256 j) .. +3 of every row.  All loads of a row (the residual piece and up
        // to eight partial sums per piece) are issued before the first is used: one round trip per row, not one
        // per split.
        constexpr int KP = kFuseMaxK / 1024, SB = 8;
        float4 v[kFuseMaxRows][KP];
        float ss[kFuseMaxRows];
#pragma unroll
        for (int r = 0; r < kFuseMaxRows; ++r) {
            ss[r] = 0.f;
#pragma unroll
            for (int j = 0; j < KP; ++j) v[r][j] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (r >= M) continue;
#pragma unroll
            for (int j = 0; j < KP; ++j) {
                const int c = 4 * (tid + 256 * j);
                if (c < K) v[r][j] = *(const float4 *)(f.x_in + (size_t)r * K + c);
            }
            for (int sp0 = 0; sp0 < f.S; sp0 += SB) {
                float4 q[SB][KP];
#pragma unroll
                for (int u = 0; u < SB; ++u)
#pragma unroll
                    for (int j = 0; j < KP; ++j) {
                        const int c = min(4 * (tid + 256 * j), K - 4);            // clamped: always a real address
                        q[u][j] = *(const float4 *)(f.part + pt_index(c, r, M) +
                                                    (size_t)min(sp0 + u, f.S - 1) * f.split_stride);
                    }
#pragma unroll
                for (int u = 0; u < SB; ++u)                  // in split order, as the stand-alone kernel sums
#pragma unroll
                    for (int j = 0; j < KP; ++j)
                        if (sp0 + u < f.S && 4 * (tid + 256 * j) < K) {
                            v[r][j].x += q[u][j].x; v[r][j].y += q[u][j].y;
                            v[r][j].z += q[u][j].z; v[r][j].w += q[u][j].w;
                        }
            }
#pragma unroll
            for (int j = 0; j < KP; ++j)
                ss[r] += v[r][j].x * v[r][j].x + v[r][j].y * v[r][j].y + v[r][j].z * v[r][j].z + v[r][j].w * v[r][j].w;
        }
        fill_ring();
#pragma unroll
        for (int r = 0; r < kFuseMaxRows; ++r) {
            float t = ss[r];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o);
            if (lane == 0) red[wave][r] = t;
        }
        __syncthreads();
        const bool writer = blockIdx.x == 0 && blockIdx.y == 0;
#pragma unroll
        for (int r = 0; r < kFuseMaxRows; ++r) {
            if (r >= M) continue;
            const float tot = ((red[0][r] + red[1][r]) + red[2][r]) + red[3][r];
            const float rs = rsqrtf(tot / (float)K + f.eps);
#pragma unroll
            for (int j = 0; j < KP; ++j) {
                const int c = 4 * (tid + 256 * j);
                if (c >= K) continue;
                const float4 a = v[r][j];
                if (writer) *(float4 *)(f.x_out + (size_t)r * K + c) = a;
                if (c >= k0 && c < k0 + kr) {
                    const bf16x4 gn = *(const bf16x4 *)(f.gain + c);
                    const bf16x4 o = {(bf16_t)(a.x * rs * (float)gn[0]), (bf16_t)(a.y * rs * (float)gn[1]),
                                      (bf16_t)(a.z * rs * (float)gn[2]), (bf16_t)(a.w * rs * (float)gn[3])};
                    *(bf16x4 *)(lds_a + (size_t)r * kr + (c - k0)) = o;
                }
            }
        }
    } else {
        // One item = four head-dim values of one (row, head) of this workgroup's share of K = n_q * 128.  The
        // threads that the items leave over share an item's splits (TPI threads per item, sixteen splits loaded
        // together: one or two round trips to memory instead of one per split).  The fold is the online form:
        // every split keeps an integral reference, so moving the running reference scales by an exact power of
        // two and the order of the rescales leaves no trace; partial folds of an item meet in LDS in thread order.
        constexpr int SB = 16;
        const int group = f.n_q / f.n_kv, F = group * f.R, per_row = kr >> 2;
        const int items = M * per_row;
        int tpi = 1;
        while (tpi < 8 && items * tpi * 2 <= 256) tpi *= 2;
        __shared__ float fold[256][6];
        const int part_i = tid % tpi;
        for (int it0 = 0; it0 < items; it0 += 256 / tpi) {               // one round when the items fit (uniform)
        const int item = it0 + tid / tpi;
        float mrun = -INFINITY, den = 0.f;
        float4 num = make_float4(0.f, 0.f, 0.f, 0.f);
        int r = 0, kk = k0;
        if (item < items) {
            r = item / per_row;
            kk = k0 + 4 * (item - r * per_row);
            const int head = kk >> 7, d0 = kk & 127;
            const int b = r / f.R, rr = r - b * f.R;
            const int kvh = head / group, hq = head - kvh * group;
            const size_t base = ((size_t)b * f.n_kv + kvh) * f.a_splits;
            const int fr = hq * f.R + rr;
            const int per_t = (f.a_splits + tpi - 1) / tpi;
            const int s_lo = part_i * per_t, s_hi = min(f.a_splits, s_lo + per_t);
            for (int sp0 = s_lo; sp0 < s_hi; sp0 += SB) {
                float m[SB], l[SB];
                float4 o[SB];
#pragma unroll
                for (int u = 0; u < SB; ++u) {
                    const size_t pi = (base + min(sp0 + u, f.a_splits - 1)) * F + fr;
                    m[u] = f.mpart[pi];
                    l[u] = f.lpart[pi];
                    o[u] = *(const float4 *)(f.opart + pi * 128 + d0);
                }
                float mc = mrun;
#pragma unroll
                for (int u = 0; u < SB; ++u)
                    if (sp0 + u < s_hi) mc = fmaxf(mc, m[u]);
                if (mc == -INFINITY) continue;                              // nothing but empty splits so far
                const float sc = exp2f(mrun - mc);                          // 0 when mrun is still -inf
                num.x *= sc; num.y *= sc; num.z *= sc; num.w *= sc;
                den *= sc;
                mrun = mc;
#pragma unroll
                for (int u = 0; u < SB; ++u) {
                    if (sp0 + u >= s_hi || m[u] == -INFINITY) continue;     // absent or empty split
                    const float wgt = exp2f(m[u] - mrun);
                    num.x += wgt * o[u].x; num.y += wgt * o[u].y; num.z += wgt * o[u].z; num.w += wgt * o[u].w;
                    den += wgt * l[u];
                }
            }
        }
        if (it0 == 0) fill_ring();
        if (tpi > 1) {
            __syncthreads();                                               // the previous round's folds were read
            fold[tid][0] = mrun; fold[tid][1] = den;
            fold[tid][2] = num.x; fold[tid][3] = num.y; fold[tid][4] = num.z; fold[tid][5] = num.w;
            __syncthreads();
            if (item < items && part_i == 0) {
                for (int t = 1; t < tpi; ++t) {
                    const float *o = fold[tid + t];
                    if (o[0] == -INFINITY) continue;
                    const float mc = fmaxf(mrun, o[0]);
                    const float sa = exp2f(mrun - mc), sb = exp2f(o[0] - mc);
                    num.x = num.x * sa + o[2] * sb; num.y = num.y * sa + o[3] * sb;
                    num.z = num.z * sa + o[4] * sb; num.w = num.w * sa + o[5] * sb;
                    den = den * sa + o[1] * sb;
                    mrun = mc;
                }
            }
        }
        if (item < items && part_i == 0) {
            const float inv = 1.f / den;
            const bf16x4 o = {(bf16_t)(num.x * inv), (bf16_t)(num.y * inv), (bf16_t)(num.z * inv), (bf16_t)(num.w * inv)};
            *(bf16x4 *)(lds_a + (size_t)r * kr + (kk - k0)) = o;
        }
        }
    }
    __syncthreads();

    f32x4 acc[MT][NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[0][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    // A fragment of k step q: lane (row n, k slots 8g .. 8g+7)
    const bf16_t *a_row = lds_a + (size_t)min(n, M - 1) * kr + 8 * g;
    const bool a_real = n < M;
    for (int qb = sr.q0; qb < sr.q1; qb += PFK) {
#pragma unroll
        for (int s = 0; s < PFK; ++s) {
            const int q = qb + s;
            bf16x8 af = {0, 0, 0, 0, 0, 0, 0, 0};
            if (a_real && q < sr.q1) af = *(const bf16x8 *)(a_row + (q - sr.q0) * 32);
#pragma unroll
            for (int j = 0; j < NT; ++j)
                acc[0][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, wbuf[s][j], acc[0][j], 0, 0, 0);
#pragma unroll
            for (int j = 0; j < NT; ++j) wbuf[s][j] = ld_w(j, q + PFK);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (tile0 >= n_tiles) return;
    ChooseArgs none = {};
    store_tiles<MT, NT>(acc, out, blockIdx.y, M, N, tile0, n_tiles, 0, lane, epi, none);
}

// ------------------------------------------------------------------ M <= 32: both operands through LDS
// A workgroup's four waves share both operands through LDS, where they go straight from memory (buffer_load ... lds), a ring of
// four chunks of 64 k (80 KB with CT = 4: two workgroups per compute unit, one fills its ring while the other ends).  MT row
// tiles of 16 x CT column tiles of 32: with two row tiles a wave takes one of them and every other column tile, with one row tile
// (CT = 4) a column tile or (CT = 2) half a column tile.  It is bound by the weight stream: 6 and 20 x 24576 x 4096 32.2 and 33.1 us
// (6.1 TB/s; with every wave streaming its own columns and all of A through register rings 35.7 and 42.3), 6 x 2048 x 1536 5.9 ->
// 4.3, 6 x 17920 x 1536 15.1 -> 13.1, 20 x 17920 x 1536 18.0 -> 14.2, 20 x 151936 x 4096 247 -> 226.  Eight chunks instead of
// four 34.2 and 225 us (one workgroup per unit), three 36.3 and 229.
// ONCE: the weights' loads are non-temporal (FEW_ONCE workgroups and more).  A stream of loads alone reaches 7.1 TB/s so, 6.4
// otherwise: 1 / 20 x 151936 x 4096 210 / 214 -> 186 / 191 us, 6 x 151936 x 1536 83.3 -> 73.5, 1 x 24576 x 4096 32.2 -> 31.4, 20 x
// 6144 x 4096 11.9 -> 11.4, 20 x 4096 x 12288 21.2 -> 20.8, 20 x 4096 x 4096 9.8 -> 9.3.  With fewer workgroups it is latency that
// counts, and theirs is longer: 6 and 20 x 17920 x 1536 (140 workgroups) 12.24 and 13.17 -> 12.38 and 13.29.
constexpr int FEW_CHUNKS = 4, FEW_ONCE = 180;
template <int MT, int CT, bool ONCE>
__global__ __launch_bounds__(256) void gemm_bf16_few_kernel(const bf16_t *__restrict__ a, const bf16_t *__restrict__ w,
                                                            float *__restrict__ out, int M, int N, int K, int splits,
                                                            int epi, ChooseArgs ch) {
    constexpr int P = FEW_CHUNKS, LOADS = CT + 1;
    constexpr int CHUNK = 4 * (CT + 1) * 1024;                      // W [k step of 16][column tile], then A [k step of 32][row tile]
    constexpr int NJ = CT * MT / 4 > 0 ? CT * MT / 4 : 1;           // column tiles (CT = 2, MT = 1: halves) of a wave
    constexpr int NH = CT * MT >= 4 ? 2 : 1;                        // halves of a column tile a wave takes
    static_assert(P * LOADS < 64, "the loads in flight are counted in six bits");
    extern __shared__ __attribute__((aligned(16))) unsigned char few_smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mh = MT == 2 ? wave & 1 : 0, ng = MT == 2 ? wave >> 1 : NH == 2 ? wave : wave >> 1, h0 = NH == 2 ? 0 : wave & 1;
    constexpr int STEP = MT == 2 ? 2 : 4;
    const int t32 = (N + 31) >> 5, tile0 = blockIdx.x * CT;
    const SplitRange sr = split_range(K, splits, blockIdx.y);
    const int n_steps = max(sr.q1 - sr.q0, 0), n_chunks = (n_steps + 1) >> 1;      // steps of 32 k
    const int4v da = raw_desc(a, (size_t)(K >> 5) * MT * 1024), dw = raw_desc(w, (size_t)t32 * 32 * K * 2);
    const unsigned dst0 = lds_address(few_smem);
    // a wave brings one of a chunk's four k steps of W and one of its 2 MT fragments of A; what does not exist is asked for
    // too, out of bounds: zeros, and the same number of loads in flight everywhere
    auto issue = [&](int c, int buf) __attribute__((always_inline)) {
        const bool ok = 2 * c + (wave >> 1) < n_steps, ok_a = MT == 2 ? ok : wave < 2 && 2 * c + wave < n_steps;
        const unsigned dst = dst0 + buf * CHUNK;
        dma16(dst + (4 * CT + wave) * 1024, ok_a ? lane * 16 : OOB, da, ok_a ? ((sr.q0 + 2 * c) * MT + wave) * 1024 : 0);
        const int src = ((2 * sr.q0 + 4 * c + wave) * t32 + tile0) * 1024;
#pragma unroll
        for (int j = 0; j < CT; ++j)
            (ONCE ? dma16_once : dma16)(dst + (wave * CT + j) * 1024, ok && tile0 + j < t32 ? lane * 16 : OOB, dw,
                                        ok ? src + j * 1024 : 0);
    };
    f32x4 acc[NJ][1][NH];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int h = 0; h < NH; ++h) acc[j][0][h] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const unsigned char *fw = few_smem + ((lane >> 5) * CT + ng) * 1024 + ((lane >> 4) & 1) * 512 + h0 * 256 + (lane & 15) * 16;
    const unsigned char *fa = few_smem + (4 * CT + mh) * 1024 + lane * 16;
#pragma unroll
    for (int c = 0; c < P - 1; ++c) issue(c, c);
    int buf = 0, far = P - 1;
    for (int c = 0; c < n_chunks; ++c) {
        wait_loads<(P - 2) * LOADS>();
        lds_barrier();                   // chunk c has landed for everyone, chunk c-1 has been read by everyone
        bf16x8 af[2], wf[2][NJ][NH];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            af[kk] = *(const bf16x8 *)(fa + buf * CHUNK + kk * MT * 1024);
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int h = 0; h < NH; ++h)
                    wf[kk][j][h] = *(const bf16x8 *)(fw + buf * CHUNK + (2 * kk * CT + STEP * j) * 1024 + h * 256);
        }
        issue(c + P - 1, far);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int h = 0; h < NH; ++h)
                    acc[j][0][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[kk], wf[kk][j][h], acc[j][0][h], 0, 0, 0);
        far = buf;
        buf = buf + 1 == P ? 0 : buf + 1;
    }
    wait_loads<0>();                     // nothing may land in LDS that is another workgroup's by then
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int t = 2 * (tile0 + ng + STEP * j) + h0;
        if (t < (N >> 4)) store_tiles<1, NH>(acc[j], out, blockIdx.y, M, N, t, N >> 4, mh, lane, epi, ch);
    }
}

// ------------------------------------------------------------------ 32 < M: 32x32x16 MFMA, A through LDS
// MTA: 32-row tiles per wave.  2 x 2 waves (WIDE false): the workgroup pass covers CTL = 2*MTA row tiles (9 when
// MTA is 5: the second row half then repeats a tile whose results are dropped) of 128 columns.  WIDE: four waves
// side by side, each over all CTL = MTA row tiles and NT 32-column tiles of the workgroup's 128 * NT columns.
// Chunk of K = 128 (8 k steps); weight ring 16 k steps.  WG: k steps whose weights are asked for together.  A compute unit returns
// loads in the order they were asked for, so activations from L2 wait behind weights from HBM each time the two alternate: with WG = 8
// a chunk's weights go out at its end, behind its A pieces, although that makes the ring one chunk deep (where: launch_side).
template <int MTA, bool WIDE, int NT = 2, int NW = 4, int WG = 1>
__global__ __launch_bounds__(64 * NW) void gemm_bf16_large_kernel(const bf16_t *__restrict__ a,
                                                              const bf16_t *__restrict__ w, float *__restrict__ out,
                                                              int M, int N, int K, int splits, int epi,
                                                              int swz_p, int swz_c, int n_pass, int n_colblk,
                                                              ChooseArgs ch) {
    constexpr int KS = 8;
    static_assert(WG == 1 || (WIDE && WG == KS), "weights by the k step or by the chunk");
    static_assert(NT == 2 || (NT == 1 && WIDE), "one column tile per wave only with the waves side by side");
    static_assert(NW == 4 || (NW == 8 && WIDE && NT == 1), "eight waves only side by side with one column tile each");
    constexpr int THREADS = 64 * NW;
    constexpr int PFK = 2 * KS;                  // weight ring depth in k steps: two chunks
    constexpr int CTL = WIDE ? MTA : (MTA == 5) ? 9 : 2 * MTA;
    // Workgroup i of a launch runs on XCD i % 8.  The row passes of a column block and split follow each other on one XCD
    // (the second read of its weights is an L2 hit) and the splits are dealt out first: with 2, 4 or 8 of them an XCD sees one
    // share of K only, so a piece of A that its L2 fetches from afar serves all its workgroups of that share, and not one in
    // `splits` of them.  Splits over blockIdx.y before: 272 / 216 x 4096 x 12288 41.4 -> 39.0, 37.6 -> 34.4 us inside a step, 4096
    // x 4096 21.3 -> 20.7, 6144 x 4096 (two splits) the same.
    // swz_p > 0, many column blocks and one split: the (pass, column block) plane is cut into super-tiles of swz_p x swz_c
    // workgroups, each handed whole to one XCD, passes fastest: the workgroups that
    // are resident together on an XCD then share their A rows and W columns through its L2 instead of each
    // streaming a private W slice from HBM.
    int bx, bz, split = 0;
    if (swz_p > 0) {
        const int i = blockIdx.x, xcd = i & 7, j = i >> 3;
        const int per = swz_p * swz_c;
        const int n_sp = (n_pass + swz_p - 1) / swz_p, n_sc = (n_colblk + swz_c - 1) / swz_c;
        const int st = (j / per) * 8 + xcd, within = j % per;
        if (st >= n_sp * n_sc) return;
        bz = (st % n_sp) * swz_p + within % swz_p;
        bx = (st / n_sp) * swz_c + within / swz_p;
        if (bz >= n_pass || bx >= n_colblk) return;
    } else {
        const int j = blockIdx.x >> 3, unit = (j / n_pass) * 8 + (blockIdx.x & 7);
        bz = j % n_pass;
        split = unit % splits;
        bx = unit / splits;
        if (bx >= n_colblk) return;
    }
    constexpr int PIECES = CTL * KS * 64;        // 16-byte pieces per chunk
    constexpr int STAGE = (PIECES + THREADS - 1) / THREADS;
    constexpr int FR = KS * MTA;                 // A fragments a wave consumes per chunk
    constexpr int AFD = NT == 1 ? 6 : 3;         // LDS -> register prefetch distance in fragments (NT MFMAs each)
    static_assert(2 * STAGE <= FR, "one staging piece is stored after every other fragment");
    extern __shared__ __attribute__((aligned(16))) unsigned char gemm_smem[];
    bf16x8 *lds = reinterpret_cast<bf16x8 *>(gemm_smem);      // [2][KS][CTL][64]

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int mh = WIDE ? 0 : wave & 1, ng = WIDE ? wave : wave >> 1;
    const int t32 = (N + 31) >> 5, m_tiles = (M + 31) >> 5;
    const int mt_base = bz * CTL;
    const int ct_here = min(CTL, m_tiles - mt_base);
    const int q_total = K >> 4;                                // k steps of 16
    const SplitRange sr32 = split_range(K, splits, split);
    const int q0 = sr32.q0 * 2, q1 = min(sr32.q1 * 2, q_total);
    const int c0 = q0 / KS, c1 = (q1 + KS - 1) / KS;
    const int tile0 = (bx * (WIDE ? NW : 2) + ng) * NT;  // first 32-column tile of this wave
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(a, (size_t)q_total * m_tiles * 1024);
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(w, (size_t)t32 * 32 * K * 2);

    int w_off[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) w_off[j] = (tile0 + j < t32) ? ((tile0 + j) * 64 + lane) * 16 : OOB;
    const int w_step = t32 * 1024;
    auto ld_w = [&](int j, int q) {
        return buf_load(rw, (q < q1 && w_off[j] != OOB) ? w_off[j] + q * w_step : OOB);
    };

    // A staging: piece p = tid + s*THREADS of the chunk = lane `lane` of fragment (wave + NW*s) -> (k step, row tile).
    // The fragment index is wave-uniform, so its address lives in scalar registers (the buffer load's scalar
    // offset) and only lane*16, or the out-of-bounds offset for a fragment that does not exist, in a VGPR.
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    const int a_chunk_step = KS * m_tiles * 1024;
    const int lane16 = lane * 16;
    bf16x8 stage[STAGE];
    auto load_a1 = [&](int s, int c) {          // piece s of chunk c -> staging register s
        const int i = wv + NW * s;
        const int ks = i / CTL, ct = i % CTL;
        const bool ok = i < CTL * KS && ct < ct_here && c < c1;
        stage[s] = __builtin_bit_cast(
            bf16x8, __builtin_amdgcn_raw_buffer_load_b128(ra, ok ? lane16 : OOB,
                                                          (ks * m_tiles + mt_base + ct) * 1024 + c * a_chunk_step, 0));
    };
    auto store_a1 = [&](int s, int buf) {
        if (STAGE * THREADS == PIECES || tid + s * THREADS < PIECES) lds[buf * PIECES + tid + s * THREADS] = stage[s];
    };

    f32x16 acc[MTA][NT];
#pragma unroll
    for (int i = 0; i < MTA; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    bf16x8 wbuf[PFK][NT];
    // The loads of the ring's second half and of the second chunk's A are issued in the order the loop issues
    // them, so that the in-flight counts the compiler derives at the loop entry equal those of the back edge.
#pragma unroll
    for (int s = 0; s < STAGE; ++s) load_a1(s, c0);
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int j = 0; j < NT; ++j) wbuf[s][j] = ld_w(j, q0 + s);
#pragma unroll
    for (int s = 0; s < STAGE; ++s) store_a1(s, 0);
#pragma unroll
    for (int f = 0; f < FR; ++f) {
        if (f % (MTA * WG) == MTA * WG - 1) {
#pragma unroll
            for (int d = WG - 1; d >= 0; --d)
#pragma unroll
                for (int j = 0; j < NT; ++j) wbuf[KS + f / MTA - d][j] = ld_w(j, q0 + KS + f / MTA - d);
        }
        if ((f & 1) && (f >> 1) < STAGE) load_a1(f >> 1, c0 + 1);
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();

    // fragment f of a chunk = (k step f / MTA, row tile f % MTA of this wave's half, clamped to a real tile)
    int frag_off[MTA];
#pragma unroll
    for (int mt = 0; mt < MTA; ++mt) frag_off[mt] = min(mh * MTA + mt, CTL - 1) * 64 + lane;
    auto lds_frag = [&](int buf, int f) { return lds[buf * PIECES + (f / MTA) * CTL * 64 + frag_off[f % MTA]]; };

    for (int cb = c0; cb < c1; cb += 2) {
#pragma unroll
        for (int ci = 0; ci < 2; ++ci) {          // two chunks = one revolution of the weight ring
            const int c = cb + ci;
            const int buf = ci;                   // chunks alternate buffers starting from buffer 0 at c0
            bf16x8 af[AFD + 1];
#pragma unroll
            for (int f = 0; f < AFD; ++f) af[f] = lds_frag(buf, f);
#pragma unroll
            for (int f = 0; f < FR; ++f) {
                if (f + AFD < FR) af[(f + AFD) % (AFD + 1)] = lds_frag(buf, f + AFD);
                const int ks = f / MTA, mt = f % MTA;
                const int slot = (ci * KS + ks) % PFK;
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[mt][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wbuf[slot][j], af[f % (AFD + 1)], acc[mt][j],
                                                                         0, 0, 0);   // W first: acc = out^T
                if (mt == MTA - 1 && ks % WG == WG - 1) {              // the ring slots of the last WG k steps are free again
#pragma unroll
                    for (int d = WG - 1; d >= 0; --d)
#pragma unroll
                        for (int j = 0; j < NT; ++j) wbuf[slot - d][j] = ld_w(j, c * KS + ks - d + PFK);
                }
                // the next chunk's A goes to the other LDS buffer one piece at a time between the MFMAs (a
                // burst of stores would sit in front of the fragment reads in the in-order LDS queue), and
                // the freed staging register at once takes the piece of the chunk after that
                if ((f & 1) && (f >> 1) < STAGE) {
                    store_a1(f >> 1, buf ^ 1);
                    load_a1(f >> 1, c + 2);
                }
                __builtin_amdgcn_sched_barrier(0);    // pin the order: LDS prefetch, MFMAs, ring reload
            }
            __syncthreads();
        }
    }

    large_epilogue<MTA, NT, NW>(acc, out, gemm_smem, epi, split, M, N, mt_base, ct_here, tile0, mh * MTA, wave, lane, ch);
}

template <int MT, int CT>
void launch_few(const bf16_t *a, const bf16_t *w, float *out, int M, int N, int K, const GemmPlan &p, int epi, hipStream_t st,
                const ChooseArgs &ch) {
    constexpr int SMEM = FEW_CHUNKS * 4 * (CT + 1) * 1024;
    const dim3 grid(((N + 31) / 32 + CT - 1) / CT, p.splits);
    auto go = [&](auto kernel, std::atomic<bool>(&granted)[kLdsDevices]) {
        grant_lds((const void *)kernel, SMEM, granted);
        kernel<<<grid, 256, SMEM, st>>>(a, w, out, M, N, K, p.splits, epi, ch);
    };
    static std::atomic<bool> granted[2][kLdsDevices];
    if (grid.x * grid.y >= FEW_ONCE) go(gemm_bf16_few_kernel<MT, CT, true>, granted[1]);
    else go(gemm_bf16_few_kernel<MT, CT, false>, granted[0]);
}

template <int MTA, bool WIDE, int NT = 2, int NW = 4, int WG = 1>
void launch_large(const bf16_t *a, const bf16_t *w, float *out, int M, int N, int K, const GemmPlan &p, int epi,
                  hipStream_t st, const ChooseArgs &ch) {
    constexpr int CTL = WIDE ? MTA : (MTA == 5) ? 9 : 2 * MTA;
    constexpr int BN = WIDE ? 32 * NW * NT : 128;
    int m_tiles = (M + 31) / 32;
    const int n_colblk = (N + BN - 1) / BN, n_pass = (m_tiles + CTL - 1) / CTL;
    dim3 grid((n_colblk * p.splits + 7) / 8 * 8 * n_pass);
    int swz_p = 0, swz_c = 0;
    if (p.swz > 0 && n_pass >= 2) {          // super-tiles of swz x swz workgroups, dealt to the XCDs in turn
        swz_p = p.swz < n_pass ? p.swz : n_pass;
        swz_c = p.swz;
        const int n_st = ((n_pass + swz_p - 1) / swz_p) * ((n_colblk + swz_c - 1) / swz_c);
        grid = dim3(8 * ((n_st + 7) / 8) * swz_p * swz_c);
    }
    // two staging buffers of a chunk's A tiles; the epilogue's per-wave transposition patches (4 x 32 x 36 floats)
    // reuse the same memory and need 18 KiB of it
    constexpr size_t PATCH = (size_t)NW * 32 * 36 * 4;
    constexpr size_t SMEM = (size_t)2 * CTL * 8 * 1024 > PATCH ? (size_t)2 * CTL * 8 * 1024 : PATCH;
    static std::atomic<bool> granted[kLdsDevices];
    grant_lds((const void *)gemm_bf16_large_kernel<MTA, WIDE, NT, NW, WG>, SMEM, granted);
    gemm_bf16_large_kernel<MTA, WIDE, NT, NW, WG><<<grid, 64 * NW, SMEM, st>>>(a, w, out, M, N, K, p.splits, epi, swz_p, swz_c, n_pass,
                                                               n_colblk, ch);
}

// Four waves side by side, one column tile each.  Which products ask for a chunk's weights together: those cut over K, with shares of
// up to 1024 k at any height of a pass, with longer ones in passes of up to five row tiles.  A chunk's activations then come one behind
// the other, and the ring is one chunk deep; where little of a launch is steady state (short shares) or a chunk is short (few row
// tiles) that pays.  One k step at a time -> together, weights from HBM, activations just written:
//   * shares of 1024: 216 / 272 / 340 / 384 / 480 x 4096 x 4096 19.0 -> 17.0, 21.4 -> 19.6, 23.0 -> 22.0, 24.2 -> 22.6, 27.3 -> 27.3 us,
//     216 / 272 / 384 x 8192 x 2048 18.3 -> 17.2, 21.1 -> 19.5, 23.9 -> 22.4 (192 rows 14.9 -> 15.7);
//   * longer: 132 / 216 / 256 x 4096 x 12288 31.2 -> 31.0, 37.3 -> 36.1, 39.1 -> 38.0, 216 x 5120 x 4096 22.0 -> 20.6, 132 / 216 x 3840 x
//     10240 26.3 -> 25.4, 30.7 -> 30.2; five row tiles 272 x 6144 x 4096 25.9 -> 26.6, 320 rows 26.8 -> 27.0, 272 x 8192 x 4096 29.8 ->
//     29.3, 272 x 4096 x 12288 41.1 -> 41.4, 8B step of 16 layers, 272 / 288 rows 3601 / 3575 -> 3586 / 3558; six and more would lose:
//     340 / 440 x 4096 x 12288 45.7 -> 47.6, 53.1 -> 55.8, 396 x 6144 x 4096 33.1 -> 34.6, 396 x 8192 x 4096 37.4 -> 39.6;
//   * one split would lose too: 100 x 16384 x 2048 17.9 -> 20.0, 216 x 28672 x 4096 63 -> 68.6, head of 210 rows, 65536 x 4096, 133 ->
//     147.
// Eight waves lose (LM head 379 -> 389), four k steps at a time are in between.
template <int MTA>
void launch_side(const bf16_t *a, const bf16_t *w, float *out, int M, int N, int K, const GemmPlan &p, int epi,
                 hipStream_t st, const ChooseArgs &ch) {
    const int units = (K + SPLIT_UNIT - 1) / SPLIT_UNIT, share = (units + p.splits - 1) / p.splits;
    if (p.splits > 1 && (share <= 2 || MTA <= 5)) launch_large<MTA, true, 1, 4, 8>(a, w, out, M, N, K, p, epi, st, ch);
    else launch_large<MTA, true, 1>(a, w, out, M, N, K, p, epi, st, ch);
}

}  // namespace

// Clamps a split count to the units there are and drops empty trailing splits.
static int fit_splits(int want, int units) {
    want = want < 1 ? 1 : want > units ? units : want;
    const int per = (units + want - 1) / want;
    return (units + per - 1) / per;
}

// Products of up to 32 rows that run with two column tiles per workgroup: those whose 64-column blocks fill the chip with three
// and more whole splits, or nearly fill it with two (figures at the launch)
static bool few_rows_two(int N) {
    const int blocks = (N + 63) / 64;
    return blocks <= 85 || (blocks >= 116 && blocks <= 128);
}

bool gemm_fuse_ok(int M, int N, int K) { return M >= 1 && M <= kFuseMaxRows && K <= kFuseMaxK && K % 32 == 0 && N % 16 == 0; }

void launch_gemm_bf16_fused(const FuseArgs &f, const bf16_t *w, float *out, int M, int N, int K, const GemmPlan &p,
                            int epi, hipStream_t st) {
    dim3 grid((N + 127) / 128, p.splits, 1);
    const int units = (K + SPLIT_UNIT - 1) / SPLIT_UNIT, per = (units + p.splits - 1) / p.splits;
    const size_t smem = (size_t)M * per * SPLIT_UNIT * 2;             // bf16 rows of the largest share of K
    if (f.kind == GEMM_FUSE_NORM)
        gemm_bf16_small_fused_kernel<GEMM_FUSE_NORM><<<grid, 256, smem, st>>>(f, w, out, M, N, K, p.splits, epi);
    else
        gemm_bf16_small_fused_kernel<GEMM_FUSE_COMBINE><<<grid, 256, smem, st>>>(f, w, out, M, N, K, p.splits, epi);
}

GemmPlan plan_gemm_bf16_fused(int M, int N, int K, bool force_single_split) {
    GemmPlan p = plan_gemm_bf16(M, N, K, force_single_split);
    if (!force_single_split) {          // column blocks of 128 whatever N: O of the 8B shape with half the splits 13.0 -> 15.0 us
        const int wgs = (N + 127) / 128, units = (K + SPLIT_UNIT - 1) / SPLIT_UNIT;
        p.splits = wgs < 128 ? fit_splits((256 + wgs / 2) / wgs, units) : 1;
    }
    return p;
}

GemmPlan plan_gemm_bf16(int M, int N, int K, bool force_single_split) {
    GemmPlan p;
    p.nt = 2;
    p.bk = 128;
    p.wide = 0;
    p.nw = 4;
    p.swz = 0;
    p.rows = 0;
    p.mid = 0;
    const int wgs = (N + 127) / 128;
    const int units = (K + SPLIT_UNIT - 1) / SPLIT_UNIT;
    auto fit = [&](int want) { return fit_splits(want, units); };
    int splits = 1;
    if (M <= 32) {
        p.mt = M <= 16 ? 1 : 2;                  // 16-row tiles per wave (narrow kernel)
        p.m_chunks = 1;
        // nearest count that brings the grid to about one wave of CUs; from half of that on a single split, which saves
        // the partial sums and, for gate/up, the SwiGLU launch (1.5B shape, 6 rows: 17.1 + 4.0 us in two splits)
        // Products in column blocks of 64: as many splits as the chip holds workgroups, and none more.  A few workgroups beyond 256
        // are a second one on some units, which the launch waits for: 6 rows, nearest count -> this, 2176 x 12288 14.7 -> 12.4 us
        // (8 -> 6 splits), 2944 x 12288 18.4 -> 14.8, 3456 x 12288 20.4 -> 16.9, 4224 x 4096 10.9 -> 9.4, 4480 x 12288 25.7 -> 20.8
        // (4 -> 3).  (A split is also a copy of the output that the next kernel reads.)
        const bool two = few_rows_two(N);
        const int blocks = two ? (N + 63) / 64 : wgs;
        if (!force_single_split && wgs < 128) splits = fit(two ? 256 / blocks : (256 + blocks / 2) / blocks);
    } else {
        // Partial sums are the expensive part of a split (each one is M x N floats written and read again), so
        // the column blocks are split over K only until about half the CUs are busy; the rest of the chip is
        // filled by cutting the rows into two workgroup passes, which costs a second read of W from L2 and no
        // extra output.  The split count is a function of (N, K) alone: a row's sum is grouped the same way
        // whatever the batch size.
        if (!force_single_split) splits = fit(128 / wgs);
        const int t = (M + 31) / 32;             // 32-row tiles
        if (!force_single_split && (t < 16 ? wgs * splits <= 64 : t <= 24 && wgs * splits <= 40)) {
            // kernels_gemm_mid.hip: the waves of a workgroup split K.  It takes the products whose two row passes
            // below would fill less than half of the compute units.  Measured at 132 / 272 / 430 rows, weights from HBM, activations
            // just written, two passes -> this: with 24-36 column blocks x splits 7.1 / 10.5 / 13.9 -> 5.5 / 7.1 / 8.4 us (1024 x
            // 2048), 6.6 / 9.7 / 13.1 -> 5.6 / 6.9 / 8.3 (4096 x 512), 7.4 / 10.5 / 14.6 -> 5.8 / 7.5 / 10.5 (the small model's O,
            // 1536 x 1536, in 3 splits either way), with 48 (its QKV, 2048 x 1536; 1536 x 2048, 3072 x 1024) 7.8 / 10.8 / 15.0 -> 7.2 /
            // 10.5 / 12.4, 7.6 / 10.8 / 15.1 -> 7.0 / 10.2 / 12.1, 7.6 / 10.8 / 15.0 -> 7.0 / 10.2 / 11.9, with 64 (2048 x 2048, 4096 x
            // 1024) 7.9 / 11.1 / 14.9 -> 7.5 / 10.9 / 12.8, 7.8 / 11.2 / 14.9 -> 7.5 / 10.6 / 12.5.  Where two passes fill more it
            // loses 10 % inside a step, where the activations come from other XCDs.
            // The narrowest keep it up to 768 rows, many-row kernel -> this at 544 / 640 / 768 rows: with 36 (1536 x 1536)
            // 21.0 / 18.9 / 20.3 -> 13.4 / 15.1 / 14.3, with 40 (2560 x 1024) 21.4 / 19.6 / 20.8 -> 13.8 / 15.9 / 17.6, with 48
            // (2048 x 1536) 20.0 / 18.7 / 20.4 -> 18.5 / 19.1 / 20.7, with 64 (2048 x 2048) 20.3 / 19.0 / 20.7 -> 22.0 / 23.0 /
            // 22.9.  The row limits are class borders (480 rows, a 256-row multiple): the four waves sum K in four
            // interleaved shares, so inside a class the choice has to be one of (N, K) alone.  (Against two
            // passes it is also faster for wide single-split products of up to five row tiles, 72 x 24576 x 4096 45.2 ->
            // 40.8 us, but not at nine, 68.2 -> 81.5; most of those have kernels_gemm_tall.hip now.)
            // Per workgroup: its fragments at the 27 B per clock that a compute unit takes in from afar, or the
            // matrix cores' rate, plus 4 us of launch, ring fill and reduction; a split also costs the partial
            // sums at 6 TB/s out and 4 TB/s back in.  The split count is the best at nine row tiles in two passes,
            // a function of (N, K) alone; the number of passes follows the rows.
            p.mid = 1;
            const int t32 = (N + 31) / 32;
            auto cost = [&](int tiles, int sc, int passes) {
                const int rt = (tiles + passes - 1) / passes;
                const int rounds = ((t32 + 1) / 2 * sc * passes + 255) / 256;
                const double load = (rt + 2) * 1024 / 27.0, mfma = rt * 2 * 8 / 0.9;
                return rounds * (K / 16.0 / sc * (load > mfma ? load : mfma) / 2100.0 + 4.0) +
                       sc * tiles * 32.0 * N * 1.67e-6;
            };
            p.splits = 1;
            for (int c = 2; c <= units && c <= 8; ++c)
                if (cost(9, fit(c), 2) < cost(9, p.splits, 2)) p.splits = fit(c);
            p.m_chunks = (t + 7) / 8;                // eight row tiles: the accumulators that fit the AGPRs
            for (int n = p.m_chunks + 1; n <= t; ++n)
                if (cost(t, p.splits, n) < cost(t, p.splits, p.m_chunks)) p.m_chunks = n;
            p.mt = (t + p.m_chunks - 1) / p.m_chunks;
            return p;
        }
        if (t >= 16) {                               // kernels_gemm_rows.hip
            // The number of row passes (of five to nine row tiles, equal to within one) and of splits that minimise an
            // estimate in microseconds: rounds of 256 workgroups x (K share x the measured time per k of a pass of h
            // row tiles and 256 columns, 7.5 + 1.6 h ns, plus 6 + h of prologue and epilogue), plus the partial sums
            // through the fabric at 6 TB/s out and 4 TB/s back in.  (Predicted / measured: 2048 x 24576 x 4096 292 /
            // 340, 2176 x 4096 x 12288 178 / 165, 1000 x 24576 x 4096 179 / 181, 600 x 24576 x 4096 149 / 146.)
            // The class begins where a layer as a whole gains over the register-ring kernel that served 512 rows and more
            // before: 8B shape at 481 / 531 rows QKV 52.9 -> 46.7 / 41.2 -> 45.6 us, O 34.0 -> 29.6 / 27.9 -> 30.1, gate/up
            // 100.6 -> 103.3 / 141.1 -> 106.7, down 76.2 -> 66.6 / 60.6 -> 63.3.
            // The split count, never above the (N, K) rule's, is taken for whole 256-row multiples: within this
            // class a row's sum is grouped the same way for every row count of the same multiple.
            p.rows = 1;
            const int cols = (N + 255) / 256, s_max = splits;
            auto best_passes = [&](int tiles, int sc, double *cost) {
                int best = 0;
                for (int n = (tiles + 8) / 9; n <= tiles / 5 && n <= (tiles + 8) / 9 + 4; ++n) {      // no pass higher than nine, none below five
                    const int h = (tiles + n - 1) / n;
                    const int rounds = (n * cols * sc + 255) / 256;
                    const double c = rounds * ((0.0075 + 0.0016 * h) * K / sc + 6.0 + h);
                    if (best == 0 || c < *cost) {
                        best = n;
                        *cost = c;
                    }
                }
                return best;
            };
            const int t8 = (t + 7) / 8 * 8;
            double best = 0.0, cost = 0.0;
            for (int c = 1; c <= s_max; ++c) {
                const int sc = fit(c);
                if (c > 1 && sc == fit(c - 1)) continue;
                (void)best_passes(t8, sc, &cost);
                cost += sc * (32.0 * t8) * N * 1.67e-6;
                if (c == 1 || cost < best) {
                    best = cost;
                    splits = sc;
                }
            }
            p.m_chunks = best_passes(t, splits, &cost);
            p.mt = (t + p.m_chunks - 1) / p.m_chunks;
            p.splits = splits;
            return p;
        }
        // The LM head of up to nine row tiles: the many-row kernel with five column tiles per workgroup, all rows in one pass.  Up to
        // five row tiles two workgroups share a compute unit, beyond that one: 160-column blocks must then fill their last round
        // of 256 (151936 columns: 950 blocks, 93 %; 65536: 410, 80 %).  At nine row tiles and long K what a unit takes in decides,
        // and the two passes below take in less.  Step of one layer with and without logits, kernels below -> this, 151936 x
        // 4096 at 42 / 72 / 132 / 182 / 210 / 240 / 272 rows: 398 -> 331, 424 -> 346, 483 -> 406, 513 -> 487, 549 -> 534, 580 -> 560, 602 ->
        // 620 us, with logits 420 -> 377, 448 -> 398, 508 -> 459, 534 -> 508, 569 -> 548, 617 -> 575, 661 -> 656; x 1536 225 -> 160, 245 ->
        // 170, 271 -> 200, 289 -> 245, 306 -> 261, 307 -> 275, 319 -> 296; 65536 x 4096 254 -> 235, 266 -> 248, 301 -> 288, 331 -> 335, 356 ->
        // 359, 372 -> 388, 390 -> 423.  Where the last round is as empty as it can be, up to five row tiles, in a step of three layers
        // without / with logits: 82000 x 4096 (513 blocks) at 42 / 72 / 132 / 156 rows 503 -> 488 / 503 -> 492, 534 -> 511 / 547 -> 529, 620 -> 602
        // / 632 -> 625, 626 -> 609 / 640 -> 635, 128256 x 4096 (802) 561 -> 542 / 565 -> 559 to 695 -> 672 / 725 -> 719, 82000 x 1536 265 ->
        // 264 / 281 -> 281 to 332 -> 322 / 347 -> 340: still no loss.  65536 x 1536 at 42 rows is 1 to 3 % behind in a model of three
        // layers, whose weights the memory-side cache keeps in part if they are loaded plainly (with plain loads even); with twelve and 28
        // layers ahead, 812 -> 792 and 1849 -> 1805 us.
        // (Asked for over and over with nothing between, 182 rows and more lose, 256 x 151936 x 4096 341 -> 381 us; in the steps around
        // them, 8B with four layers, they gain: 182 / 210 / 240 rows 967 -> 940, 1051 -> 1039, 1100 -> 1101.)
        const int vocab_blocks = (N + 159) / 160, vocab_rounds = (vocab_blocks + 255) / 256;
        if (force_single_split && wgs >= 512 &&
            (t <= 5 || (10 * vocab_blocks >= 9 * 256 * vocab_rounds && (t <= 8 || (t == 9 && K <= 2048))))) {
            p.wide = 3;
            p.nt = 5;
            p.mt = t;
            p.m_chunks = 1;
            p.splits = 1;
            return p;
        }
        const bool row_split = !force_single_split && wgs * splits <= 128;
        const int t32 = (N + 31) / 32;
        // kernels_gemm_tall.hip: all row tiles (up to twelve) in one workgroup, both operands by LDS-DMA.  It adds the products of a
        // row in the same order as the kernels below (one 16x16x32 MFMA for two 32x32x16 of theirs: the same bits,
        // tests/test_gpu_row_class.py), so the choice may follow the row count.  It needs most of the compute units at one
        // workgroup each and a share of K that is long against its ring fill.  Kernels below -> it, weights from HBM, activations
        // just written:
        //   * wide single splits, three column tiles per workgroup (gate/up): the weights are read once, by every unit.  40 / 72 /
        //     132 / 216 / 272 rows: 24576 x 4096 37.9 -> 32.6, 46.5 -> 37.0, 54.3 -> 43.0, 56.6 -> 49.9, 64.2 -> 54.7 us; 17920 x 1536
        //     15.8 -> 12.1, 18.8 -> 13.8, 22.5 -> 16.0, 23.3 -> 18.9, 25.5 -> 20.7 (to nine row tiles; 340 rows 29.1 -> 25.4, but 384
        //     27.7 -> 28.0 and 440 29.0 -> 36.0).  From eleven on only where 256-column workgroups do not fit one round any more:
        //     340 / 440 x 24576 x 4096 125.8 -> 62.9, 136.6 -> 87.6.  More than 256 workgroups: the second round is ragged and
        //     loses, 72 / 272 x 28672 x 4096 46.0 -> 62.6, 69.6 -> 97.4.
        //   * two column tiles where K is cut into many short shares (the small model's down): 72 / 132 / 216 / 272 / 300 x 1536 x 8960
        //     10.9 -> 9.8, 12.7 -> 12.5, 15.7 -> 15.6, 18.0 -> 17.5, 18.6 -> 18.7, but 192 13.9 -> 15.1 and 256 16.5 -> 16.9: two passes
        //     of three and of four row tiles are an even deal.  (With both kernels as they were when the line was drawn 272 rows read 20.8
        //     -> 17.5.)  With fewer splits up to three row tiles, shares from 2048 k on: 72 x 4096 x 12288 26.0 -> 21.5, 72 x 3072 x
        //     8192 17.0 -> 14.1, 72 x 6144 x 4096 16.5 -> 14.3.  Higher it is ahead here (272 x 4096 x 12288 38.9 -> 37.5, x 6144 x 4096
        //     25.5 -> 24.1) but was not inside a step, where QKV, O and down of the 8B shape at 272 and 216 rows read 25.9 -> 29.6,
        //     18.8 -> 18.6, 37.6 -> 39.3 us.
        // Where column blocks x splits is a multiple of eight, many short shares come here from seven row tiles on only.  The line is
        // older than the numbering of the two-pass workgroups: their passes shared weights in an XCD's L2 at those counts alone, and
        // do now at all of them.  With the kernels as they are it gives away what this one gains up to five row tiles, at 40 / 96 / 160 /
        // 192 / 216 / 256 / 272 rows 1536 x 8192 9.1 -> 8.0, 10.2 -> 9.2, 12.3 -> 11.2, 12.9 -> 12.5, 15.2 -> 13.6, 15.3 -> 14.7, 17.0 ->
        // 15.4, and keeps what it loses at six: 2560 x 6144 9.7 -> 8.6, 11.2 -> 10.3, 12.7 -> 12.3, 13.6 -> 14.4, 15.4 -> 15.2, 15.9 ->
        // 16.4, 17.3 -> 17.1; 3072 x 5120 9.7 -> 8.8, 11.0 -> 10.3, 12.7 -> 12.8, 13.4 -> 15.1, 15.4 -> 15.7, 15.9 -> 16.8, 17.4 -> 17.5.
        // Another count, 1536 x 9216: 9.7 -> 8.7, 11.2 -> 10.3, 13.1 -> 13.1, 14.0 -> 14.7, 15.7 -> 15.7, 16.7 -> 17.1, 18.1 -> 17.7.
        int ct = 0;
        if (!force_single_split) {
            const int share = splits == 1 ? K : (units + splits - 1) / splits * SPLIT_UNIT;
            const bool short_shares = splits >= 5 && share <= 1024;
            const int t_min = short_shares && wgs * splits % 8 == 0 ? 7 : 1;
            const int t_max = short_shares ? 10 : splits > 1 && share >= 2048 ? 3 : 0;
            if (row_split && t >= t_min && t <= t_max) ct = 2;
            if (splits == 1 && wgs > 128 && (t <= 9 || (N + 255) / 256 * ((t + 4) / 5) > 256)) ct = 3;
            const int n = ct ? (t32 + ct - 1) / ct * splits : 0;
            if (share < 1024 || n < 180 || n > 256) ct = 0;
        }
        if (ct) {
            p.wide = 2;
            p.nt = ct;
            p.splits = splits;
            p.m_chunks = (t + 11) / 12;
            p.mt = (t + p.m_chunks - 1) / p.m_chunks;
            return p;
        }
        const int per_pass = row_split ? (t + 1) / 2 : t;
        p.mt = per_pass <= 2 ? 1 : per_pass <= 4 ? 2 : per_pass <= 6 ? 3 : 5;      // per wave (wide kernel)
        int ctl = p.mt == 5 ? 9 : 2 * p.mt;
        // Two row passes of three to five tiles (129-320 rows): the four waves side by side, each over all row tiles of
        // the pass and one 32-column tile of the workgroup's 128 columns - at 272 rows five MFMAs per wave and k step
        // where the 2 x 2 arrangement runs six (two passes of six tile slots for nine tiles), and no weight fragment
        // is loaded twice
        if (row_split) {
            p.wide = 1;
            p.nt = 1;
            p.mt = per_pass;
            ctl = per_pass;
        }
        // many column blocks, one split, more than five row tiles: 256-column workgroups over five row tiles
        // (four waves side by side, no weight fragment loaded twice) in two or more row passes.  Only when the
        // whole grid is resident at once: the passes of a column block then run together and the second read
        // of its weights hits L2 (measured on the LM head, whose grid takes several rounds: 30 % slower in
        // plain launch order)
        const int wide_wgs = ((N + 255) / 256) * ((t + 4) / 5);
        if (splits == 1 && wgs >= 128 && (t == 6 || t == 7)) {
            // Six or seven row tiles, one split, many column blocks (gate/up and the LM head at 161-224 rows): one
            // row pass of 128-column workgroups, every wave over all row tiles and one column tile - t MFMAs per
            // wave and k step where two passes of five tile slots ran ten, the weights read once.  Measured per
            // GEMM: -12 % at six tiles, -10 % at seven, nothing at eight, +5 % at nine (a workgroup then stages all
            // of A for half as many columns), so from eight tiles on the two passes stay.
            p.wide = 1;
            p.nt = 1;
            p.mt = t;
            ctl = t;
        } else if (splits == 1 && wgs >= 128 && t > 5 && wide_wgs <= 256) {
            p.wide = 1;
            p.nt = 1;
            p.nw = 8;
            p.mt = 5;
            ctl = 5;
        } else if (splits == 1 && wgs >= 512 && t > 5) {
            // The LM head: its grid takes several rounds either way.  With the (row pass, column block) plane
            // dealt to the XCDs in super-tiles the passes of a column block run on one XCD at about the same
            // time and share the weights through its L2: 436 -> 402 us at 272 rows.
            p.wide = 1;
            p.nt = 1;
            p.nw = 8;
            p.mt = 5;
            ctl = 5;
            p.swz = 4;
        }
        p.m_chunks = (t + ctl - 1) / ctl;
    }
    p.splits = splits;
    return p;
}

void launch_gemm_bf16(const bf16_t *a, const bf16_t *w, float *out, int M, int N, int K, const GemmPlan &p,
                      int out_row_major, hipStream_t st, const ChooseArgs *choose) {
    ChooseArgs ch = {};
    if (choose && out_row_major == GEMM_EPI_ARGMAX) ch = *choose;
    if (p.wide == 2) {
        launch_gemm_bf16_tall(a, w, out, M, N, K, p, out_row_major, st);
    } else if (p.wide == 3) {
        launch_gemm_bf16_vocab(a, w, out, M, N, K, p, out_row_major, st, ch);
    } else if (p.rows) {
        launch_gemm_bf16_rows(a, w, out, M, N, K, p, out_row_major, st, ch);
    } else if (p.mid && (out_row_major == GEMM_EPI_TILED || out_row_major == GEMM_EPI_SWIGLU)) {
        launch_gemm_bf16_mid(a, w, out, M, N, K, p, out_row_major == GEMM_EPI_SWIGLU, st);
    } else if (p.mid) {        // no vocabulary epilogue there: those take a single split
        launch_gemm_bf16(a, w, out, M, N, K, plan_gemm_bf16(M, N, K, true), out_row_major, st, choose);
    } else if (M <= 32) {
        // Two column tiles per workgroup where partial sums of a narrow product leave compute units idle otherwise, four where there
        // are enough of them (and for the epilogues that need gate and up, or a column group, in one wave).  Four / two at 6 rows:
        // 2048 x 1536 5.2 / 4.3 us, 1536 x 8960 7.9 / 7.2, 4096 x 12288 22.3 / 21.2, 4096 x 4096 9.4 / 9.3, 6144 x 4096 11.5 / 12.4.
        // Wider, where 64-column blocks have room for two splits only: 6016 x 12288 25.8 / 32.6, 5760 x 4096 10.5 / 12.4, 6656 x 8192
        // 20.3 / 21.2, 7424 x 8192 21.6 / 21.2, 8064 x 4096 14.5 / 14.0, 8192 x 8192 28.2 / 24.2 (20 rows 29.0 / 25.6).
        const bool two = out_row_major == GEMM_EPI_TILED && few_rows_two(N);
        if (p.mt == 1 && two) launch_few<1, 2>(a, w, out, M, N, K, p, out_row_major, st, ch);
        else if (p.mt == 1) launch_few<1, 4>(a, w, out, M, N, K, p, out_row_major, st, ch);
        else if (two) launch_few<2, 2>(a, w, out, M, N, K, p, out_row_major, st, ch);
        else launch_few<2, 4>(a, w, out, M, N, K, p, out_row_major, st, ch);
    } else if (p.wide && p.nt == 1 && p.nw == 8) {     // eight waves side by side, one column tile each
        launch_large<5, true, 1, 8>(a, w, out, M, N, K, p, out_row_major, st, ch);
    } else if (p.wide && p.nt == 1 && p.mt == 1) {
        launch_side<1>(a, w, out, M, N, K, p, out_row_major, st, ch);
    } else if (p.wide && p.nt == 1 && p.mt == 2) {
        launch_side<2>(a, w, out, M, N, K, p, out_row_major, st, ch);
    } else if (p.wide && p.nt == 1 && p.mt == 3) {
        launch_side<3>(a, w, out, M, N, K, p, out_row_major, st, ch);
    } else if (p.wide && p.nt == 1 && p.mt == 4) {
        launch_side<4>(a, w, out, M, N, K, p, out_row_major, st, ch);
    } else if (p.wide && p.nt == 1 && p.mt == 5) {
        launch_side<5>(a, w, out, M, N, K, p, out_row_major, st, ch);
    } else if (p.wide && p.nt == 1 && p.mt == 6) {
        launch_side<6>(a, w, out, M, N, K, p, out_row_major, st, ch);
    } else if (p.wide && p.nt == 1 && p.mt == 7) {
        launch_side<7>(a, w, out, M, N, K, p, out_row_major, st, ch);
    } else if (p.wide && p.nt == 1) {
        launch_side<8>(a, w, out, M, N, K, p, out_row_major, st, ch);
    } else if (p.mt == 1) {
        launch_large<1, false>(a, w, out, M, N, K, p, out_row_major, st, ch);
    } else if (p.mt == 2) {
        launch_large<2, false>(a, w, out, M, N, K, p, out_row_major, st, ch);
    } else if (p.mt == 3) {
        launch_large<3, false>(a, w, out, M, N, K, p, out_row_major, st, ch);
    } else {
        launch_large<5, false>(a, w, out, M, N, K, p, out_row_major, st, ch);
    }
}
