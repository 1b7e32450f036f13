// bf16 GEMM of many rows (large batches, prefill and scoring passes): out = A[M][K] x W[N][K]^T, fp32 accumulation,
// same operand layouts, epilogues and split-K rule as kernels_gemm.hip.
//
// Here every weight byte is used hundreds of times and the matrix cores decide - or rather the power they take: with
// all of them busy the clock settles far below its limit (the same launch on zeros is a quarter faster), so a
// variant that spends less energy per product is faster even where it issues no faster.  Hence 16x16x32 MFMAs, and
// as few LDS reads per MFMA as the registers allow: a workgroup of four waves, one per SIMD, owns up to nine row
// tiles x 8 column tiles of 32, a wave one half of every row tile x 4 column tiles (up to 288 accumulator registers,
// 17 fragment reads per 72 MFMAs).
// Both operands go from memory straight into LDS (buffer_load ... lds): they are stored as 32x32x16 register images,
// and a 16x16x32 fragment is four contiguous 256-byte runs of two of those, so every read is conflict-free.
// LDS holds four chunks of K = 32; a chunk's loads are issued more than three chunks (3000 cycles) before they are
// needed.  With one wave per SIMD nothing else covers a stall, so everything is spread between the MFMAs: fragments
// of the next chunk and the loads of the chunk after the next three go out one at a time, each behind an MFMA of its own
// (an MFMA occupies the matrix core for 16 cycles, the three or four operations of a row in one lump take longer: 8B step of
// 8 sequences 40855 -> 40188 us, scoring of 2000 tokens (1.5B) 17192 -> 16859), and after the one barrier of a chunk there
// are always fragments in registers to go on with.
// The row passes of a launch are equally high, or differ by one row tile (the plan picks their number).
// Measured against four waves of 256 x 64 with 32x32x16 MFMAs, weights in a register ring: 2176 x 24576 x 4096 440 -> 339
// us (1.29 PFLOP/s), 2176 x 4096 x 12288 220 -> 165, 4000 x 17920 x 1536 248 -> 203; 23 instead of 25 ns per k of a
// 256 x 256 tile with every compute unit busy, 18 on zeros.
#include <type_traits>

#include "gemm_device.h"
#include "lds_dma.h"

namespace {

constexpr int BUFS = 4;                           // chunks in LDS

// RT: row tiles of the higher passes; the first n_tall of the n_pass passes have RT row tiles, the others RT - 1.
// CB: column tiles of 32 of a workgroup.  Eight; or five for the LM head of a few row tiles, in one pass: less of a last round that
// is nearly empty, weights that nobody else reads (non-temporal), up to five row tiles two workgroups per compute unit (figures at
// the rule in plan_gemm_bf16).
template <int RT, int EPI, int CB>
__global__ __launch_bounds__(256) void gemm_bf16_rows_kernel(const bf16_t *__restrict__ a, const bf16_t *__restrict__ w,
                                                             float *__restrict__ out, int M, int N, int K, int splits,
                                                             int n_pass, int n_tall, int n_colblk, ChooseArgs ch) {
    constexpr int CT = CB;                             // 16-column tiles of a wave
    constexpr int LOADS = RT > CB ? RT : CB;           // loads of a wave and chunk, at most
    constexpr int CHUNK = 4 * LOADS * 1024;            // A [k step][row tile], then W [k step][column tile], 1 KiB each
    extern __shared__ __attribute__((aligned(16))) unsigned char rows_smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mh = wave >> 1, ng = wave & 1;
    const int t32 = (N + 31) >> 5, m_tiles = (M + 31) >> 5;

    // Workgroup i of a launch runs on XCD i % 8.  Each XCD takes one contiguous eighth of the (row pass, column block)
    // plane, four column blocks wide and passes downwards, so that what is resident on it together shares A rows
    // and W columns through its L2.
    int bx, bz;
    {
        const int n_wg = n_pass * n_colblk, q = n_wg >> 3, r = n_wg & 7, x = blockIdx.x & 7;
        const int i = x * q + min(x, r) + (blockIdx.x >> 3), band = 4 * n_pass;
        const int g = i / band, o = i - g * band, wd = min(4, n_colblk - 4 * g);
        bz = o / wd;
        bx = 4 * g + o - bz * wd;
    }
    const int mt_base = bz * (RT - 1) + min(bz, n_tall), ct_here = bz < n_tall ? RT : RT - 1;
    const SplitRange sr = split_range(K, splits, blockIdx.y);
    const int n_chunks = max(sr.q1 - sr.q0, 0);                 // one chunk = 32 k

    // loads: waves 0 and 1 bring the W tiles of the chunk's two k steps, waves 2 and 3 the A tiles
    const bool ld_w = wave < 2;
    const int ld_tiles = ld_w ? t32 : m_tiles, ld_t0 = ld_w ? bx * CB : mt_base;
    const int ld_here = ld_w ? min(CB, t32 - bx * CB) : ct_here;
    const int4v ld_desc = raw_desc(ld_w ? w : a, (size_t)(K >> 4) * ld_tiles * 1024);
    const unsigned ld_dst = lds_address(rows_smem) + ((ld_w ? 2 : 0) + (wave & 1)) * LOADS * 1024;
    const int ld_src = ((sr.q0 * 2 + (wave & 1)) * ld_tiles + ld_t0) * 1024, ld_step = 2 * ld_tiles * 1024;
    int ld_off[LOADS];
#pragma unroll
    for (int i = 0; i < LOADS; ++i) ld_off[i] = i < ld_here ? lane * 16 : OOB;
    // Tiles that do not exist and chunks past the last are asked for too, out of bounds: no traffic, and the number
    // of loads in flight is the same for every wave and chunk
    // (a chunk past the last by a buffer without records).  Four tiles side by side share their base addresses: what a
    // load needs of scalar work is as much in the way of the MFMAs as the load itself (with addresses of their own, a
    // select per load and per tile: 8B step of 8 sequences 38831 us, now 37910; 4096-token prefill 57191, 55564; scoring of
    // 2000 tokens (1.5B) 16168, 15727).
    auto load = [&](int c, int i) __attribute__((always_inline)) {
        const unsigned dst = ld_dst + (c & (BUFS - 1)) * CHUNK;
        if constexpr (CB == 8) dma16_tile(dst, ld_off[i], ld_desc, c < n_chunks, ld_src + c * ld_step, i);
        else if (!ld_w) {                              // a wave asks for its tiles only, and weights are read once
            if (i < RT) dma16_tile(dst, ld_off[i], ld_desc, c < n_chunks, ld_src + c * ld_step, i);
        } else if (i < CB) dma16_tile<true>(dst, ld_off[i], ld_desc, c < n_chunks, ld_src + c * ld_step, i);
    };
    auto wait_chunks = [&](auto n) __attribute__((always_inline)) {      // until no more than the last n chunks are in flight
        if constexpr (CB == 8) wait_loads<n * LOADS>();
        else if (ld_w) wait_loads<n * CB>();
        else wait_loads<n * RT>();
    };

    // The wave's row tile i (16 rows) is half mh of the pass's 32-row tile i.
    f32x4 acc[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    bf16x8 af[2][RT], wf[2][CT];
    // lane (n, g) of a 16x16x32 fragment takes k slots 8g .. 8g+7 of row n: stored k step g/2, stored lane (g%2)*32 + n
    const unsigned char *frag0 = rows_smem + (lane >> 5) * LOADS * 1024 + ((lane >> 4) & 1) * 512 + (lane & 15) * 16;
    // the wave's even and odd 16-column tiles, CT from ng * CT on (of eight, halves of the tiles ng * 4 and on)
    const int w_frag[2] = {(ng * CT >> 1) * 1024 + (ng * CT & 1) * 256, ((ng * CT + 1) >> 1) * 1024 + ((ng * CT + 1) & 1) * 256};
    auto read = [&](int s, int c, int f) __attribute__((always_inline)) {      // W fragments first: all of them are
        const unsigned char *b = frag0 + (c & (BUFS - 1)) * CHUNK;             // needed before the second A fragment
        if (f < CT && CT == 8) wf[s][f] = *(const bf16x8 *)(b + (2 * LOADS + ng * 4 + (f >> 1)) * 1024 + (f & 1) * 256);
        else if (f < CT) wf[s][f] = *(const bf16x8 *)(b + 2 * LOADS * 1024 + w_frag[f & 1] + (f >> 1) * 1024);
        else af[s][f - CT] = *(const bf16x8 *)(b + (f - CT) * 1024 + mh * 256);
    };

#pragma unroll
    for (int c = 0; c < BUFS; ++c)
#pragma unroll
        for (int i = 0; i < LOADS; ++i) load(c, i);
    wait_chunks(std::integral_constant<int, BUFS - 1>());
    lds_barrier_counted();
    // the k loop over RA row tiles
    auto k_loop = [&](auto ra_tag) __attribute__((always_inline)) {
        constexpr int RA = decltype(ra_tag)::value, READS = CT + RA;
        // a row of MFMAs with the n operations op(0 .. n-1) one by one between them
        auto row = [&](int s, int i, int n, auto op) __attribute__((always_inline)) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < CT; ++j) {
                // The ninth row's accumulators do not fit the 256 AGPRs any more; left to the compiler, which wants
                // all of them there, they are copied in and out around every use.  (The wait that their reader needs
                // stands behind the loop and names them.)
                if (i == 8 && CT == 8)
                    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc[i][j]) : "v"(wf[s][j]), "v"(af[s][i]));
                else
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[s][j], af[s][i], acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k = (n * j + CT - 1) / CT; k < (n * (j + 1) + CT - 1) / CT; ++k) op(k);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        auto chunk = [&](int s, int c) __attribute__((always_inline)) {
            row(s, 0, 0, [](int) {});
            wait_chunks(std::integral_constant<int, BUFS - 2>());
            lds_barrier_counted();                       // chunk c+1 has landed for everyone, chunk c has been read by everyone
#pragma unroll
            for (int i = 1; i < RA; ++i) {
                const int f0 = READS * (i - 1) / (RA - 1), nf = READS * i / (RA - 1) - f0;
                const int l0 = LOADS * (i - 1) / (RA - 1), nl = LOADS * i / (RA - 1) - l0;
                row(s, i, nf + nl, [&](int k) __attribute__((always_inline)) {
                    if (k < nf) read(s ^ 1, c + 1, f0 + k);
                    else load(c + BUFS, l0 + k - nf);
                });
            }
        };
#pragma unroll
        for (int f = 0; f < READS; ++f) read(0, 0, f);
        // two chunks at a time (the fragment sets alternate); an odd one at the end runs with a chunk of zeros, so
        // that the loop stays one piece of code and the accumulators stay where they are
        for (int c = 0, end = n_chunks & ~1;; end += 2) {
            for (; c < end; c += 2) {
                chunk(0, c);
                chunk(1, c + 1);
            }
            if (end >= n_chunks) break;
            bf16x8 *z = reinterpret_cast<bf16x8 *>(rows_smem + (n_chunks & (BUFS - 1)) * CHUNK);
#pragma unroll
            for (int i = 0; i < CHUNK / 4096; ++i) z[threadIdx.x + 256 * i] = (bf16x8){0, 0, 0, 0, 0, 0, 0, 0};
        }
        // The compiler does not see the ninth row's MFMAs finish: the wait (32 states; the longest MFMA asks for
        // fewer than 20 before its result is read) takes their results in and hands them on, so no use comes before it
        if constexpr (RA == 9 && CT == 8)
            asm volatile("s_nop 15\n\ts_nop 15" : "+v"(acc[8][0]), "+v"(acc[8][1]), "+v"(acc[8][2]), "+v"(acc[8][3]),
                         "+v"(acc[8][4]), "+v"(acc[8][5]), "+v"(acc[8][6]), "+v"(acc[8][7]));
    };
    if constexpr (CB < 8) k_loop(std::integral_constant<int, RT>());      // a single pass
    else if (ct_here == RT) k_loop(std::integral_constant<int, RT>());
    else k_loop(std::integral_constant<int, RT - 1>());
    wait_loads<0>();
    lds_barrier_counted();

    // ---- epilogue
    const int n = lane & 15, g = lane >> 4;
    const int col_w = bx * 32 * CB + ng * 16 * CT;                       // the wave's first column
    auto row_of = [&](int i) { return (mt_base + i) * 32 + mh * 16; };
    auto exists = [&](int i) { return i < RT - 1 || ct_here == RT; };
    if constexpr (EPI == GEMM_EPI_SWIGLU) {
        // tile 2j: gate, tile 2j + 1: up, of the same 16 features; a lane's four are half of a 16-byte piece of the
        // next GEMM's A fragment
        typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
        bf16_t *ho = reinterpret_cast<bf16_t *>(out);
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            if (!exists(i)) continue;
#pragma unroll
            for (int j = 0; j < CT; j += 2) {
                const int tile = (col_w >> 5) + (j >> 1);
                bf16x4 h;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float gt = acc[i][j][e], u = acc[i][j + 1][e];
                    h[e] = (bf16_t)(gt * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * gt)) * u);
                }
                if (tile < t32)
                    *(bf16x4 *)(ho + (((size_t)tile * m_tiles + (row_of(i) >> 5)) * 64 + (g >> 1) * 32 + mh * 16 + n) * 8 +
                                (g & 1) * 4) = h;
            }
        }
    } else if constexpr (EPI == GEMM_EPI_ARGMAX) {
        // per row and group of PG column tiles (64 columns; the 80 of a wave where it has five): a lane walks its columns in
        // rising order (strict > keeps the lowest column of a tie), then the four lanes of a row are folded
        constexpr int P = CT == 8 ? 2 : 1, PG = CT / P;
        const int G = CT == 8 ? (t32 + 1) >> 1 : 2 * n_colblk;
        float *pmax = out;
        int *pidx = (int *)(out + (size_t)G * M);
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            if (!exists(i)) continue;
            const int row = row_of(i) + n;
            float best[P];
            int bi[P];
#pragma unroll
            for (int p = 0; p < P; ++p) {
                best[p] = -INFINITY;
                bi[p] = col_w + 16 * PG * p + 4 * g;
            }
            const RowChoice rc = row_choice(ch, row, M);
            if (__any(rc.noisy || rc.sel >= 0)) {            // wave-uniform: rows a token is taken from.  Few of them:
                // a loop over values the lane parks in LDS (the staging buffers are free) instead of unrolled code
                f32x4 *park = reinterpret_cast<f32x4 *>(rows_smem) + threadIdx.x;
#pragma unroll
                for (int j = 0; j < CT; ++j) park[256 * j] = acc[i][j];
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll 1
                    for (int t = 0; t < 4 * PG; ++t) {
                        const int col = col_w + 16 * PG * p + 16 * (t >> 2) + 4 * g + (t & 3);
                        float v = reinterpret_cast<const float *>(park + 256 * (PG * p + (t >> 2)))[t & 3];
                        if (rc.sel >= 0 && col < N) ch.sel_logits[(size_t)rc.sel * N + col] = v;
                        if (rc.noisy) v = perturbed_logit(v, rc.inv_t, rc.key, (uint32_t)col);
                        if (col < N && v > best[p]) {
                            best[p] = v;
                            bi[p] = col;
                        }
                    }
            } else {
#pragma unroll
                for (int j = 0; j < CT; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int col = col_w + 16 * j + 4 * g + e;
                        if (col < N && acc[i][j][e] > best[j / PG]) {
                            best[j / PG] = acc[i][j][e];
                            bi[j / PG] = col;
                        }
                    }
            }
#pragma unroll
            for (int p = 0; p < P; ++p) {
#pragma unroll
                for (int o = 16; o < 64; o <<= 1) {
                    const float ob = __shfl_xor(best[p], o);
                    const int oi = __shfl_xor(bi[p], o);
                    if (ob > best[p] || (ob == best[p] && oi < bi[p])) {
                        best[p] = ob;
                        bi[p] = oi;
                    }
                }
                const int group = (bx * 2 + ng) * P + p;
                if (g == 0 && row < M && group < G) {
                    pmax[(size_t)group * M + row] = best[p];
                    pidx[(size_t)group * M + row] = bi[p];
                }
            }
        }
    } else {
        float *o = out + (size_t)blockIdx.y * pt_split_stride(M, N);
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            if (!exists(i)) continue;
#pragma unroll
            for (int j = 0; j + 1 < CT; j += 2)
                store_pair<EPI == GEMM_EPI_ROWMAJOR>(acc[i][j], acc[i][j + 1], o, row_of(i), col_w + 16 * j, M, N, lane);
            if constexpr (CT & 1) {                    // (logits only)
                static_assert(EPI == GEMM_EPI_ROWMAJOR, "an odd number of column tiles");
                const int row = row_of(i) + n, col = col_w + 16 * (CT - 1) + 4 * g;
                if (row < M && col < N) *(f32x4 *)(o + (size_t)row * N + col) = acc[i][CT - 1];
            }
        }
    }
}

template <int RT, int EPI, int CB = 8>
void launch_rows(const bf16_t *a, const bf16_t *w, float *out, int M, int N, int K, const GemmPlan &p, hipStream_t st,
                 const ChooseArgs &ch) {
    constexpr int SMEM = BUFS * 4 * (RT > CB ? RT : CB) * 1024;
    const int n_colblk = (N + 32 * CB - 1) / (32 * CB), n_tall = (M + 31) / 32 - p.m_chunks * (RT - 1);
    static std::atomic<bool> granted[kLdsDevices];
    grant_lds((const void *)gemm_bf16_rows_kernel<RT, EPI, CB>, SMEM, granted);
    gemm_bf16_rows_kernel<RT, EPI, CB><<<dim3(p.m_chunks * n_colblk, p.splits), 256, SMEM, st>>>(
        a, w, out, M, N, K, p.splits, p.m_chunks, n_tall, n_colblk, ch);
}

template <int EPI>
void launch_rows_epi(const bf16_t *a, const bf16_t *w, float *out, int M, int N, int K, const GemmPlan &p, hipStream_t st,
                     const ChooseArgs &ch) {
    if (p.mt == 9) launch_rows<9, EPI>(a, w, out, M, N, K, p, st, ch);
    else if (p.mt == 8) launch_rows<8, EPI>(a, w, out, M, N, K, p, st, ch);
    else if (p.mt == 7) launch_rows<7, EPI>(a, w, out, M, N, K, p, st, ch);
    else launch_rows<6, EPI>(a, w, out, M, N, K, p, st, ch);
}

template <int EPI>
void launch_vocab(const bf16_t *a, const bf16_t *w, float *out, int M, int N, int K, const GemmPlan &p, hipStream_t st,
                  const ChooseArgs &ch) {
    if (p.mt <= 2) launch_rows<2, EPI, 5>(a, w, out, M, N, K, p, st, ch);
    else if (p.mt == 3) launch_rows<3, EPI, 5>(a, w, out, M, N, K, p, st, ch);
    else if (p.mt == 4) launch_rows<4, EPI, 5>(a, w, out, M, N, K, p, st, ch);
    else if (p.mt == 5) launch_rows<5, EPI, 5>(a, w, out, M, N, K, p, st, ch);
    else if (p.mt == 6) launch_rows<6, EPI, 5>(a, w, out, M, N, K, p, st, ch);
    else if (p.mt == 7) launch_rows<7, EPI, 5>(a, w, out, M, N, K, p, st, ch);
    else if (p.mt == 8) launch_rows<8, EPI, 5>(a, w, out, M, N, K, p, st, ch);
    else launch_rows<9, EPI, 5>(a, w, out, M, N, K, p, st, ch);
}

}  // namespace

void launch_gemm_bf16_vocab(const bf16_t *a, const bf16_t *w, float *out, int M, int N, int K, const GemmPlan &p, int epi,
                            hipStream_t st, const ChooseArgs &ch) {
    if (epi == GEMM_EPI_ARGMAX) launch_vocab<GEMM_EPI_ARGMAX>(a, w, out, M, N, K, p, st, ch);
    else launch_vocab<GEMM_EPI_ROWMAJOR>(a, w, out, M, N, K, p, st, ch);
}

void launch_gemm_bf16_rows(const bf16_t *a, const bf16_t *w, float *out, int M, int N, int K, const GemmPlan &p, int epi,
                           hipStream_t st, const ChooseArgs &ch) {
    if (epi == GEMM_EPI_SWIGLU) launch_rows_epi<GEMM_EPI_SWIGLU>(a, w, out, M, N, K, p, st, ch);
    else if (epi == GEMM_EPI_ARGMAX) launch_rows_epi<GEMM_EPI_ARGMAX>(a, w, out, M, N, K, p, st, ch);
    else if (epi == GEMM_EPI_ROWMAJOR) launch_rows_epi<GEMM_EPI_ROWMAJOR>(a, w, out, M, N, K, p, st, ch);
    else launch_rows_epi<GEMM_EPI_TILED>(a, w, out, M, N, K, p, st, ch);
}
