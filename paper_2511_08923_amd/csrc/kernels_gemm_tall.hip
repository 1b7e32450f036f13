// bf16 GEMM of 33 to 480 rows: out = A[M][K] x W[N][K]^T, fp32 accumulation, same operand layouts and epilogues as
// kernels_gemm.hip, and the same products added in the same order per output value (two 32x32x16 MFMAs and one 16x16x32 over the
// same 32 k give the same bits: tests/test_gpu_row_class.py), so that the results are the same bits.
//
// At these row counts the weights come from HBM once and the activations (the step's 272 rows: 2.2 MB at K = 4096) from L2
// into every workgroup.  What bounds it is how much a compute unit takes in: with weights from HBM among the loads about
// 58 GB/s, whatever the kernel and whichever waves bring which operand (272 x 24576 x 4096: loads alone 52 us, weights alone 33,
// activations alone 22; MFMAs and LDS reads alone 42), in the order asked for, which is why a deeper ring or fewer LDS
// reads change little beyond this:
//   * a workgroup owns all row tiles of the pass (up to twelve) and two or three column tiles, one workgroup per compute unit:
//     a pass reads no weight twice, all of them stream, by non-temporal loads (from 385 rows on there are two passes, whose
//     workgroups follow each other on one XCD: plain / non-temporal 396, 440, 480 x 24576 x 4096 89.3 / 90.0, 93.4 / 92.2, 98.1 / 100.2
//     us, x 22016 83.2 / 82.9, 86.6 / 85.2, 93.7 / 94.8);
//   * both operands go straight into LDS (buffer_load ... lds), PA chunks of 64 k of A and PW of W: the weights, which
//     are longer on their way, are asked for up to seven chunks ahead, two chunks at a time;
//   * 16x16x32 MFMAs, four waves as 2 x 2: a wave owns one half of every row tile and half of the columns, RT x CT tiles of 16 x
//     16, so that nine row tiles are an even deal (whole 32-row tiles dealt to four waves gave one of them three and the others
//     two); the fragments of the next half chunk and the loads are spread between the MFMAs, one barrier per chunk of 64 k.
// With 32x32x16 MFMAs, four waves over whole row tiles and plain loads gate/up read 58.7 us inside a step of 272 rows, now 57.5; 55.3
// and 52.7 at 216 rows (8B step k = 16 7835 -> 7740 us, 3 x k = 8 6910 -> 6860, 1.5B k = 16 2970 -> 2957).  The non-temporal loads'
// part, plain -> so, weights from HBM, activations just written: 40 / 132 / 272 x 24576 x 4096 34.9 -> 33.5, 44.1 -> 42.7, 59.8 -> 58.2,
// 132 / 272 x 17920 x 1536 17.0 -> 16.4, 22.5 -> 22.1, 72 / 272 x 1536 x 8960 10.2 -> 9.8, 18.1 -> 17.7, 72 x 4096 x 12288 23.8 -> 22.0.
// The accumulators are tied to AGPRs by inline assembly: left to the compiler they are copied between the register files
// around every use (85 instead of 63 us).
// Measured sizes stand at the rule in plan_gemm_bf16.
#include <type_traits>

#include "gemm_device.h"
#include "lds_dma.h"

namespace {

constexpr int LDS_KB = 160;
// LDS holds PA chunks of A and PW of W; a chunk is 64 k, a 32-row or 32-column tile's share of it 4 KiB
constexpr int a_chunks(int rt, int ct) {
    int p = 4;
    while (p > 2 && 4 * (p * rt + (p + 1) * ct) > LDS_KB) --p;
    return p;
}
constexpr int w_chunks(int rt, int ct) {
    int p = a_chunks(rt, ct) + 1;
    while (p < 8 && 4 * (a_chunks(rt, ct) * rt + (p + 1) * ct) <= LDS_KB) ++p;
    return p;
}

// f(LO), ..., f(HI - 1), each index a constant of the code (left to the unroller, the larger kernels stayed loops, with their
// fragments in scratch memory)
template <int LO, int HI, class F>
__device__ __attribute__((always_inline)) inline void each(F &&f) {
    if constexpr (LO < HI) {
        f(std::integral_constant<int, LO>());
        each<LO + 1, HI>(f);
    }
}

// RT: row tiles of the higher passes, CT: column tiles of a workgroup
template <int RT, int CT>
__global__ __launch_bounds__(256) void gemm_bf16_tall_kernel(const bf16_t *__restrict__ a, const bf16_t *__restrict__ w,
                                                             float *__restrict__ out, int M, int N, int K, int splits,
                                                             int epi, int n_pass, int n_tall) {
    constexpr int PA = a_chunks(RT, CT), PW = w_chunks(RT, CT);
    constexpr int A_CHUNK = 4 * RT * 1024, W_CHUNK = 4 * CT * 1024;
    static_assert(PA * A_CHUNK + PW * W_CHUNK <= LDS_KB * 1024, "LDS of a compute unit");
    static_assert(PW * CT + PA * RT < 62, "the loads in flight are counted in six bits");
    extern __shared__ __attribute__((aligned(16))) unsigned char tall_smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mh = wave >> 1, ng = wave & 1;
    const int t32 = (N + 31) >> 5, m_tiles = (M + 31) >> 5;
    const int j8 = blockIdx.x >> 3, unit = (j8 / n_pass) * 8 + (blockIdx.x & 7);
    const int bz = j8 % n_pass, split = unit % splits, tile0 = (unit / splits) * CT;
    if (tile0 >= t32) return;
    const int mt_base = bz * (RT - 1) + min(bz, n_tall), ct_here = bz < n_tall ? RT : RT - 1;
    const SplitRange sr = split_range(K, splits, split);
    const int n_steps = 2 * max(sr.q1 - sr.q0, 0), n_chunks = ((n_steps + 7) >> 3) * 2;      // steps of 16 k; an odd last chunk has one of zeros behind it

    // loads: a wave brings one of a chunk's four k steps, of A and of W.  Tiles that do not exist and steps past the last are
    // asked for too, out of bounds: no traffic, zeros in LDS, and the same number of loads in flight everywhere
    const int lane16 = lane * 16;
    const int4v da = raw_desc(a, (size_t)(K >> 4) * m_tiles * 1024), dw = raw_desc(w, (size_t)t32 * 32 * K * 2);
    const unsigned lds0 = lds_address(tall_smem), a_dst = lds0 + wave * RT * 1024, w_dst = lds0 + PA * A_CHUNK + wave * CT * 1024;
    const int a_src = ((sr.q0 * 2 + wave) * m_tiles + mt_base) * 1024, w_src = ((sr.q0 * 2 + wave) * t32 + tile0) * 1024;
    const int w_here = min(CT, t32 - tile0);
    // (steps past the last: a buffer without records).  Tiles side by side share their base addresses: what a load needs of
    // scalar work stands between the MFMAs as well (8B step k = 16 with addresses and selects per load 7884 us, now 7822;
    // 216 rows 6885, 6886).
    const int a_last = ct_here == RT ? lane16 : OOB;
    int w_off[CT];
#pragma unroll
    for (int j = 0; j < CT; ++j) w_off[j] = j < w_here ? lane16 : OOB;
    auto load_a = [&](int c, int buf, int i) __attribute__((always_inline)) {
        dma16_tile(a_dst + buf * A_CHUNK, i < RT - 1 ? lane16 : a_last, da, 4 * c + wave < n_steps, a_src + 4 * c * m_tiles * 1024, i);
    };
    auto load_w = [&](int c, int buf, int j) __attribute__((always_inline)) {
        dma16_tile<true>(w_dst + buf * W_CHUNK, w_off[j], dw, 4 * c + wave < n_steps, w_src + 4 * c * t32 * 1024, j);
    };
    auto next = [](int b, int n) { return b + 1 == n ? 0 : b + 1; };
    // The wave's row tile i (16 rows) is half mh of the pass's tile i.  Its column tiles (16 columns): the halves of column tile
    // ng and, of three, half ng of the third one.
    f32x4 acc[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    // Generation g of the loads goes out when chunk g has been read, one half in the second half of that chunk, the other in the
    // first half of the next.  It brings chunk g + PA of A and, if g is odd, before that the two chunks g + PW - 1 and g + PW of W:
    // a compute unit returns loads in the order they were asked for, so activations that lie in its L2 wait behind weights from HBM,
    // and the fewer times the two alternate the better (both operands' loads of 272 x 24576 x 4096 alone: weights one, two and
    // three chunks at a time 51.4, 46.6 and 44.4 us; three do not fit).  Weights chunk by chunk -> in pairs: gate/up at 216 rows
    // 52.4 -> 51.0 us, at 272 57.2 -> 57.0, 1.5B gate/up and down at 272 23.4 -> 22.5 and 18.6 -> 17.8; 3 x k = 8 6820 -> 6750, 1.5B k =
    // 16 2952 -> 2917, 8B k = 16 7700 -> 7665.
    // With two chunks of A (eleven and twelve row tiles) the next chunk's barrier waits for all of A: it goes out at once, and one
    // chunk of weights behind it (8B step of 330 / 364 rows in pairs 8570 / 8860 us, so 7990 / 8375).
    constexpr bool PAIRS = PA > 2;
    constexpr int N_LOADS[2] = {RT + (PAIRS ? 0 : CT), RT + (PAIRS ? 2 * CT : CT)};                 // even, odd generations
    constexpr int FIRST[2] = {N_LOADS[0] / (PAIRS ? 2 : 1), N_LOADS[1] / (PAIRS ? 2 : 1)};
    auto load = [&](int g, int odd, int ba, int bw_before, int bw, int l) __attribute__((always_inline)) {
        const int a = PAIRS && odd ? l - 2 * CT : l;           // tile of A
        if (a < 0) load_w(g + PW - 1 + l / CT, l < CT ? bw_before : bw, l % CT);
        else if (a < RT) load_a(g + PA, ba, a);
        else load_w(g + PW, bw, a - RT);
    };
    // what may be in flight when chunk g + 1 has to be there: the n = PA - 2 generations before g, and weights asked for behind A
    auto in_flight = [](int g, int n) constexpr {
        int s = PAIRS ? 0 : CT;
        for (int i = 1; i <= n; ++i) s += N_LOADS[(g - i) & 1];
        return s;
    };
    constexpr int W_FIRST = PAIRS ? PW - 2 * (PA / 2 + (PA & 1)) : PW - PA;      // chunks of W that generations before -PA have brought
    static_assert(W_FIRST >= 0, "W is asked for in pairs, PW - 1 and PW chunks ahead");
#pragma unroll
    for (int c = 0; c < W_FIRST; ++c)
#pragma unroll
        for (int j = 0; j < CT; ++j) load_w(c, c, j);
#pragma unroll
    for (int g = -PA; g < 0; ++g)
#pragma unroll
        for (int l = 0; l < (g < -1 ? N_LOADS[g & 1] : FIRST[1]); ++l) load(g, g & 1, g + PA, g + PW - 1, g + PW, l);
    wait_loads<in_flight(-1, PA - 2) + FIRST[1]>();
    lds_barrier_counted();
    // lane (n, g) of a 16x16x32 fragment takes k slots 8g .. 8g+7 of row n: stored k step g/2, stored lane (g%2)*32 + n
    const int frag = ((lane >> 4) & 1) * 512 + (lane & 15) * 16;
    const unsigned char *fa = tall_smem + (lane >> 5) * RT * 1024 + frag + mh * 256;
    const unsigned char *fw = tall_smem + PA * A_CHUNK + (lane >> 5) * CT * 1024 + frag;
    const unsigned char *fw01 = fw + ng * 1024, *fw2 = fw + 2 * 1024 + ng * 256;
    auto k_loop = [&](auto ra_tag) __attribute__((always_inline)) {
        constexpr int RA = decltype(ra_tag)::value, NM = RA * CT, READS = RA + CT;
        constexpr int B = NM >= 12 ? 3 : 1;           // MFMAs in front of the barrier
        bf16x8 af[2][RA], wf[2][CT];
        // fragments of half `half` of a chunk, in the order of use: W 0, A 0, the other W, the other A
        auto read = [&](int s, int half, int a_buf, int w_buf, int f) __attribute__((always_inline)) {
            const int ao = a_buf * A_CHUNK + half * 2 * RT * 1024, wo = w_buf * W_CHUNK + half * 2 * CT * 1024;
            const int j = f == 0 ? 0 : f - 1, i = f == 1 ? 0 : f - CT;
            if (f == 0 || (f > 1 && f <= CT)) wf[s][j] = *(const bf16x8 *)(j < 2 ? fw01 + wo + j * 256 : fw2 + wo);
            else af[s][i] = *(const bf16x8 *)(fa + ao + i * 1024);
        };
#pragma unroll
        for (int f = 0; f < READS; ++f) read(0, 0, 0, 0, f);
        // buffers of chunk c; of the generation under way
        int c = 0, ba = 0, bw = 0, ga = PA - 1, gw = PW - 1, gw_before = PW - 2;
        auto chunk = [&](auto odd_tag) __attribute__((always_inline)) {
            constexpr int ODD = decltype(odd_tag)::value;
            const int na = next(ba, PA), nw = next(bw, PW);
            each<0, 2>([&](auto q_tag) __attribute__((always_inline)) {
                constexpr int q = q_tag;
                if constexpr (q == 1) {
                    ga = ba;
                    gw_before = gw;
                    gw = bw;
                }
                constexpr int odd = q ? ODD : !ODD, l0 = q ? 0 : FIRST[odd], n_l = q ? FIRST[odd] : N_LOADS[odd] - FIRST[odd];
                each<0, NM>([&](auto m_tag) __attribute__((always_inline)) {
                    constexpr int m = m_tag;
                    if constexpr (q == 1 && m == B) {
                        wait_loads<in_flight(ODD, PA - 2)>();
                        lds_barrier_counted();           // chunk c+1 has landed for everyone, chunk c has been read by everyone
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    // The compiler does not see the MFMAs finish, and where the loop ends it may copy their results at once, so
                    // the last one of the last chunk brings the wait (32 states; it asks for fewer than 20 before its result is
                    // read) in the same piece of assembly
                    if constexpr (ODD && q == 1 && m == NM - 1)
                        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\t"
                                     "s_cmp_lg_i32 %3, %4\n\ts_cbranch_scc1 .Lmore%=\n\ts_nop 15\n\ts_nop 15\n.Lmore%=:"
                                     : "+a"(acc[m / CT][m % CT])
                                     : "v"(wf[q][m % CT]), "v"(af[q][m / CT]), "s"(c + 1), "s"(n_chunks)
                                     : "scc");
                    else
                        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
                                     : "+a"(acc[m / CT][m % CT])
                                     : "v"(wf[q][m % CT]), "v"(af[q][m / CT]));
                    __builtin_amdgcn_sched_barrier(0);
                    constexpr int x = q ? m - B : m, n = q ? NM - B : NM;        // reads and loads behind this MFMA
                    if constexpr (x >= 0) {
                        each<READS * x / n, READS * (x + 1) / n>([&](auto f) __attribute__((always_inline)) {
                            read(q ^ 1, q ^ 1, q ? na : ba, q ? nw : bw, f);
                        });
                        each<l0 + n_l * x / n, l0 + n_l * (x + 1) / n>([&](auto l) __attribute__((always_inline)) {
                            load(q ? c : c - 1, odd, ga, gw_before, gw, l);
                        });
                    }
                });
            });
            ba = na;
            bw = nw;
            ++c;
        };
        while (c < n_chunks) {
            chunk(std::integral_constant<int, 0>());
            chunk(std::integral_constant<int, 1>());
        }
    };
    const bool last_here = ct_here == RT && (mt_base + RT - 1) * 32 + mh * 16 < M;
    if (last_here) k_loop(std::integral_constant<int, RT>());
    else k_loop(std::integral_constant<int, RT - 1>());
    wait_loads<0>();
    lds_barrier_counted();

    // ---- epilogue: lane (n, g) holds activation row n and weight columns 4g .. 4g+3 of each 16 x 16 tile
    const int n = lane & 15, g = lane >> 4;
    auto row_of = [&](int i) { return (mt_base + i) * 32 + mh * 16; };
    auto exists = [&](int i) { return i < RT - 1 || last_here; };
    if (epi == GEMM_EPI_SWIGLU) {
        // The halves of a column tile are gate and up of the same 16 features; a lane's four are half of a 16-byte piece of the
        // next GEMM's A fragment.  Of the third column tile one wave has the gates, its neighbour the ups: they trade, and each
        // finishes every other row tile.
        bf16_t *ho = reinterpret_cast<bf16_t *>(out);
        auto put = [&](int i, int tile, const f32x4 &gt, const f32x4 &up) __attribute__((always_inline)) {
            typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
            bf16x4 h;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                h[e] = (bf16_t)(gt[e] * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * gt[e])) * up[e]);
            if (tile < t32 && exists(i))
                *(bf16x4 *)(ho + (((size_t)tile * m_tiles + mt_base + i) * 64 + (g >> 1) * 32 + mh * 16 + n) * 8 + (g & 1) * 4) = h;
        };
        f32x4 *trade = reinterpret_cast<f32x4 *>(tall_smem) + mh * RT * 64 + lane;
        if constexpr (CT == 3) {
#pragma unroll
            for (int i = 0; i < RT; ++i)
                if ((i & 1) != ng) trade[i * 64] = acc[i][2];
            lds_barrier_counted();
        }
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            put(i, tile0 + ng, acc[i][0], acc[i][1]);
            if constexpr (CT == 3)
                if ((i & 1) == ng) {
                    const f32x4 other = trade[i * 64];
                    put(i, tile0 + 2, ng ? other : acc[i][2], ng ? acc[i][2] : other);
                }
        }
        return;
    }
    float *o = out + (size_t)split * pt_split_stride(M, N);
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        if (!exists(i)) continue;
        const int col = (tile0 + ng) * 32, col2 = (tile0 + 2) * 32 + ng * 16 + 4 * g, row = row_of(i) + n;
        store_pair<false>(acc[i][0], acc[i][1], o, row_of(i), col, M, N, lane);
        if constexpr (CT == 3)
            if (row < M && col2 < N) *(f32x4 *)(o + pt_index(col2, row, M)) = acc[i][2];
    }
}

template <int RT, int CT>
void launch_tall(const bf16_t *a, const bf16_t *w, float *out, int M, int N, int K, const GemmPlan &p, int epi, hipStream_t st) {
    constexpr int SMEM = 4 * 1024 * (a_chunks(RT, CT) * RT + w_chunks(RT, CT) * CT);
    static_assert(SMEM >= 2 * RT * 1024, "the epilogue's trade");
    const int units = ((N + 31) / 32 + CT - 1) / CT * p.splits, n_tall = (M + 31) / 32 - p.m_chunks * (RT - 1);
    static std::atomic<bool> granted[kLdsDevices];
    grant_lds((const void *)gemm_bf16_tall_kernel<RT, CT>, SMEM, granted);
    gemm_bf16_tall_kernel<RT, CT><<<dim3((units + 7) / 8 * 8 * p.m_chunks), 256, SMEM, st>>>(
        a, w, out, M, N, K, p.splits, epi, p.m_chunks, n_tall);
}

template <int CT>
void launch_tall_rows(const bf16_t *a, const bf16_t *w, float *out, int M, int N, int K, const GemmPlan &p, int epi, hipStream_t st) {
    if (p.mt <= 2) launch_tall<2, CT>(a, w, out, M, N, K, p, epi, st);
    else if (p.mt == 3) launch_tall<3, CT>(a, w, out, M, N, K, p, epi, st);
    else if (p.mt == 4) launch_tall<4, CT>(a, w, out, M, N, K, p, epi, st);
    else if (p.mt == 5) launch_tall<5, CT>(a, w, out, M, N, K, p, epi, st);
    else if (p.mt == 6) launch_tall<6, CT>(a, w, out, M, N, K, p, epi, st);
    else if (p.mt == 7) launch_tall<7, CT>(a, w, out, M, N, K, p, epi, st);
    else if (p.mt == 8) launch_tall<8, CT>(a, w, out, M, N, K, p, epi, st);
    else if (p.mt == 9) launch_tall<9, CT>(a, w, out, M, N, K, p, epi, st);
    else if constexpr (CT == 2) launch_tall<10, CT>(a, w, out, M, N, K, p, epi, st);       // the plan has no higher ones there
    else if (p.mt <= 11) launch_tall<11, CT>(a, w, out, M, N, K, p, epi, st);
    else launch_tall<12, CT>(a, w, out, M, N, K, p, epi, st);
}

}  // namespace

// Partial sums in the tiled layout, or (three column tiles, one split) SwiGLU of the interleaved gate/up matrix: products with a
// single split forced, the row-major logits among them, are not planned here.
void launch_gemm_bf16_tall(const bf16_t *a, const bf16_t *w, float *out, int M, int N, int K, const GemmPlan &p, int epi,
                           hipStream_t st) {
    if (p.nt == 2) launch_tall_rows<2>(a, w, out, M, N, K, p, epi, st);
    else launch_tall_rows<3>(a, w, out, M, N, K, p, epi, st);
}
