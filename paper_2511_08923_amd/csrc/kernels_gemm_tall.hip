// bf16 GEMM of 33 to 480 rows: out = A[M][K] x W[N][K]^T, fp32 accumulation, same operand layouts and epilogues as
// kernels_gemm.hip, and the same 32x32x16 MFMAs in the same order per output tile, so that the results are the same bits.
//
// At these row counts the weights come from HBM once and the activations (the step's 272 rows: 2.2 MB at K = 4096) from L2
// into every workgroup.  What bounds it is how much a compute unit takes in: with weights from HBM among the loads about
// 57 GB/s whatever the kernel (272 x 24576 x 4096: loads alone 57 us, MFMAs and LDS reads alone 48; activations alone 82
// GB/s per unit, everything from L2 102), which is why a deeper ring or fewer LDS reads change nothing beyond this:
//   * a workgroup owns all row tiles of the pass (up to twelve) and two or three column tiles, one workgroup per compute unit:
//     no weight is read twice, all of them stream;
//   * both operands go straight into LDS (buffer_load ... lds), PA chunks of 64 k of A and PW of W: the weights, which
//     are longer on their way, are asked for up to seven chunks ahead, in front of the activations of nearer chunks;
//   * four waves over the rows (wave, wave + 4, ...): an A fragment is read from LDS once, a W fragment by every wave; the
//     fragments of the next k step and the loads are spread between the MFMAs, one barrier per chunk of 64 k.
// The accumulators are tied to AGPRs by inline assembly: left to the compiler they are copied between the register files
// around every use (85 instead of 63 us).  The waves sharing K (16x16x32 MFMAs, half the LDS reads) were no faster.
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

// RT: row tiles of the higher passes, CT: column tiles of a workgroup
template <int RT, int CT>
__global__ __launch_bounds__(256) void gemm_bf16_tall_kernel(const bf16_t *__restrict__ a, const bf16_t *__restrict__ w,
                                                             float *__restrict__ out, int M, int N, int K, int splits,
                                                             int epi, int n_pass, int n_tall) {
    constexpr int PA = a_chunks(RT, CT), PW = w_chunks(RT, CT), RW = (RT + 3) / 4;
    constexpr int A_CHUNK = 4 * RT * 1024, W_CHUNK = 4 * CT * 1024;
    static_assert(PA * A_CHUNK + PW * W_CHUNK <= LDS_KB * 1024, "LDS of a compute unit");
    static_assert(PW * CT + PA * RT < 62, "the loads in flight are counted in six bits");
    extern __shared__ __attribute__((aligned(16))) unsigned char tall_smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t32 = (N + 31) >> 5, m_tiles = (M + 31) >> 5;
    const int j8 = blockIdx.x >> 3, unit = (j8 / n_pass) * 8 + (blockIdx.x & 7);
    const int bz = j8 % n_pass, split = unit % splits, tile0 = (unit / splits) * CT;
    if (tile0 >= t32) return;
    const int mt_base = bz * (RT - 1) + min(bz, n_tall), ct_here = bz < n_tall ? RT : RT - 1;
    const SplitRange sr = split_range(K, splits, split);
    const int n_steps = 2 * max(sr.q1 - sr.q0, 0), n_chunks = (n_steps + 3) >> 2;      // steps of 16 k

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
        dma16_tile(w_dst + buf * W_CHUNK, w_off[j], dw, 4 * c + wave < n_steps, w_src + 4 * c * t32 * 1024, j);
    };
    auto next = [](int b, int n) { return b + 1 == n ? 0 : b + 1; };
    f32x16 acc[RW][CT];
#pragma unroll
    for (int i = 0; i < RW; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
#pragma unroll
    for (int c = 0; c < PW - PA; ++c)
#pragma unroll
        for (int j = 0; j < CT; ++j) load_w(c, c, j);
    // generation g of the loads brings chunks g + PA of A and g + PW of W into the buffers that chunk g leaves; a quarter of it
    // goes out in step 3 of chunk g, the others in steps 0, 1 and 2 of chunk g + 1
    constexpr int LOADS = RT + CT;
    auto load = [&](int g, int ba, int bw, int l) __attribute__((always_inline)) {
        if (l < RT) load_a(g + PA, ba, l);
        else load_w(g + PW, bw, l - RT);
    };
#pragma unroll
    for (int c = 0; c < PA; ++c)
#pragma unroll
        for (int l = 0; l < (c < PA - 1 ? LOADS : LOADS / 4); ++l) load(c - PA, c, c + PW - PA, l);
    wait_loads<CT + (PA - 2) * LOADS + LOADS / 4>();
    lds_barrier_counted();
    // the wave's row tiles: wave, wave + 4, ...
    const unsigned char *fa = tall_smem + (wave * 64 + lane) * 16, *fw = tall_smem + PA * A_CHUNK + lane * 16;
    auto k_loop = [&](auto ra_tag) __attribute__((always_inline)) {
        constexpr int RA = decltype(ra_tag)::value, NM = RA * CT, READS = RA ? RA + CT : 0;
        bf16x8 af[2][RA ? RA : 1], wf[2][CT];
        auto read = [&](int s, int step, const unsigned char *ca, const unsigned char *cw, int f) __attribute__((always_inline)) {
            // in the order of use: W 0, A 0, the other W, the other A
            if (f == 0) wf[s][0] = *(const bf16x8 *)(cw + step * CT * 1024);
            else if (f == 1) af[s][0] = *(const bf16x8 *)(ca + step * RT * 1024);
            else if (f <= CT) wf[s][f - 1] = *(const bf16x8 *)(cw + (step * CT + f - 1) * 1024);
            else af[s][f - CT] = *(const bf16x8 *)(ca + (step * RT + 4 * (f - CT)) * 1024);
        };
#pragma unroll
        for (int f = 0; f < READS; ++f) read(0, 0, fa, fw, f);
        int ba = 0, bw = 0, g = -1, ga = PA - 1, gw = PW - 1;      // buffers of chunk c; generation under way and its buffers
        for (int c = 0; c < n_chunks; ++c) {
            const int na = next(ba, PA), nw = next(bw, PW);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int s = q & 1;
                const unsigned char *ca = fa + (q == 3 ? na : ba) * A_CHUNK, *cw = fw + (q == 3 ? nw : bw) * W_CHUNK;
                if (q == 3) {
                    ga = ba;
                    gw = bw;
                    g = c;
                }
                const int l0 = LOADS * ((q + 1) & 3) / 4, l1 = LOADS * (((q + 1) & 3) + 1) / 4;
                constexpr int B = NM > 1 ? 1 : 0;         // MFMAs in front of the barrier
                auto ops = [&](int x, int n) __attribute__((always_inline)) {
                    const int r0 = READS * x / n, r1 = READS * (x + 1) / n;
                    for (int f = r0; f < r1; ++f) read(s ^ 1, (q + 1) & 3, ca, cw, f);
                    const int m0 = l0 + (l1 - l0) * x / n, m1 = l0 + (l1 - l0) * (x + 1) / n;
                    for (int l = m0; l < m1; ++l) load(g, ga, gw, l);
                };
                auto sync = [&]() __attribute__((always_inline)) {
                    wait_loads<CT + (PA - 2) * (RT + CT)>();
                    lds_barrier_counted();               // chunk c+1 has landed for everyone, chunk c has been read by everyone
                };
                if constexpr (NM == 0) {
                    if (q == 3) sync();
                    ops(0, 1);
                }
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    if (q == 3 && m == B) sync();
                    __builtin_amdgcn_sched_barrier(0);
                    // The compiler does not see the MFMAs finish, and where the loop ends it may copy their results at once, so
                    // the last one of the last chunk brings the wait (32 states; it asks for 12 before its result is read) in
                    // the same piece of assembly
                    if (q == 3 && m == NM - 1)
                        asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0\n\t"
                                     "s_cmp_lg_i32 %3, %4\n\ts_cbranch_scc1 .Lmore%=\n\ts_nop 15\n\ts_nop 15\n.Lmore%=:"
                                     : "+a"(acc[m / CT][m % CT])
                                     : "v"(wf[s][m % CT]), "v"(af[s][m / CT]), "s"(c + 1), "s"(n_chunks)
                                     : "scc");
                    else
                        asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0"
                                     : "+a"(acc[m / CT][m % CT])
                                     : "v"(wf[s][m % CT]), "v"(af[s][m / CT]));
                    __builtin_amdgcn_sched_barrier(0);
                    if (q != 3) ops(m, NM);
                    else if (m >= B) ops(m - B, NM - B);
                }
            }
            ba = na;
            bw = nw;
        }
    };
    const int mine = (ct_here - wave + 3) >> 2;              // row tiles of this wave: RW or one less
    if (mine == RW) k_loop(std::integral_constant<int, RW>());
    else k_loop(std::integral_constant<int, RW - 1>());
    wait_loads<0>();
    lds_barrier_counted();
    ChooseArgs none = {};
    large_epilogue<RW, CT, 4>(acc, out, tall_smem, epi, split, M, N, mt_base, ct_here, tile0, wave, 4, wave, lane, none);
}

template <int RT, int CT>
void launch_tall(const bf16_t *a, const bf16_t *w, float *out, int M, int N, int K, const GemmPlan &p, int epi, hipStream_t st) {
    constexpr int SMEM = 4 * 1024 * (a_chunks(RT, CT) * RT + w_chunks(RT, CT) * CT);
    static_assert(SMEM >= 4 * 32 * 36 * 4, "the epilogue's patches");
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
    else if (p.mt == 10) launch_tall<10, CT>(a, w, out, M, N, K, p, epi, st);
    else if (p.mt == 11) launch_tall<11, CT>(a, w, out, M, N, K, p, epi, st);
    else launch_tall<12, CT>(a, w, out, M, N, K, p, epi, st);
}

}  // namespace

void launch_gemm_bf16_tall(const bf16_t *a, const bf16_t *w, float *out, int M, int N, int K, const GemmPlan &p, int epi,
                           hipStream_t st) {
    if (p.nt == 2) launch_tall_rows<2>(a, w, out, M, N, K, p, epi, st);
    else launch_tall_rows<3>(a, w, out, M, N, K, p, epi, st);
}
