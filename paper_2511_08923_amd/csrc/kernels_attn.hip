// Hybrid-mask paged attention for the decode step (bf16 MFMA path) and its split-KV combine.
//
// Work item = (sequence, kv head, chunk of 32-row query tiles, split of the key range).  The query rows of a
// kv head are the rows of all query heads in its group, flattened (head-in-group major), so a K/V tile that
// is brought into LDS once serves every query head that shares it.  Four waves split the query tiles; each wave
// keeps its Q fragments, its O^T accumulators and its softmax state in registers for the whole key range.
//
// MFMA: v_mfma_f32_32x32x16_bf16 (on gfx950 twice the rate of the 16x16x32 form).  Scores are formed
// transposed, S^T[key][q] = K . Q^T, so that in the result layout a lane holds one query column and 16 of the
// 32 keys of a block.  After exponentiation and without any data movement a lane's registers 0-7 (first page of
// the pair) and 8-15 (second page) are the B operands (P^T) of two MFMAs O^T[d][q] += V^T[d][key] . P^T[key][q];
// V is kept transposed in HBM ([head_dim][16 tokens] per page).
//
// K/V tiles go from HBM straight into LDS (buffer_load ... lds, 16 bytes per lane), three buffers deep, two
// key-pair iterations ahead of their use: no staging registers, no LDS stores, and the loads of a tile have two
// iterations to arrive.  A wave's lanes choose *which* 16 bytes they fetch, which is where the LDS layout comes
// from: K rows of 256 bytes whose 16-byte pieces are XOR-swizzled by the row (conflict-free fragment reads without
// padding), rows 4-7 and 8-11 of a unit exchanged so that a lane's score registers of a unit are eight consecutive
// keys, the same eight that one 16-byte piece of V^T holds.
//
// Softmax numerators are taken against an integral power-of-two reference (ceil of a running maximum in log2
// units): their bf16 rounding is then independent of the reference in force, i.e. of tiling and splits, and
// every rescale is exact.  The reference is lazy: a row's reference is set by its first visible block and moves
// only when the scores outgrow it by 2^60, which in practice is never; the loop over plain prefix keys therefore
// has no rescale arm at all (attn_block_fixed_ref), and leaves for the general loop if that ever happens.
//
// Keys come in units of 16: cache pages 0 .. ceil((L+nc)/16)-1, then the mask rows' scratch tiles.  Pages that
// lie wholly below L need no mask at all (every row sees the whole prefix); everything else goes through the
// (row, key) predicate and a per-(query tile, key pair) skip when nothing is visible.
#include <algorithm>
#include <type_traits>

#include "lds_dma.h"
#include "tidar_internal.h"

namespace {

constexpr int HD = 128;
constexpr int TILE = 32 * HD;           // bf16 elements of one K tile (32 keys) and of one V^T tile

struct AttnArgs {
    const bf16_t *q;
    KvView kv;
    const bf16_t *k_scr, *v_scr;
    const int32_t *prefix_len;
    RowDesc d;
    int n_q, group;
    int n_chunks, tiles_per_chunk, splits, per;
    int n_groups;                         // batch x kv heads
    int xcd_q;                            // 0: plain order; q >= 1: a group's chunks go to q XCDs (see the kernel)
    float scale_log2e;
    float *opart, *mpart, *lpart;
    bf16_t *out;               // single split only: [rows][n_q][HD], or the A-fragment layout (out_af)
    int out_af;
    ActLayout lay;
    AttnRope rp;               // ROPE kernels only
};

struct PlainOrder {};          // instead of a WorkOrder: by index

// Key-pair iterations a workgroup can need at all: cache units up to the furthest key any of its rows sees, then the
// mask units of its rows' own blocks, [0, a1) and [b0, b1) with a1 <= b0.  (Rows of one query head only; a workgroup
// that straddles two heads keeps the whole range.)  Inside a prefill or scoring pass most of the range falls away:
// causal rows see neither the later rows of the pass nor any mask row, a mask block only the text before it and
// itself.  Iterations are dropped whole, so the pairing of keys into iterations and splits is untouched.
struct KeySpan {
    int a1, b0, b1;
};
__host__ __device__ inline int imin(int x, int y) { return x < y ? x : y; }
__host__ __device__ inline int imax(int x, int y) { return x > y ? x : y; }
__host__ __device__ inline KeySpan key_span(const RowDesc &d, int L, int F, int t0, int t1) {
    const int n_cache_units = (L + d.nc + 15) >> 4, n_it = (n_cache_units + ((d.nm + 15) >> 4) + 1) >> 1;
    const int f_lo = t0 * 32, f_hi = imin(F, t1 * 32) - 1;
    const int h_lo = f_lo / d.R, h_hi = f_hi / d.R;
    if (h_lo != h_hi) return {n_it, n_it, n_it};
    const int r_lo = f_lo - h_lo * d.R, r_hi = f_hi - h_lo * d.R;
    int vis_max = imin(r_hi, d.nc - 1) + 1;                      // the causal rows among them
    int um0 = 0, um1 = 0;                                        // mask units [um0, um1)
    if (r_hi >= d.nc) {
        const int j_lo = (imax(r_lo, d.nc) - d.nc) / d.bl, j_hi = (r_hi - d.nc) / d.bl;
        if (r_lo >= d.nc) vis_max = 0;
        vis_max = imax(vis_max, d.cond0 + j_hi * d.cstride);
        um0 = (j_lo * d.bl) >> 4;
        um1 = (imin((j_hi + 1) * d.bl, d.nm) + 15) >> 4;
    }
    KeySpan k;
    const int uc1 = imin(n_cache_units, (L + imin(vis_max, d.nc) + 15) >> 4);
    k.a1 = (uc1 + 1) >> 1;
    k.b0 = imax(k.a1, (n_cache_units + um0) >> 1);
    k.b1 = um1 > um0 ? imax(k.b0, (n_cache_units + um1 + 1) >> 1) : k.b0;
    return k;
}

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

// One 32-query x 32-key block: S^T = K.Q^T, online softmax against the integral reference, O^T += V^T.P^T.
// c = softmax scale * log2(e).  VIS: bit e set = register e's key is visible to this lane's query row (only read
// when MASKED).  Kept lean: per score one max, one fma, one v_exp_f32, half a pack and half a dot2.
// Tile layout in LDS (see the kernel): K rows of 256 bytes with the 16-byte pieces XOR-swizzled by the row, rows
// 4-7 and 8-11 of a unit exchanged so that score register e of unit u is key 8*(lane/32) + e%8; V^T as
// [unit][key half][d] 16-byte pieces in natural key order.
template <bool MASKED>
__device__ inline void attn_block(const bf16_t *k_lds, const bf16_t *v_lds, int lq, int lh, const bf16x8 (&qf)[8],
                                  f32x16 (&acc)[4], float &m_run, float &l_run, float c, unsigned vis) {
    const unsigned char *kb = reinterpret_cast<const unsigned char *>(k_lds);
    const unsigned char *vb = reinterpret_cast<const unsigned char *>(v_lds);
    // K as A operand: lane = (tile row, hd half of the k step); V^T as A operand: lane = (d, key half of the unit)
    auto k_frag = [&](int ks) { return *(const bf16x8 *)(kb + lq * 256 + (((2 * ks + lh) ^ (lq & 15)) << 4)); };
    auto v_frag = [&](int dt, int u) { return *(const bf16x8 *)(vb + (((u * 2 + lh) * 128 + 32 * dt + lq) << 4)); };
    // K as A operand (lane = key, hd half of the k step); fragments are consumed as they arrive.  One
    // accumulation chain: a second one costs 16 registers, and the other resident wave covers the dependency
    f32x16 s;
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
        const bf16x8 kf0 = k_frag(ks);
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf0, qf[ks], s, 0, 0, 0);
    }
    // V^T as A operand (lane = d, key chunk): the first half is issued now and is needed after the softmax
    // arithmetic; the second half is read once the scores are dead and takes over their registers
    bf16x8 vf[2][2];
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int u = 0; u < 2; ++u)
            vf[dt][u] = v_frag(dt, u);
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        if (MASKED) s[e] = ((vis >> e) & 1u) ? s[e] : -INFINITY;
        mx = fmaxf(mx, s[e]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    // The reference of a row moves only when its scores outgrow it by 2^60 (or it is still -inf): the same rule
    // that makes attn_block_fixed_ref refuse a block, so that which of the two ran a block (that depends on how
    // much of the key range is plain prefix, i.e. on the sequence length) leaves no trace in the result.  (The
    // numerators' mantissas do not depend on the reference in exact arithmetic, but fma(s, c, -m) is rounded.)
    const bool grow = !(mx * c <= m_run + 60.f);
    const float m_new = grow ? fmaxf(m_run, ceilf(mx * c)) : m_run;
    const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
    const bf16x2 ones = {(bf16_t)1.0f, (bf16_t)1.0f};
    float psum = 0.f;
    bf16x8 pf[2];
#pragma unroll
    for (int e = 0; e < 16; e += 2) {
        bf16x2 pk = {(bf16_t)__builtin_amdgcn_exp2f(fmaf(s[e], c, -m_safe)),
                     (bf16_t)__builtin_amdgcn_exp2f(fmaf(s[e + 1], c, -m_safe))};
        psum = __builtin_amdgcn_fdot2_f32_bf16(pk, ones, psum, false);   // the denominator sums the rounded values
        pf[e >> 3][e & 7] = pk[0];
        pf[e >> 3][(e & 7) + 1] = pk[1];
    }
    // O^T += V^T.P^T.  The rescale by the exact 2^(old - new) is rare after the first blocks; it shares its arm of
    // the branch with a copy of the accumulation so that the common arm updates the accumulators in place (a
    // rescale arm that rejoined before the MFMAs made the compiler copy all 64 accumulator registers per block)
    auto accumulate = [&]() __attribute__((always_inline)) {
        bf16x8 vg[2][2];
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int u = 0; u < 2; ++u) vg[dt][u] = v_frag(dt + 2, u);
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int u = 0; u < 2; ++u)
                acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[dt][u], pf[u], acc[dt], 0, 0, 0);
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int u = 0; u < 2; ++u)
                acc[dt + 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vg[dt][u], pf[u], acc[dt + 2], 0, 0, 0);
    };
    if (__builtin_expect(__any(m_new != m_run), 0)) {
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_safe);
        l_run = l_run * alpha + psum;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[dt][e] *= alpha;
        m_run = m_new;
        accumulate();
    } else {
        l_run += psum;
        accumulate();
    }
}

// The same block for keys that are all visible, without the arm that moves the reference: the numerators are
// 2^(s.c - m_run) with the reference of an earlier block, so they may exceed 1 (by less than 2^60, or the block
// is refused before it changes anything: the caller then runs attn_block, which moves the reference by the same
// rule).  bf16 rounding is a matter of the mantissa alone, and every quantity (numerators, denominator, O^T)
// carries the same power of two.  No rescale arm means no branch that rejoins around the accumulators: with one,
// the compiler copied all 64 accumulator registers twice per block.
template <bool PRIO>
__device__ inline bool attn_block_fixed_ref(const bf16_t *k_lds, const bf16_t *v_lds, int lq, int lh,
                                            const bf16x8 (&qf)[8], f32x16 (&acc)[4], float m_run, float &l_run,
                                            float c) {
    const unsigned char *kb = reinterpret_cast<const unsigned char *>(k_lds);
    const unsigned char *vb = reinterpret_cast<const unsigned char *>(v_lds);
    // K as A operand: lane = (tile row, hd half of the k step); V^T as A operand: lane = (d, key half of the unit)
    auto k_frag = [&](int ks) { return *(const bf16x8 *)(kb + lq * 256 + (((2 * ks + lh) ^ (lq & 15)) << 4)); };
    auto v_frag = [&](int dt, int u) { return *(const bf16x8 *)(vb + (((u * 2 + lh) * 128 + 32 * dt + lq) << 4)); };
    // all eight K fragments are asked for before the first MFMA: read one or two ahead of its MFMA, as the compiler
    // orders them by itself, every link of the score chain waits out a full LDS round trip
    bf16x8 kf[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) kf[ks] = k_frag(ks);
    __builtin_amdgcn_sched_barrier(0);
    f32x16 s;
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], s, 0, 0, 0);
    // PRIO (launches in which all four waves hold a query tile): the softmax section runs at a raised wave priority.
    // The SIMD's other wave is then the one that waits while it is in an MFMA chain of its own, and the two fall into
    // opposite phases more often (measured: -3 % at 272 rows, -1 % at batch 8; raising the priority of the MFMA
    // chains instead changes nothing).  Not for the few-row shapes, whose three other waves only move tiles: there
    // the raised wave holds up their loads (1-token step at batch 8: +2.6 %).
    if (PRIO) __builtin_amdgcn_s_setprio(3);
    bf16x8 vf[2][2];
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int u = 0; u < 2; ++u) vf[dt][u] = v_frag(dt, u);
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[e]);
    if (__any(!(mx * c <= m_run + 60.f))) {                       // also refuses a reference that is still -inf
        if (PRIO) __builtin_amdgcn_s_setprio(0);
        return false;
    }
    const bf16x2 ones = {(bf16_t)1.0f, (bf16_t)1.0f};
    float psum = 0.f;
    bf16x8 pf[2];
#pragma unroll
    for (int e = 0; e < 16; e += 2) {
        bf16x2 pk = {(bf16_t)__builtin_amdgcn_exp2f(fmaf(s[e], c, -m_run)),
                     (bf16_t)__builtin_amdgcn_exp2f(fmaf(s[e + 1], c, -m_run))};
        psum = __builtin_amdgcn_fdot2_f32_bf16(pk, ones, psum, false);
        pf[e >> 3][e & 7] = pk[0];
        pf[e >> 3][(e & 7) + 1] = pk[1];
    }
    l_run += psum;
    if (PRIO) __builtin_amdgcn_s_setprio(0);
    bf16x8 vg[2][2];
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int u = 0; u < 2; ++u) vg[dt][u] = v_frag(dt + 2, u);
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int u = 0; u < 2; ++u)
            acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[dt][u], pf[u], acc[dt], 0, 0, 0);
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int u = 0; u < 2; ++u)
            acc[dt + 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vg[dt][u], pf[u], acc[dt + 2], 0, 0, 0);
    return true;
}

// QT: 32-row query tiles per wave.
template <int QT, bool PRIO, bool ROPE, class SG, class ORD>
__global__ __launch_bounds__(256, 2) void attn_bf16_kernel(AttnArgs a, SG sg, ORD ord) {
    constexpr int NBUF = 3, K_TILE = TILE, V_TILE = TILE;
    __shared__ __attribute__((aligned(16))) bf16_t k_lds[NBUF][K_TILE];
    __shared__ __attribute__((aligned(16))) bf16_t v_lds[NBUF][V_TILE];
    __shared__ __attribute__((aligned(16))) bf16_t q_lds[ROPE ? 32 * HD : 8];     // ROPE: the rotated Q rows of the group

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // known to be uniform: scalar registers
    const int lq = lane & 31, lh = lane >> 5;
    // Workgroup i of a launch runs on XCD i % 8 (the grid's x extent is then a multiple of 8, so the split index
    // does not change that).  Where the (sequence, kv head) groups divide evenly over the XCDs, or the XCDs over
    // the groups, the query chunks of one group are dealt to one XCD (or to 8 / groups of them), whose L2 then
    // fetches that head's K and V once instead of once per XCD that happens to run one of its chunks.
    int grp, chunk, split = blockIdx.y;
    if constexpr (sizeof(ORD) == sizeof(WorkOrder)) {
        const int xcd = blockIdx.x & 7;
        const int i = (blockIdx.x >> 3) * a.xcd_q + xcd % a.xcd_q;
        if (i >= ord.n) return;                      // padding of the last round (whole workgroup)
        const unsigned item = (ord.item2[i >> 1] >> (16 * (i & 1))) & 0xffffu;
        grp = xcd / a.xcd_q;
        chunk = item & 1023;
        split = item >> 10;
    } else if (a.xcd_q == 0) {
        chunk = blockIdx.x % a.n_chunks;
        grp = blockIdx.x / a.n_chunks;
    } else if (a.n_groups >= 8) {
        const int xj = blockIdx.x >> 3;
        grp = (xj / a.n_chunks) * 8 + (blockIdx.x & 7);
        chunk = xj % a.n_chunks;
    } else {
        const int xcd = blockIdx.x & 7;
        grp = xcd / a.xcd_q;
        chunk = (blockIdx.x >> 3) * a.xcd_q + xcd % a.xcd_q;
        if (chunk >= a.n_chunks) return;             // padding of the last round (whole workgroup)
    }
    const int g = grp % a.kv.n_kv;
    const int b = grp / a.kv.n_kv;
    int row_base;                                    // the sequence's first row of the forward
    const RowDesc d = seq_desc(a.d, sg, b, &row_base);
    const int F = a.group * d.R;                     // flattened query rows of this kv head
    const int TQ = (F + 31) >> 5;
    const int t0 = chunk * a.tiles_per_chunk;
    if (kSegs<SG> && t0 >= TQ) return;                            // a shorter sequence than the longest (whole workgroup)
    const int t1 = min(TQ, t0 + a.tiles_per_chunk);
    const int L = clamp_prefix(a.kv, a.prefix_len[d.seq_base + b], d.nc);   // never walks past the page table
    const int n_mask = d.nm;
    const int n_cache_units = (L + d.nc + 15) >> 4;
    const int n_pure = L >> 4;
    const int n_mt = (n_mask + 15) >> 4;
    const int U = n_cache_units + n_mt;
    const int n_it = (U + 1) >> 1;
    // Split s takes key-pair iterations [s*per, (s+1)*per) with per fixed by the host from its bound on the key
    // count: which split a key falls into does not depend on how long the sequence is right now, so the same
    // query over the same keys is reduced in the same grouping at every step (the last split takes whatever a
    // loose bound leaves over; splits past the end write an empty partial).
    const int per = a.per;
    const int it0 = min(n_it, split * per);
    const int it1 = (split == a.splits - 1) ? n_it : min(n_it, it0 + per);
    const KeySpan ks = key_span(d, L, F, t0, t1);
    // this split's share of the two ranges, walked as one sequence of nA + nB iterations
    const int a0 = it0, a1 = max(a0, min(it1, ks.a1));
    const int b0 = max(it0, ks.b0), b1 = max(b0, min(it1, ks.b1));
    const int nA = a1 - a0, n_seq = nA + (b1 - b0);
    auto seq_it = [&](int n) { return n < nA ? a0 + n : b0 + (n - nA); };

    if constexpr (ROPE) {
        // One row per sequence (R = 1): the group's query heads are the tile's rows.  A thread takes one rotation pair
        // (d, d + 64) of one head: it adds the split-K partial sums of the QKV projection and rotates by the row's
        // angles, exactly as the RoPE kernel does.  The workgroup whose key range holds the new row's position does
        // the same for K and copies V, and stores both into the cache page before any of its tile loads starts
        // (the stores are waited for, then a workgroup barrier: the loads that follow read them back from L2).
        const AttnRope &rp = a.rp;
        const int row = b;                                   // the call's row of this sequence
        const float *cs = rp.rope_cs + (size_t)row * (HD / 2) * 2;
        // sums of the splits in rising order (the RoPE kernel's order), two columns at a time and eight splits'
        // loads in flight for each: one load per trip would cost a memory round trip per split
        auto summed2 = [&](int col0, int col1, float &x, float &y) {
            const float *p0 = rp.part + pt_index(col0, row, rp.M_all), *p1 = rp.part + pt_index(col1, row, rp.M_all);
            x = 0.f;
            y = 0.f;
            for (int s0 = 0; s0 < rp.S; s0 += 8) {
                float t0[8], t1[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const size_t o = (size_t)min(s0 + j, rp.S - 1) * rp.split_stride;
                    t0[j] = p0[o];
                    t1[j] = p1[o];
                }
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (s0 + j < rp.S) {
                        x += t0[j];
                        y += t1[j];
                    }
            }
        };
        // The writing workgroup: its page id is asked for first, and every thread issues the loads of its K or V pair
        // together with those of its Q pair (a thread without a pair repeats a valid column and drops the sums), so
        // that the whole prologue is one memory round trip before the stores.
        const int L_raw = a.prefix_len[d.seq_base + b];
        const int it_new = (L >> 4) >> 1;                    // the key-pair iteration of position L
        const bool writes = it_new >= a0 && it_new < a1 && seq_fits(a.kv, L_raw, 1);
        int page = -1;
        if (writes) page = a.kv.page_table[(size_t)(d.seq_base + b) * a.kv.pages_per_seq + (L >> 4)];
        const int n_qp = a.group * (HD / 2);
        const int wi = tid & (HD / 2 - 1);
        const int wcol = (tid < HD / 2 ? rp.q_dim : rp.q_dim + rp.kv_dim) + g * HD + wi;
        float wx, wy;
        {
            const int idx = min(tid, n_qp - 1);
            const int hq = idx / (HD / 2), i = idx - hq * (HD / 2);
            const int col = (g * a.group + hq) * HD + i;
            float x, y;
            summed2(col, col + HD / 2, x, y);
            summed2(wcol, wcol + HD / 2, wx, wy);
            const float c = cs[2 * i], sn = cs[2 * i + 1];
            if (tid < n_qp) {
                q_lds[hq * HD + i] = (bf16_t)(x * c - y * sn);
                q_lds[hq * HD + i + HD / 2] = (bf16_t)(y * c + x * sn);
            }
        }
        for (int idx = tid + 256; idx < n_qp; idx += 256) {          // more than four query heads per kv head
            const int hq = idx / (HD / 2), i = idx - hq * (HD / 2);
            const int col = (g * a.group + hq) * HD + i;
            float x, y;
            summed2(col, col + HD / 2, x, y);
            const float c = cs[2 * i], sn = cs[2 * i + 1];
            q_lds[hq * HD + i] = (bf16_t)(x * c - y * sn);
            q_lds[hq * HD + i + HD / 2] = (bf16_t)(y * c + x * sn);
        }
        if (writes) {
            const int slot = L & 15;
            if (page_ok(a.kv, page) && tid < HD) {
                if (tid < HD / 2) {
                    const float c = cs[2 * wi], sn = cs[2 * wi + 1];
                    bf16_t *kdst = (bf16_t *)a.kv.k_pages + k_page_offset(a.kv, page, g, slot, 0);
                    kdst[wi] = (bf16_t)(wx * c - wy * sn);
                    kdst[wi + HD / 2] = (bf16_t)(wy * c + wx * sn);
                } else {
                    bf16_t *vp = (bf16_t *)a.kv.v_pages;
                    vp[v_page_offset(a.kv, page, g, slot, wi)] = (bf16_t)wx;
                    vp[v_page_offset(a.kv, page, g, slot, wi + HD / 2)] = (bf16_t)wy;
                }
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        __syncthreads();
    }

    // ---- this wave's query tiles: Q fragments (B operand: lane = (q row, hd half of the k step)), row info
    bf16x8 qf[QT][8];
    int r_vis[QT], r_blk[QT];
    int vis_min = 0x3fffffff;                        // fewest new keys any real row of this wave's tiles sees
    f32x16 acc[QT][4];
    float m_run[QT], l_run[QT];
#pragma unroll
    for (int i = 0; i < QT; ++i) {
        const int tile = t0 + wave + 4 * i;
        const int f = tile * 32 + lq;
        const bool ok = tile < t1 && f < F;
        const int hq = ok ? f / d.R : 0;
        const int r = ok ? f - hq * d.R : 0;
        const RowInfo ri = row_info(d, r, L);
        r_vis[i] = ok ? ri.vis : 0;
        r_blk[i] = ok ? ri.blk : -2;
        if (ok) vis_min = min(vis_min, ri.vis);
        const bf16_t *qp = ROPE ? q_lds + (ok ? f : 0) * HD + 8 * lh
                                : a.q + ((size_t)(row_base + r) * a.n_q + (g * a.group + hq)) * HD + 8 * lh;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            bf16x8 v = {0, 0, 0, 0, 0, 0, 0, 0};
            if (ok) v = *(const bf16x8 *)(qp + 16 * ks);
            qf[i][ks] = v;
        }
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][dt][e] = 0.f;
        m_run[i] = -INFINITY;
        l_run[i] = 0.f;
    }

    const size_t page_elems = (size_t)a.kv.n_kv * 16 * HD;
    const size_t scr_elems = (size_t)a.n_groups * (n_mt > 0 ? n_mt : 1) * 16 * HD;   // B * n_kv tiles
    const int32_t *pt = a.kv.page_table + (size_t)(d.seq_base + b) * a.kv.pages_per_seq;

    // one key-pair iteration of every query tile of this wave against LDS buffer `buf`
    // (pure_c: both units lie wholly inside the prefix, no predicate.  The pure iterations are the leading ones of
    // the sequence and get a loop of their own: with both forms in one loop body the compiler copied all 64
    // accumulator registers back and forth at the point where the two paths meet, in every iteration.)
    auto compute = [&](auto pure_c, int it, int buf) __attribute__((always_inline)) {
        constexpr bool pure = decltype(pure_c)::value;
#pragma unroll
        for (int i = 0; i < QT; ++i) {
            const int tile = t0 + wave + 4 * i;
            if (tile >= t1) continue;                       // wave-uniform
            if constexpr (pure) {
                attn_block<false>(k_lds[buf], v_lds[buf], lq, lh, qf[i], acc[i], m_run[i], l_run[i],
                                       a.scale_log2e, 0xffffu);
            } else {
                // A row sees a contiguous key range of each unit: cache positions below L + vis, or the mask rows
                // of its own block.  The range becomes a 16-bit mask over the unit's keys, from which the lane
                // picks its eight: register e of unit u <-> key 8*lh + e%8 of that unit.
                unsigned vis_bits = 0;                      // bit 8u+e: visible to this lane's query row
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int uu = 2 * it + u;
                    unsigned m16 = 0;
                    if (uu < n_cache_units) {               // uniform
                        const int lim = min(max(L + r_vis[i] - 16 * uu, 0), 16);
                        m16 = (1u << lim) - 1u;
                    } else if (uu < U) {
                        const int m0 = 16 * (uu - n_cache_units);
                        const int lo = min(max(r_blk[i] * d.bl - m0, 0), 16);
                        const int hi = min(max(min((r_blk[i] + 1) * d.bl, n_mask) - m0, 0), 16);
                        m16 = (r_blk[i] >= 0 && hi > lo) ? (((1u << hi) - 1u) & ~((1u << lo) - 1u)) : 0u;
                    }
                    vis_bits |= ((m16 >> (8 * lh)) & 0xffu) << (8 * u);
                }
                if (!__any(vis_bits != 0)) continue;        // nothing of this pair is visible to this tile
                attn_block<true>(k_lds[buf], v_lds[buf], lq, lh, qf[i], acc[i], m_run[i], l_run[i],
                                      a.scale_log2e, vis_bits);
            }
        }
    };

    const std::true_type pure_c;
    const std::false_type masked_c;
    // Leading iterations whose two units every row of this wave's tiles sees in full: the prefix, and in a prefill
    // or scoring pass also the rows of the pass that lie before the tile (all but the diagonal of a causal pass).
    // The count differs from wave to wave; the loops below pass the same one barrier per iteration.
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) vis_min = min(vis_min, __shfl_xor(vis_min, o));
    const int n_pure_w = __builtin_amdgcn_readfirstlane(min(n_cache_units, max(n_pure, (L + min(vis_min, d.nc)) >> 4)));
    const int n_fast = min(max(min(a1, n_pure_w >> 1) - a0, 0), nA);
    {
        // Direct loads: wave w moves unit w/2 of the pair: for K the LDS rows 8*(w%2) .. +7 of that unit (two
        // instructions of 1 KiB: lane = (row, 16-byte slot), the slot holds piece slot ^ row%16 of the key the row
        // stands for), for V^T the key half w%2 of all 128 d (lane = d).  The tiles land in buffer n % 3 two
        // iterations ahead of their use; a wave waits for its own loads of iteration n (vmcnt), then the workgroup
        // barrier makes all four waves' parts visible and at the same time frees the buffer of iteration n-1 for
        // the loads of iteration n+2.
        const int u_w = wave >> 1, half_w = wave & 1;
        int k_voff[2], v_voff[2];
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
            const int row = 8 * half_w + 4 * jj + (lane >> 4);                    // LDS row within the unit
            const int key = (row & 3) | ((row & 4) << 1) | ((row & 8) >> 1);     // rows 4-7 <-> keys 8-11
            k_voff[jj] = key * (HD * 2) + (((lane & 15) ^ row) << 4);
            v_voff[jj] = (64 * jj + lane) * 32 + half_w * 16;
        }
        // An odd unit count leaves the second half of the last pair's tiles unwritten.  Its scores are masked by
        // a select, so stale K bits do no harm, but its V^T is multiplied by probabilities of exactly zero and
        // must not be NaN or Inf: the workgroup that runs that last pair clears the V^T tiles first.
        if ((U & 1) && n_seq > 0 && seq_it(n_seq - 1) == n_it - 1) {
            for (int i = tid; i < NBUF * V_TILE / 8; i += 256)
                reinterpret_cast<bf16x8 *>(&v_lds[0][0])[i] = (bf16x8){0, 0, 0, 0, 0, 0, 0, 0};
            __syncthreads();
        }
        // the Q fragments must have arrived before the loop: a wait for them inside it would be a vmcnt(0) and
        // drain the tile loads in flight
#pragma unroll
        for (int i = 0; i < QT; ++i)
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) asm volatile("" : "+v"(qf[i][ks]));
        const int4v dk = raw_desc(a.kv.k_pages, (size_t)a.kv.n_pages * page_elems * 2);
        const int4v dv = raw_desc(a.kv.v_pages, (size_t)a.kv.n_pages * page_elems * 2);
        const int4v dks = raw_desc(a.k_scr, scr_elems * 2), dvs = raw_desc(a.v_scr, scr_elems * 2);
        typedef __attribute__((address_space(3))) unsigned char lds_byte;
        const unsigned k_lds0 = (unsigned)(size_t)(lds_byte *)reinterpret_cast<unsigned char *>(&k_lds[0][0]);
        const unsigned v_lds0 = (unsigned)(size_t)(lds_byte *)reinterpret_cast<unsigned char *>(&v_lds[0][0]);
        // the page table does not change while the kernel runs: read through the constant address space, the page
        // ids come by scalar loads (no vector-memory traffic that the vmcnt bookkeeping below would have to count)
        const __attribute__((address_space(4))) int32_t *ptc = (const __attribute__((address_space(4))) int32_t *)pt;
        // V^T slots past the data of a unit (the page the sequence ends in, the last mask tile) may hold anything:
        // they are cleared in LDS before use (uniform, at most twice in a workgroup's life)
        auto clear_tail = [&](int it, int buf) __attribute__((always_inline)) {
            bool any = false;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int uu = 2 * it + u;
                int valid = 16;
                if (uu < n_cache_units) valid = min(16, L + d.nc - 16 * uu);
                else if (uu < U) valid = min(16, n_mask - 16 * (uu - n_cache_units));
                if (valid < 16) {
                    any = true;
                    if (tid < 128) {
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            bf16x8 *pv = reinterpret_cast<bf16x8 *>(&v_lds[buf][0]) + (u * 2 + h) * 128 + tid;
                            bf16x8 vv = *pv;
#pragma unroll
                            for (int j = 0; j < 8; ++j)
                                if (8 * h + j >= valid) vv[j] = (bf16_t)0.f;
                            *pv = vv;
                        }
                    }
                }
            }
            if (any) lds_barrier();
        };
        auto unit_of = [&](int m) { return 2 * seq_it(m) + u_w; };
        auto page_of = [&](int m) {                          // page id of this wave's unit in iteration m (or 0)
            const int uu = unit_of(m);
            return (m < n_seq && uu < n_cache_units) ? ptc[uu] : 0;
        };
        int b_cur = 0, b_nxt = 1, b_far = 2;                // buffers of iterations n, n+1, n+2
        int c_nxt = 0;                                      // loads this wave issued last (0 or 4)
        int page = page_of(0);                              // page id of the next loads to be issued
        auto issue = [&](int m, int buf) __attribute__((always_inline)) {      // this wave's loads of iteration m
            const int uu = unit_of(m);
            c_nxt = 0;
            if (m < n_seq && uu < U) {
                const unsigned kd = k_lds0 + buf * (K_TILE * 2) + (u_w * 16 + 8 * half_w) * 256;
                const unsigned vd = v_lds0 + buf * (V_TILE * 2) + (u_w * 2 + half_w) * 2048;
                if (uu < n_cache_units) {
                    const int base = (int)((((size_t)page * a.kv.n_kv + g) * 16 * HD) * 2);
#pragma unroll
                    for (int jj = 0; jj < 2; ++jj) {
                        dma16(kd + 1024 * jj, k_voff[jj], dk, base);
                        dma16(vd + 1024 * jj, v_voff[jj], dv, base);
                    }
                } else {
                    const int mt = uu - n_cache_units;
                    const int base = (int)(((((size_t)b * a.kv.n_kv + g) * n_mt + mt) * 16 * HD) * 2);
#pragma unroll
                    for (int jj = 0; jj < 2; ++jj) {
                        dma16(kd + 1024 * jj, k_voff[jj], dks, base);
                        dma16(vd + 1024 * jj, v_voff[jj], dvs, base);
                    }
                }
                c_nxt = 4;
            }
            page = page_of(m + 1);
        };
        // make the tiles of iteration n usable and start the loads of iteration n+2 into the buffer that the
        // barrier has just freed (every wave is past iteration n-1).  A wave's loads of iteration n have landed
        // once no more than those of n+1, its latest, are in flight.
        auto ready = [&](int n) __attribute__((always_inline)) {
            if (c_nxt == 4) __builtin_amdgcn_s_waitcnt(4 | (7 << 4) | (15 << 8));
            else __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (15 << 8));
            lds_barrier();
            issue(n + 2, b_far);
        };
        auto rotate = [&]() __attribute__((always_inline)) {
            const int t = b_cur;
            b_cur = b_nxt;
            b_nxt = b_far;
            b_far = t;
        };
        auto general = [&](int n) __attribute__((always_inline)) {
            const int it = seq_it(n);
            clear_tail(it, b_cur);
            compute(masked_c, it, b_cur);
        };
        issue(0, b_cur);
        issue(1, b_nxt);
        int n = 0;
        if (n_seq > 0) {
            ready(0);
            // the first iteration moves the references off -inf; the iterations that follow, while both their
            // units lie inside the prefix, keep them where they are (no rescale arm in that loop); a wave whose
            // scores outgrow its reference by 2^60 leaves for the general loop (the waves of a workgroup may
            // be in different loops: each iteration of either passes the same one barrier)
            if (n_fast > 0) compute(pure_c, seq_it(0), b_cur);
            else general(0);
            for (n = 1; n < n_fast; ++n) {
                rotate();
                ready(n);
                bool ok = true;
#pragma unroll
                for (int i = 0; i < QT; ++i) {
                    const int tile = t0 + wave + 4 * i;
                    if (tile < t1)
                        ok = ok && attn_block_fixed_ref<PRIO>(k_lds[b_cur], v_lds[b_cur], lq, lh, qf[i], acc[i], m_run[i],
                                                             l_run[i], a.scale_log2e);
                }
                if (!ok) break;
            }
            if (n < n_fast) {          // refused: this iteration's tiles are ready, only the block has to run
                general(n);
                ++n;
            }
            for (; n < n_seq; ++n) {
                rotate();
                ready(n);
                general(n);
            }
        }
    }

    // ---- a single split is the whole answer: normalise in registers and store it (a lane holds, for its query
    // row, 16 runs of four consecutive head-dim values), no partial results and no combine launch
    if (a.splits == 1) {
#pragma unroll
        for (int i = 0; i < QT; ++i) {
            const int tile = t0 + wave + 4 * i;
            if (tile >= t1) continue;
            float l = l_run[i];
            l += __shfl_xor(l, 32);
            const int f = tile * 32 + lq;
            if (f >= F) continue;
            const float inv = 1.f / l;
            const int hq = f / d.R, r = f - hq * d.R;
            const int row = row_base + r, col0 = (g * a.group + hq) * HD + 4 * lh;
            typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const bf16x4 o = {(bf16_t)(acc[i][dt][4 * r4] * inv), (bf16_t)(acc[i][dt][4 * r4 + 1] * inv),
                                      (bf16_t)(acc[i][dt][4 * r4 + 2] * inv), (bf16_t)(acc[i][dt][4 * r4 + 3] * inv)};
                    const int col = col0 + 32 * dt + 8 * r4;
                    const size_t idx = a.out_af ? af_index(row, col, a.lay) : (size_t)row * a.n_q * HD + col;
                    *(bf16x4 *)(a.out + idx) = o;
                }
        }
        return;
    }

    // ---- write this split's partial (unnormalised O, reference in log2 units, denominator)
    const size_t pbase = (size_t)row_base * a.n_q * a.splits + ((size_t)g * a.splits + split) * F;
#pragma unroll
    for (int i = 0; i < QT; ++i) {
        const int tile = t0 + wave + 4 * i;
        if (tile >= t1) continue;
        float l = l_run[i];
        l += __shfl_xor(l, 32);
        const int f = tile * 32 + lq;
        if (f < F) {
            // PRIO (AttnPlan::tiled): the tile as it lies in the registers, 16 bytes per row side by side, a store being one
            // contiguous KiB; otherwise row by row
            const int n_rows = min(32, F - 32 * tile);
            float *op = PRIO ? a.opart + (pbase + 32 * tile) * HD + 4 * (lh * n_rows + lq) : a.opart + (pbase + f) * HD + 4 * lh;
            const int piece = PRIO ? 8 * n_rows : 8;
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    f32x4 v = {acc[i][dt][4 * r4], acc[i][dt][4 * r4 + 1], acc[i][dt][4 * r4 + 2],
                               acc[i][dt][4 * r4 + 3]};
                    *(f32x4 *)(op + (4 * dt + r4) * piece) = v;
                }
            if (lh == 0) {
                a.mpart[pbase + f] = m_run[i];
                a.lpart[pbase + f] = l;
            }
        }
    }
}

// out[row][head][d] = sum_s w_s O_s / sum_s w_s l_s,  w_s = 2^(m_s - max m): exact powers of two, since every
// split keeps an integral reference.  One wave per (row, head): lane = (8-value head-dim chunk, one of 4 split
// lanes); the split lanes share the splits between them and are folded with two shuffles.  The 16-byte result
// goes out row-major or in the A-fragment layout of the O projection's input.
// It is bound by the partial results, so no lane asks for more splits than there are (J).  Forwards of up to three query tiles per
// kv head come here.  LINES, from 481 rows on: the workgroups of the rows that share an output line run on one XCD, us by index ->
// so: 640 rows x 32 heads in 2 splits 12.5 -> 11.1, 660 x 32 12.6 -> 11.1, 648 x 12 in 4 splits 7.1 -> 6.2.
template <int J, bool LINES, class SG>
__global__ __launch_bounds__(64) void attn_combine_kernel(const float *__restrict__ opart,
                                                          const float *__restrict__ mpart,
                                                          const float *__restrict__ lpart, RowDesc d, SG sg, int n_q,
                                                          int n_kv, int splits, int M, bf16_t *__restrict__ out, int out_af,
                                                          ActLayout lay) {
    const int row = LINES ? line_row(blockIdx.x) : blockIdx.x;
    if (LINES && row >= M) return;
    const int head = blockIdx.y;
    const int b = seq_of_row(d, sg, row);
    int row_base;
    const int R = seq_desc(d, sg, b, &row_base).R, r = row - row_base;
    const int group = n_q / n_kv;
    const int F = group * R;
    const int g = head / group, hq = head - g * group;
    const int f = hq * R + r;
    const int lane = threadIdx.x, d0 = 8 * (lane & 15), sl = lane >> 4;
    const size_t base = (size_t)row_base * n_q * splits + (size_t)g * splits * F + f;      // partial result of split 0
    // reference of the whole row: lane s reads split s's (there are at most 64 splits), then a wave-wide maximum
    float mmax = lane < splits ? mpart[base + (size_t)lane * F] : -INFINITY;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) mmax = fmaxf(mmax, __shfl_xor(mmax, o));
    float num[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, den = 0.f;
    // J splits of this split lane at a time: all their loads are issued before the first is used (an absent split re-reads
    // the last one and is given the weight of an empty split)
    for (int sp0 = sl; sp0 < splits; sp0 += 4 * J) {
        float m[J], l[J];
        float4 a[J], c[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int sp = sp0 + 4 * j;
            const size_t pi = base + (size_t)min(sp, splits - 1) * F;
            m[j] = mpart[pi];
            l[j] = lpart[pi];
            const float *op = opart + pi * HD + d0;
            a[j] = *(const float4 *)op;
            c[j] = *(const float4 *)(op + 4);
            if (sp >= splits) m[j] = -INFINITY;
        }
#pragma unroll
        for (int j = 0; j < J; ++j) {
            if (m[j] == -INFINITY) continue;
            const float wgt = exp2f(m[j] - mmax);
            num[0] += wgt * a[j].x; num[1] += wgt * a[j].y; num[2] += wgt * a[j].z; num[3] += wgt * a[j].w;
            num[4] += wgt * c[j].x; num[5] += wgt * c[j].y; num[6] += wgt * c[j].z; num[7] += wgt * c[j].w;
            den += wgt * l[j];
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        num[e] += __shfl_xor(num[e], 16);
        num[e] += __shfl_xor(num[e], 32);
    }
    den += __shfl_xor(den, 16);
    den += __shfl_xor(den, 32);
    if (sl == 0) {
        const float inv = 1.f / den;
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (bf16_t)(num[e] * inv);
        const size_t idx = out_af ? af_index(row, head * HD + d0, lay) : ((size_t)row * n_q + head) * HD + d0;
        *(bf16x8 *)(out + idx) = o;
    }
}

// The same for partial results that lie as query tiles (AttnPlan::tiled).  A wave takes 16 head-dim values of the 32 rows of a
// tile: lane = (row, half of each eight), so every load is one contiguous KiB, and so is the store to the A-fragment layout
// where the rows do not straddle two of its row tiles.  The sums are grouped as above (four runs of every fourth split,
// folded in pairs): the same bits.  With row-by-row partial results every store of the attention kernel was 64 pieces of 16
// bytes in 32 lines: attention, its K/V placement and the combine at 8B heads, 272 rows and 4096 keys 46.3 -> 44.2 us,
// 8B step k = 16 7726 -> 7620, 1.5B 3086 -> 3037.  Up to three tiles the waves per row stay: their rows are too few to
// fill the chip by tiles.
template <class SG>
__global__ __launch_bounds__(256) void attn_combine_tiles_kernel(const float *__restrict__ opart, const float *__restrict__ mpart,
                                                                 const float *__restrict__ lpart, RowDesc d, SG sg, int n_q,
                                                                 int n_kv, int splits, int n_tiles, int n_groups,
                                                                 bf16_t *__restrict__ out, int out_af, ActLayout lay) {
    const int lane = threadIdx.x & 63, dt = threadIdx.x >> 6, pr = blockIdx.y;
    const int lq = lane & 31, lh = lane >> 5;
    int grp, t;
    if (n_groups % 8 == 0) {                         // the XCD that ran the group's attention
        const int j = blockIdx.x >> 3;
        grp = (j / n_tiles) * 8 + (blockIdx.x & 7);
        t = j % n_tiles;
    } else {
        grp = blockIdx.x / n_tiles;
        t = blockIdx.x % n_tiles;
    }
    const int b = grp / n_kv, g = grp - b * n_kv, group = n_q / n_kv;
    int row_base;
    const int R = seq_desc(d, sg, b, &row_base).R, F = group * R;
    const int n_rows = min(32, F - 32 * t);
    if (n_rows <= 0) return;                         // a shorter sequence than the longest (whole workgroup)
    const int lr = min(lq, n_rows - 1);              // lanes past the rows repeat the last and store nothing
    const int f = 32 * t + lr;
    const size_t base = (size_t)row_base * n_q * splits + (size_t)g * splits * F;
    const float *mp = mpart + base + f, *lp = lpart + base + f;
    const float *op = opart + (base + 32 * t) * HD + ((4 * dt + 2 * pr) * 2 + lh) * 4 * n_rows + 4 * lr;
    float mmax = -INFINITY;
#pragma unroll 8
    for (int s = 0; s < splits; ++s) mmax = fmaxf(mmax, mp[(size_t)s * F]);
    f32x4 num[4][2];
    float den[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        num[j][0] = num[j][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
        den[j] = 0.f;
    }
    for (int s0 = 0; s0 < splits; s0 += 4) {
        f32x4 x[4], y[4];
        float m[4], l[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const size_t o = (size_t)min(s0 + j, splits - 1) * F;
            x[j] = *(const f32x4 *)(op + o * HD);
            y[j] = *(const f32x4 *)(op + o * HD + 8 * n_rows);
            m[j] = s0 + j < splits ? mp[o] : -INFINITY;
            l[j] = lp[o];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (m[j] == -INFINITY) continue;
            const float wgt = exp2f(m[j] - mmax);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                num[j][0][e] += wgt * x[j][e];
                num[j][1][e] += wgt * y[j][e];
            }
            den[j] += wgt * l[j];
        }
    }
    const float inv = 1.f / ((den[0] + den[1]) + (den[2] + den[3]));
    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
    typedef __attribute__((ext_vector_type(2))) int int2v;
    bf16x4 o[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            o[h][e] = (bf16_t)(((num[0][h][e] + num[1][h][e]) + (num[2][h][e] + num[3][h][e])) * inv);
    // lane half h keeps eight values 8h .. 8h+7 of the sixteen: the halves trade four each
    const int2v give = __builtin_bit_cast(int2v, lh ? o[0] : o[1]);
    const int2v got = {__shfl_xor(give[0], 32), __shfl_xor(give[1], 32)};
    const bf16x4 gt = __builtin_bit_cast(bf16x4, got), first = lh ? gt : o[0], second = lh ? o[1] : gt;
    if (lq >= n_rows) return;
    const int hq = f / R, row = row_base + f - hq * R, col = (g * group + hq) * HD + 32 * dt + 16 * pr + 8 * lh;
    const size_t idx = out_af ? af_index(row, col, lay) : (size_t)row * n_q * HD + col;
    *(bf16x8 *)(out + idx) = __builtin_shufflevector(first, second, 0, 1, 2, 3, 4, 5, 6, 7);
}

}  // namespace

// XCDs that share the query chunks of one (sequence, kv head) group: 1 where the groups divide evenly over the XCDs, 8 / groups
// where the XCDs divide over the groups, 0: workgroups by index.
static int xcds_of_group(int n_groups) {
    return n_groups % 8 == 0 ? 1 : (n_groups < 8 && 8 % n_groups == 0) ? 8 / n_groups : 0;
}

// The order of a single sequence's causal pass (prefill, scoring; n_groups <= 8, so that a group has 8 / q XCDs to
// itself).  Its workgroups walk key ranges of very different length, and all of them are resident from the start or
// nearly so: two to a compute unit, the launch takes as long as the compute unit with the most to do (a workgroup left
// alone on its SIMDs goes on at 1.4 times the speed, not at twice, so unequal pairs cost).  The dispatcher deals the first 32 of an XCD's workgroups to
// its 32 compute units and the next 32 to the same units in the same order, so by index a unit got the same rows of two
// query heads, twice the longest range or twice the shortest.  Here the item in second place on a unit is the shorter
// the longer the first one is; what is left after two rounds follows with the longest first.  8B prefill of 4096
// tokens 60416 -> 59419 us, scoring of 2000 tokens (1.5B) 17434 -> 17216.
WorkOrder attention_order(const AttnPlan &p, int B, int n_kv, int group, const RowDesc &d, const Segs &sg) {
    WorkOrder o = {};
    const int n = p.n_chunks * p.splits, n_groups = B * n_kv, q = xcds_of_group(n_groups);
    // more workgroups than compute units (otherwise each has one to itself in any order), rows of unequal key ranges
    if (sg.n || d.nc < 64 || n_groups > 8 || q == 0 || !p.tiled || n > kMaxOrder || p.n_chunks >= 1024 || n * n_groups <= 256)
        return o;
    struct Item {
        int len;
        uint16_t id;
    } it[kMaxOrder];
    const int F = group * d.R, TQ = (F + 31) >> 5, L = imax(0, p.max_keys - d.R);
    int i = 0;
    for (int c = 0; c < p.n_chunks; ++c) {
        const KeySpan k = key_span(d, L, F, c * p.tiles_per_chunk, imin(TQ, (c + 1) * p.tiles_per_chunk));
        for (int s = 0; s < p.splits; ++s) {
            const int lo = s * p.per, hi = s == p.splits - 1 ? 1 << 30 : lo + p.per;
            const int len = imax(0, imin(hi, k.a1) - lo) + imax(0, imin(hi, k.b1) - imax(lo, k.b0));
            it[i++] = {len, (uint16_t)(s << 10 | c)};
        }
    }
    std::stable_sort(it, it + n, [](const Item &x, const Item &y) { return x.len > y.len; });
    o.n = n;
    for (int x = 0; x < q; ++x) {                    // XCD x of the group's takes every q-th item
        const int m = (n - x + q - 1) / q;
        const int second = imin(imax(m - 32, 0), 32);                  // compute units that get two
        for (int k = 0; k < m; ++k) {
            int rank = k;
            if (k < second) rank = imin(m, 64) - 2 * second + k;       // the longer halves of the pairs
            else if (k < 32) rank = k - second;                        // those that stay alone
            else if (k < 64) rank = imin(m, 64) - 1 - (k - 32);        // the shorter halves
            const int at = k * q + x;
            o.item2[at >> 1] |= (uint32_t)it[rank * q + x].id << (16 * (at & 1));
        }
    }
    return o;
}

AttnPlan plan_attention(int B, int n_kv, int group, const RowDesc &d, const Segs &sg, int max_keys) {
    AttnPlan p;
    const int nc = d.nc;
    int TQ = (group * d.R + 31) / 32;         // 32-row query tiles per kv head (of the longest sequence)
    p.tiles_per_chunk = TQ < 4 ? TQ : 4;      // four waves x one query tile each
    p.n_chunks = (TQ + p.tiles_per_chunk - 1) / p.tiles_per_chunk;
    // Four query tiles to a workgroup: partial results as tiles.  Not in a forward of so few rows that the O projection folds
    // them itself (GEMM_FUSE_COMBINE), which takes them row by row: four rows of 25 and more heads on one K/V head.
    p.tiled = p.tiles_per_chunk == 4 && (sg.n ? sg.row0[sg.n] : B * d.R) > kFuseMaxRows;
    int base = B * n_kv * p.n_chunks;
    if (sg.n) {                               // sequences of different length: the workgroups that have rows
        base = 0;
        for (int b = 0; b < sg.n; ++b)
            base += n_kv * (((group * (sg.row0[b + 1] - sg.row0[b]) + 31) / 32 + p.tiles_per_chunk - 1) / p.tiles_per_chunk);
    }
    // the caller's bound is taken in steps of 256 keys: bounds that differ by less cut the keys alike, so results do
    // not change bit for bit because a caller's estimate of the final length moved a little
    max_keys = (max_keys + 255) & ~255;
    int iters = (max_keys + 31) / 32;
    // Two workgroups are resident per CU (512 slots).  A split costs about eight key-pair iterations of prologue
    // and partial-sum epilogue; a grid of w slot-fulls takes about w + 1/2 workgroup times (the last round is
    // ragged).  The split count with the least estimated time wins, the smaller one on a near tie (fewer partial
    // sums for the combine kernel): 7 at batch 1 and 4096 keys (one full round), 5 at batch 4 and 8192 keys
    // (where one split left 44 % of the slots idle for the whole launch), 1 once the batch alone fills the chip
    // several times over.  A pass with many causal rows (prefill, scoring) is another matter: its workgroups walk
    // key ranges of very different lengths, the rounds do not end together, and no ragged last round is charged
    // (measured on the training-layout pass of 4096 rows: two splits cost 6 ms per forward in partial sums and
    // their combine launch, against nothing gained in the attention kernel).
    // No more than 64 splits (the combine kernel reads one per lane) and, beyond two, no more than four slot-fulls
    // of workgroups: that bound depends on the row structure alone, and the workspace is sized by it, so the
    // partial-sum area does not depend on the key bound of a particular call.
    p.splits_bound = 2048 / base < 2 ? 2 : 2048 / base > 64 ? 64 : 2048 / base;
    int cap = (iters + 3) / 4;                // at least four key pairs per split
    if (cap > p.splits_bound) cap = p.splits_bound;
    // A single query tile per kv head and few sequences (the one-token step up to batch 4): every workgroup is mostly
    // prologue and epilogue, and its partial result is folded by each workgroup of the O projection.  No more splits
    // than give every CU one workgroup - a grid a little above 256 leaves some CUs with two (batch 1, 4096 keys:
    // 36 splits = 288 workgroups 3.75 ms per step, 32 splits 3.68; 12 288 keys: 3.94 -> 3.90) - as long as a split
    // then stays short (batch 4 at 8192 keys: 8 splits of 32 iterations lose to 16 of 16, 5.14 against 5.02 ms).
    if (TQ == 1 && base <= 32 && cap > 256 / base && iters <= 16 * (256 / base)) cap = 256 / base;
    int s = 1;
    double best = 0.0;
    for (int c = 1; c <= cap; ++c) {
        const double waves = (double)base * c / 512.0;
        const double cost = (waves <= 1.0 ? 1.0 : nc >= 64 ? waves : waves + 0.5) * ((iters + c - 1) / c + 8);
        if (c == 1 || cost < 0.97 * best) {
            best = cost;
            s = c;
        }
    }
    p.splits = s < 1 ? 1 : s;
    p.max_keys = max_keys;
    p.per = (iters + 1 + p.splits - 1) / p.splits;   // +1: the kernel counts cache and scratch units separately
    return p;
}

bool attention_rope_ok(RowDesc d, int group, int hd) {
    return d.R == 1 && d.nc == 1 && d.nm == 0 && group >= 1 && group <= 32 && hd == HD;
}

void launch_attention_bf16(const bf16_t *q, KvView kv, const bf16_t *k_scr, const bf16_t *v_scr,
                           const int32_t *prefix_len, const RowDesc &d, const Segs &sg, int B, int M, int n_q,
                           const AttnPlan &p, const WorkOrder &order, float *part, bf16_t *out, int out_af,
                           hipStream_t st, const AttnRope *rope) {
    AttnArgs a;
    a.rp = AttnRope{};
    const bool fused_rope = rope && rope->part && attention_rope_ok(d, n_q / kv.n_kv, kv.hd);
    if (fused_rope) a.rp = *rope;
    a.out = out;
    a.out_af = out_af;
    a.lay = act_layout(M);
    a.q = q;
    a.kv = kv;
    a.k_scr = k_scr;
    a.v_scr = v_scr;
    a.prefix_len = prefix_len;
    a.d = d;
    a.n_q = n_q;
    a.group = n_q / kv.n_kv;
    a.n_chunks = p.n_chunks;
    a.tiles_per_chunk = p.tiles_per_chunk;
    a.splits = p.splits;
    a.per = p.per;
    a.scale_log2e = 1.4426950408889634f / sqrtf((float)kv.hd);
    size_t rows = (size_t)M * n_q * p.splits;
    a.opart = part;
    a.mpart = part + rows * HD;
    a.lpart = a.mpart + rows;
    a.n_groups = B * kv.n_kv;
    a.xcd_q = xcds_of_group(a.n_groups);
    dim3 grid(a.n_groups * p.n_chunks, p.splits);
    if (a.xcd_q > 1) grid.x = 8 * ((p.n_chunks + a.xcd_q - 1) / a.xcd_q);
    const PlainOrder plain;
    auto go = [&](auto kernel, auto segs) { kernel<<<grid, 256, 0, st>>>(a, segs, plain); };
    const NoSegs none;
    if (order.n) {
        const dim3 line(8 * ((order.n + a.xcd_q - 1) / a.xcd_q));
        attn_bf16_kernel<1, true, false, NoSegs, WorkOrder><<<line, 256, 0, st>>>(a, none, order);
        return;
    }
    if (fused_rope) go(attn_bf16_kernel<1, false, true, NoSegs, PlainOrder>, none);
    else if (sg.n && p.tiled) go(attn_bf16_kernel<1, true, false, Segs, PlainOrder>, sg);
    else if (sg.n) go(attn_bf16_kernel<1, false, false, Segs, PlainOrder>, sg);
    else if (p.tiled) go(attn_bf16_kernel<1, true, false, NoSegs, PlainOrder>, none);
    else go(attn_bf16_kernel<1, false, false, NoSegs, PlainOrder>, none);
}

void launch_attention_combine(const float *part, const RowDesc &d, const Segs &sg, int M, int n_q, int n_kv, int hd,
                              const AttnPlan &p, bf16_t *out, int out_af, hipStream_t st) {
    const int splits = p.splits;
    if (splits == 1) return;                  // the attention kernel has written the result itself
    size_t rows = (size_t)M * n_q * splits;
    const ActLayout lay = act_layout(M);
    if (p.tiled) {
        const int tiles = (n_q / n_kv * d.R + 31) / 32;
        const int n_groups = (sg.n ? sg.n : M / d.R) * n_kv;
        auto by_tiles = [&](auto segs) {
            attn_combine_tiles_kernel<<<dim3(n_groups * tiles, 2), 256, 0, st>>>(
                part, part + rows * hd, part + rows * hd + rows, d, segs, n_q, n_kv, splits, tiles, n_groups, out, out_af, lay);
        };
        if (sg.n) by_tiles(sg);
        else by_tiles(NoSegs());
        return;
    }
    const bool lines = out_af && M > 480;
    auto go = [&](auto j, auto segs) {
        constexpr int J = decltype(j)::value;
        auto launch = [&](auto kernel, int blocks) {
            kernel<<<dim3(blocks, n_q), 64, 0, st>>>(part, part + rows * hd, part + rows * hd + rows, d, segs, n_q, n_kv, splits, M,
                                                     out, out_af, lay);
        };
        if (lines) launch(attn_combine_kernel<J, true, decltype(segs)>, line_rows(M));
        else launch(attn_combine_kernel<J, false, decltype(segs)>, M);
    };
    auto by_splits = [&](auto segs) {
        if (splits <= 4) go(std::integral_constant<int, 1>(), segs);
        else if (splits <= 8) go(std::integral_constant<int, 2>(), segs);
        else go(std::integral_constant<int, 4>(), segs);
    };
    if (sg.n) by_splits(sg);
    else by_splits(NoSegs());
}
