// Small kernels of the decode step: weight packing, row assembly + embedding gather, RMSNorm with fused
// residual/split-K reduction, RoPE + K/V placement, SwiGLU, vocabulary argmax / Gumbel-max, verify/accept.
// Also the fp32-mode GEMM and attention (plain ALU kernels used by the fp32 configuration).
#include <type_traits>

#include "tidar_internal.h"

namespace {

template <typename T> __device__ inline float to_f(T v);
template <> __device__ inline float to_f<float>(float v) { return v; }
template <> __device__ inline float to_f<bf16_t>(bf16_t v) { return (float)v; }
template <typename T> __device__ inline T from_f(float v);
template <> __device__ inline float from_f<float>(float v) { return v; }
template <> __device__ inline bf16_t from_f<bf16_t>(float v) { return (bf16_t)v; }   // round to nearest even

template <typename T> __device__ inline void store4(T *p, float a, float b, float c, float d);
template <> __device__ inline void store4<float>(float *p, float a, float b, float c, float d) {
    *(float4 *)p = make_float4(a, b, c, d);
}
template <> __device__ inline void store4<bf16_t>(bf16_t *p, float a, float b, float c, float d) {
    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
    bf16x4 v = {(bf16_t)a, (bf16_t)b, (bf16_t)c, (bf16_t)d};
    *(bf16x4 *)p = v;
}

__device__ inline float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}
__device__ inline float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}

// ------------------------------------------------------------------ weight packing
// bf16 destination: [k step of 16][32-row tile][lane][8], lane = (k/8 % 2) * 32 + row % 32: the register image
// of the 32x32x16 MFMA B operand.  The k step is outermost: all workgroups of a GEMM advance through K together,
// so at any moment they read one contiguous front of the matrix, which spreads over every HBM channel.
// Source row r lands in destination row 16 * (tile_off + (r / 16) * tile_stride) + r % 16.
__global__ void pack_bf16_kernel(const bf16_t *__restrict__ src, int rows, int K, bf16_t *__restrict__ dst,
                                 int dst_tiles32, int tile_off, int tile_stride) {
    const int k8 = K / 8;
    size_t n = (size_t)rows * k8;                               // one 16-byte piece per index
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n;
         idx += (size_t)gridDim.x * blockDim.x) {
        int r = (int)(idx / k8);
        int k = 8 * (int)(idx % k8);
        int rd = 16 * (tile_off + (r >> 4) * tile_stride) + (r & 15);
        size_t o = ((((size_t)(k >> 4) * dst_tiles32 + (rd >> 5)) * 64) + ((k >> 3) & 1) * 32 + (rd & 31)) * 8;
        *(bf16x8 *)(dst + o) = *(const bf16x8 *)(src + (size_t)r * K + k);
    }
}

// fp32: plain row-major; tile placement only.
__global__ void pack_f32_kernel(const float *__restrict__ src, int rows, int K, float *__restrict__ dst,
                                int tile_off, int tile_stride) {
    size_t n = (size_t)rows * K;
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += (size_t)gridDim.x * blockDim.x) {
        int r = (int)(idx / K);
        int c = (int)(idx % K);
        size_t dr = (size_t)(tile_off + (r / 16) * tile_stride) * 16 + (r % 16);
        dst[dr * K + c] = src[idx];
    }
}

// ------------------------------------------------------------------ row assembly + embedding gather (+ RoPE table)
template <typename T, class SG>
__global__ void embed_rows_kernel(const T *__restrict__ embed, const int32_t *__restrict__ tokens, int tok_stride,
                                  const int32_t *__restrict__ prefix_len, RowDesc d_any, SG sg, int d_model,
                                  int mask_id, int vocab, KvView kv, int hd, float rope_base, float *__restrict__ x,
                                  int32_t *__restrict__ pos_out, int n_head, float *__restrict__ rope_cs) {
    int row = blockIdx.x;
    int b = seq_of_row(d_any, sg, row), row_base;
    const RowDesc d = seq_desc(d_any, sg, b, &row_base);
    int r = row - row_base;
    int L = clamp_prefix(kv, prefix_len[d.seq_base + b], d.nc);
    RowInfo ri = row_info(d, r, L);
    int tok = (r < d.nc) ? tokens[(size_t)b * tok_stride + r] : mask_id;
    if ((unsigned)tok >= (unsigned)vocab) tok = mask_id;      // an id outside the table is never dereferenced (the
                                                              // kernel that finishes the call reports it)
    // sequences of different row counts: the n_head rows of each that go through the LM head, one after the other
    if (threadIdx.x == 0) {
        if (!kSegs<SG>) pos_out[row] = ri.pos;
        else if (r >= d.R - n_head) pos_out[b * n_head + r - (d.R - n_head)] = ri.pos;
    }
    const T *e = embed + (size_t)tok * d_model;
    float *xo = x + (size_t)row * d_model;
    for (int c = threadIdx.x; c < d_model; c += blockDim.x) xo[c] = to_f<T>(e[c]);
    // cos/sin of pos * base^(-2i/hd), angle formed in double so that long contexts keep their phase
    int half = hd / 2;
    for (int i = threadIdx.x; i < half; i += blockDim.x) {
        double inv = exp2(-(double)(2 * i) / (double)hd * log2((double)rope_base));
        double ang = (double)ri.pos * inv;
        double s, c;
        sincos(ang, &s, &c);
        rope_cs[((size_t)row * half + i) * 2 + 0] = (float)c;
        rope_cs[((size_t)row * half + i) * 2 + 1] = (float)s;
    }
}

// ------------------------------------------------------------------ residual add (split-K partials) + RMSNorm
// One block per output row.  part: tiled GEMM output over M_all rows; out: A-fragment layout over the selected rows.
// A row is a workgroup's only work and what bounds it is latency, so the host gives it a thread per 4-column piece (up to
// 1024): all loads are in flight at once and a piece stays in its thread's registers across the barrier (pieces beyond the
// first of a thread, in rows wider than that, are read again).  Where the output is in lines of eight rows (LINES) the
// workgroups of a line's rows run on one XCD.  Against 256 threads per row above 64 rows, the row read again and lines
// written by eight XCDs: 1.5B step k = 16 3106 -> 3048 us, 8B 8178 -> 8117, 8B k = 4 4324 -> 4293, one-token step of 6
// sequences (1.5B) 1562 -> 1548.
template <typename T, bool LINES, class SG>
__global__ __launch_bounds__(1024) void rmsnorm_kernel(float *__restrict__ x, const float *__restrict__ part, int S,
                                                      size_t split_stride, const T *__restrict__ gain, float eps,
                                                      int n_rows, int R, SG sg, int d_model, int M_all, int rows,
                                                      T *__restrict__ out, ActLayout lay) {
    const int o_row = LINES ? line_row(blockIdx.x) : blockIdx.x;
    if (LINES && o_row >= rows) return;              // whole workgroup
    const int b = o_row / n_rows;
    const int o = o_row - b * n_rows;
    int row = (b + 1) * R - n_rows + o;
    if constexpr (kSegs<SG>) row = sg.row0[b + 1] - n_rows + o;
    float *xr = x + (size_t)row * d_model;
    auto residual = [&](int c) __attribute__((always_inline)) {
        float4 v = *(const float4 *)(xr + c);
        if (S > 0) {
            const float *pp = part + pt_index(c, row, M_all);
            int sp = 0;
            for (; sp + 4 <= S; sp += 4) {         // four independent loads at a time, summed in split order
                const float4 q0 = *(const float4 *)(pp + (size_t)sp * split_stride);
                const float4 q1 = *(const float4 *)(pp + (size_t)(sp + 1) * split_stride);
                const float4 q2 = *(const float4 *)(pp + (size_t)(sp + 2) * split_stride);
                const float4 q3 = *(const float4 *)(pp + (size_t)(sp + 3) * split_stride);
                v.x = (((v.x + q0.x) + q1.x) + q2.x) + q3.x;
                v.y = (((v.y + q0.y) + q1.y) + q2.y) + q3.y;
                v.z = (((v.z + q0.z) + q1.z) + q2.z) + q3.z;
                v.w = (((v.w + q0.w) + q1.w) + q2.w) + q3.w;
            }
            for (; sp < S; ++sp) {
                const float4 q = *(const float4 *)(pp + (size_t)sp * split_stride);
                v.x += q.x; v.y += q.y; v.z += q.z; v.w += q.w;
            }
            *(float4 *)(xr + c) = v;
        }
        return v;
    };
    auto squares = [](const float4 &v) { return v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w; };
    const int c0 = 4 * threadIdx.x;
    float4 mine = {0.f, 0.f, 0.f, 0.f}, g0 = mine;
    if (c0 < d_model) {
        g0 = {to_f<T>(gain[c0]), to_f<T>(gain[c0 + 1]), to_f<T>(gain[c0 + 2]), to_f<T>(gain[c0 + 3])};
        mine = residual(c0);
    }
    float ss = squares(mine);
    for (int c = c0 + 4 * blockDim.x; c < d_model; c += 4 * blockDim.x) ss += squares(residual(c));
    __shared__ float red[16];
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) tot += red[w];
    const float rs = rsqrtf(tot / (float)d_model + eps);
    if (c0 < d_model)
        store4<T>(out + af_index(o_row, c0, lay), mine.x * rs * g0.x, mine.y * rs * g0.y, mine.z * rs * g0.z, mine.w * rs * g0.w);
    for (int c = c0 + 4 * blockDim.x; c < d_model; c += 4 * blockDim.x) {
        float4 v = *(const float4 *)(xr + c);          // this thread's own writes
        store4<T>(out + af_index(o_row, c, lay), v.x * rs * to_f<T>(gain[c]), v.y * rs * to_f<T>(gain[c + 1]),
                  v.z * rs * to_f<T>(gain[c + 2]), v.w * rs * to_f<T>(gain[c + 3]));
    }
}

// The same for many rows (bf16): a wave per row, four consecutive rows per workgroup, and the two workgroups of eight rows on
// one XCD (workgroup i of a launch runs on XCD i % 8).  With one workgroup per row a 128-byte line of the output holds
// pieces of eight rows and is written by eight workgroups on eight XCDs, a part each, and the row is read again behind
// a workgroup barrier; here a line stays in one L2, and the row in registers (JP pieces of 8 columns per lane: up to
// 512 JP columns), with the loads of the residual stream and of the first split in flight together.  It is bound by memory
// (2176 x 4096 in two splits: 160 MB).  One workgroup per row -> this: 2176 x 4096 47 -> 37 us, 2048 x 4096 39.5 -> 28.4,
// 4000 x 1536 27.1 -> 20.5, 816 x 4096 20.6 -> 17.7, 544 x 4096 14.8 -> 14.1, 544 x 1536 7.3 -> 7.1; 272 x 4096 9.7 -> 12.3.
template <int JP, class SG>
__global__ __launch_bounds__(256) void rmsnorm_rows_kernel(float *__restrict__ x, const float *__restrict__ part, int S,
                                                           size_t split_stride, const bf16_t *__restrict__ gain, float eps,
                                                           int n_rows, int R, SG sg, int d_model, int M_all, int rows,
                                                           bf16_t *__restrict__ out, ActLayout lay) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int eight = (blockIdx.x >> 4) * 8 + (blockIdx.x & 7), half = (blockIdx.x >> 3) & 1;
    const int o_row = eight * 8 + half * 4 + wave;
    if (o_row >= rows) return;                      // no barrier in this kernel
    const int b = o_row / n_rows;
    int row = (b + 1) * R - n_rows + (o_row - b * n_rows);
    if constexpr (kSegs<SG>) row = sg.row0[b + 1] - n_rows + (o_row - b * n_rows);
    float *xr = x + (size_t)row * d_model;
    float4 v[JP][2], q[JP][2];
    auto load = [&](int sp) __attribute__((always_inline)) {
        const float *pp = part + (size_t)sp * split_stride;
#pragma unroll
        for (int j = 0; j < JP; ++j) {
            const float *s = pp + pt_index(min(8 * (lane + 64 * j), d_model - 8), row, M_all);      // clamped: a real address
            q[j][0] = *(const float4 *)s;
            q[j][1] = *(const float4 *)(s + 4);
        }
    };
#pragma unroll
    for (int j = 0; j < JP; ++j) {
        const int k = min(8 * (lane + 64 * j), d_model - 8);
        v[j][0] = *(const float4 *)(xr + k);
        v[j][1] = *(const float4 *)(xr + k + 4);
    }
    if (S > 0) load(0);
    __builtin_amdgcn_sched_barrier(0);
    for (int sp = 0; sp < S; ++sp) {                // in split order
#pragma unroll
        for (int j = 0; j < JP; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                v[j][h].x += q[j][h].x; v[j][h].y += q[j][h].y; v[j][h].z += q[j][h].z; v[j][h].w += q[j][h].w;
            }
        if (sp + 1 < S) load(sp + 1);
    }
    float ss = 0.f;
#pragma unroll
    for (int j = 0; j < JP; ++j) {
        const int k = 8 * (lane + 64 * j);
        if (k >= d_model) continue;
#pragma unroll
        for (int h = 0; h < 2; ++h)
            ss += v[j][h].x * v[j][h].x + v[j][h].y * v[j][h].y + v[j][h].z * v[j][h].z + v[j][h].w * v[j][h].w;
        if (S > 0) {
            *(float4 *)(xr + k) = v[j][0];
            *(float4 *)(xr + k + 4) = v[j][1];
        }
    }
    const float rs = rsqrtf(wave_sum(ss) / (float)d_model + eps);
#pragma unroll
    for (int j = 0; j < JP; ++j) {
        const int k = 8 * (lane + 64 * j);
        if (k >= d_model) continue;
        const bf16x8 g = *(const bf16x8 *)(gain + k);
        const bf16x8 o = {(bf16_t)(v[j][0].x * rs * (float)g[0]), (bf16_t)(v[j][0].y * rs * (float)g[1]),
                          (bf16_t)(v[j][0].z * rs * (float)g[2]), (bf16_t)(v[j][0].w * rs * (float)g[3]),
                          (bf16_t)(v[j][1].x * rs * (float)g[4]), (bf16_t)(v[j][1].y * rs * (float)g[5]),
                          (bf16_t)(v[j][1].z * rs * (float)g[6]), (bf16_t)(v[j][1].w * rs * (float)g[7])};
        *(bf16x8 *)(out + af_index(o_row, k, lay)) = o;
    }
}

// ------------------------------------------------------------------ RoPE + K/V placement
// blockIdx.x < rows: one row, blockIdx.y = slice of the row's work (Q rotation, K rotation and placement).
// blockIdx.x >= rows: one 16-key V tile of one sequence (a cache page the causal rows touch, or a scratch tile of
// the mask rows), blockIdx.y = slice of its (kv head, d) pairs.  V is kept transposed ([d][16 keys]); written row
// by row that is one 2-byte store per value, 32 bytes apart (measured: 2.8 times the bytes at the memory side and
// half of this kernel's time at batch 32), so the tile blocks gather by (head, d) and write whole pieces.
// qkv_part: tiled GEMM output, [S] x (q_dim + 2 kv_dim) columns.  Q rows -> q_out [M][q_dim];
// K/V of causal rows -> cache at position L + r; K/V of mask rows -> scratch tiles
// k_scr [B][n_kv][n_mtiles][16][hd], v_scr [B][n_kv][n_mtiles][hd][16].
template <typename T, class SG>
__global__ __launch_bounds__(256) void rope_kv_kernel(const float *__restrict__ part, int S, size_t split_stride,
                                                      const float *__restrict__ rope_cs,
                                                      const int32_t *__restrict__ prefix_len, RowDesc d_any, SG sg,
                                                      int n_q, int M_all, KvView kv, T *__restrict__ q_out,
                                                      T *__restrict__ k_scr, T *__restrict__ v_scr) {
    const int hd = kv.hd, half = hd / 2, n_kv = kv.n_kv;
    const int q_dim = n_q * hd, kv_dim = n_kv * hd;
    if ((int)blockIdx.x >= M_all) {
        // item = (kv head, d, quarter of the tile's 16 keys): four keys gathered, 8 bytes (bf16) written; the four
        // quarters of a d are neighbouring lanes, so a wave still writes one contiguous run
        const int n_ct = (d_any.nc + 15) / 16 + 1;       // cache pages the causal rows (of the longest sequence) can touch
        const int n_mtiles = (d_any.nm + 15) / 16;
        const int items = n_kv * hd * 4;
        const int per_blk = gridDim.y * blockDim.x;
        const int parts = (items + per_blk - 1) / per_blk;
        int vb = blockIdx.x - M_all;
        const int part_i = vb % parts;
        vb /= parts;
        const int b = vb / (n_ct + n_mtiles), t = vb - b * (n_ct + n_mtiles);
        int row_base;
        const RowDesc d = seq_desc(d_any, sg, b, &row_base);
        const int idx = (part_i * gridDim.y + blockIdx.y) * blockDim.x + threadIdx.x;
        if (idx >= items) return;
        const int L_raw = prefix_len[d.seq_base + b];
        const int L = clamp_prefix(kv, L_raw, d.nc);
        int r0, lo, hi;                                  // the tile's key s is row r0 + s; keys [lo, hi) exist
        T *base;                                         // [n_kv][hd][16] of this tile, strided per head by hstride
        size_t hstride;
        if (t < n_ct) {
            if (!seq_fits(kv, L_raw, d.nc)) return;      // a sequence that does not fit stores nothing in the cache
            const int p = (L >> 4) + t;
            r0 = 16 * p - L;
            lo = max(0, -r0);
            hi = min(16, d.nc - r0);
            if (hi <= lo) return;
            const int page = kv.page_table[(size_t)(d.seq_base + b) * kv.pages_per_seq + p];
            if (!page_ok(kv, page)) return;
            base = (T *)kv.v_pages + v_page_offset(kv, page, 0, 0, 0);
            hstride = (size_t)hd * 16;
        } else {
            const int mt = t - n_ct;
            r0 = d.nc + 16 * mt;
            lo = 0;
            hi = min(16, d.nm - 16 * mt);
            base = v_scr + (size_t)b * n_kv * n_mtiles * hd * 16 + (size_t)mt * hd * 16;
            hstride = (size_t)n_mtiles * hd * 16;
        }
        const int qd = idx & 3, hdd = idx >> 2;
        const int h = hdd / hd, dd = hdd - h * hd;
        const int s0 = 4 * qd;
        T *dst = base + h * hstride + (size_t)dd * 16 + s0;
        const bool keep = t < n_ct && (s0 < lo || s0 + 4 > hi);     // slots of earlier or later tokens in this piece
        T vals[4];
        if (keep) {
#pragma unroll
            for (int e = 0; e < 4; ++e) vals[e] = dst[e];
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) vals[e] = from_f<T>(0.f);
        }
        const float *pp[4];
        float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int s = min(max(s0 + e, lo), hi - 1);       // clamped: an existing row, value unused if outside
            pp[e] = part + pt_index(q_dim + kv_dim + h * hd + dd, row_base + r0 + s, M_all);
        }
#pragma unroll 4
        for (int sp = 0; sp < S; ++sp) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += pp[e][(size_t)sp * split_stride];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (s0 + e >= lo && s0 + e < hi) vals[e] = from_f<T>(v[e]);
        typedef T vec4 __attribute__((ext_vector_type(4)));
        *(vec4 *)dst = (vec4){vals[0], vals[1], vals[2], vals[3]};
        return;
    }
    const int row = blockIdx.x;
    const int b = seq_of_row(d_any, sg, row);
    int row_base;
    const RowDesc d = seq_desc(d_any, sg, b, &row_base);
    const int r = row - row_base;
    const int per_head = half / 4;                   // groups of four rotation pairs
    const float *cs = rope_cs + (size_t)row * half * 2;
    auto val4 = [&](int col) {
        const float *pp = part + pt_index(col, row, M_all);
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
        for (int sp = 0; sp < S; ++sp) {
            float4 q = *(const float4 *)(pp + (size_t)sp * split_stride);
            v.x += q.x; v.y += q.y; v.z += q.z; v.w += q.w;
        }
        return v;
    };
    auto rotate = [&](float4 a, float4 bb, int i, float4 &lo, float4 &hi) {
        float4 c0 = *(const float4 *)(cs + 2 * i), c1 = *(const float4 *)(cs + 2 * i + 4);   // (cos,sin) x 4
        lo = make_float4(a.x * c0.x - bb.x * c0.y, a.y * c0.z - bb.y * c0.w, a.z * c1.x - bb.z * c1.y,
                         a.w * c1.z - bb.w * c1.w);
        hi = make_float4(bb.x * c0.x + a.x * c0.y, bb.y * c0.z + a.y * c0.w, bb.z * c1.x + a.z * c1.y,
                         bb.w * c1.z + a.w * c1.w);
    };
    // blockIdx.y: the first q_blocks workgroups of a row rotate Q (one item per thread), the rest place K/V
    const int q_blocks = (n_q * per_head + blockDim.x - 1) / blockDim.x;
    if ((int)blockIdx.y < q_blocks) {
        const int idx = blockIdx.y * blockDim.x + threadIdx.x;
        if (idx < n_q * per_head) {
            int h = idx / per_head, i = 4 * (idx - h * per_head);
            float4 lo, hi;
            rotate(val4(h * hd + i), val4(h * hd + i + half), i, lo, hi);
            T *qo = q_out + (size_t)row * q_dim + h * hd + i;
            store4<T>(qo, lo.x, lo.y, lo.z, lo.w);
            store4<T>(qo + half, hi.x, hi.y, hi.z, hi.w);
        }
        return;
    }
    // destination of this row's K/V
    const bool causal = r < d.nc;
    const int L_raw = prefix_len[d.seq_base + b];
    const int L = clamp_prefix(kv, L_raw, d.nc);
    int page = 0, slot = 0, mt = 0;
    const int n_mtiles = (d.nm + 15) / 16;
    if (causal) {
        int p = L + r;
        page = kv.page_table[(size_t)(d.seq_base + b) * kv.pages_per_seq + (p >> 4)];
        slot = p & 15;
        if (!seq_fits(kv, L_raw, d.nc) || !page_ok(kv, page)) return;     // nothing of this row reaches the cache
    } else {
        int m = r - d.nc;
        mt = m >> 4;
        slot = m & 15;
    }
    T *kp = (T *)kv.k_pages;
    for (int idx = (blockIdx.y - q_blocks) * blockDim.x + threadIdx.x; idx < n_kv * per_head;
         idx += (gridDim.y - q_blocks) * blockDim.x) {
        int h = idx / per_head, i = 4 * (idx - h * per_head);
        float4 lo, hi;
        rotate(val4(q_dim + h * hd + i), val4(q_dim + h * hd + i + half), i, lo, hi);
        T *kdst;                   // K: [slot][hd] contiguous in d (V goes by tiles, above)
        if (causal) {
            kdst = kp + k_page_offset(kv, page, h, slot, 0);
        } else {
            size_t tile = ((size_t)b * n_kv + h) * n_mtiles + mt;
            kdst = k_scr + (tile * 16 + slot) * hd;
        }
        store4<T>(kdst + i, lo.x, lo.y, lo.z, lo.w);
        store4<T>(kdst + i + half, hi.x, hi.y, hi.z, hi.w);
    }
}

// K/V given directly (attention entry point): same placement, no rotation.
template <typename T>
__global__ void place_kv_kernel(const T *__restrict__ k_new, const T *__restrict__ v_new,
                                const int32_t *__restrict__ prefix_len, RowDesc d, KvView kv, T *__restrict__ k_scr,
                                T *__restrict__ v_scr) {
    int row = blockIdx.x;
    int b = row / d.R;
    int r = row - b * d.R;
    int hd = kv.hd, n_kv = kv.n_kv;
    bool causal = r < d.nc;
    const int L_raw = prefix_len[d.seq_base + b];
    int L = clamp_prefix(kv, L_raw, d.nc);
    int page = 0, slot = 0, mt = 0;
    int n_mtiles = (d.nm + 15) / 16;
    if (causal) {
        int p = L + r;
        page = kv.page_table[(size_t)(d.seq_base + b) * kv.pages_per_seq + (p >> 4)];
        slot = p & 15;
        if (!seq_fits(kv, L_raw, d.nc) || !page_ok(kv, page)) return;
    } else {
        int m = r - d.nc;
        mt = m >> 4;
        slot = m & 15;
    }
    T *kp = (T *)kv.k_pages;
    T *vp = (T *)kv.v_pages;
    for (int idx = threadIdx.x; idx < n_kv * hd; idx += blockDim.x) {
        int h = idx / hd, i = idx - h * hd;
        T kk = k_new[(size_t)row * n_kv * hd + idx], vv = v_new[(size_t)row * n_kv * hd + idx];
        if (causal) {
            kp[k_page_offset(kv, page, h, slot, i)] = kk;
            vp[v_page_offset(kv, page, h, slot, i)] = vv;
        } else {
            size_t tile = ((size_t)b * n_kv + h) * n_mtiles + mt;
            k_scr[(tile * 16 + slot) * hd + i] = kk;
            v_scr[(tile * hd + i) * 16 + slot] = vv;
        }
    }
}

// ------------------------------------------------------------------ SwiGLU over interleaved gate/up columns
// part: tiled GEMM output with 2*d_ff columns (tile 2t = gate, 2t+1 = up); out: A-fragment layout, K = d_ff.
template <typename T>
__global__ void swiglu_kernel(const float *__restrict__ part, int S, size_t split_stride, int M, int d_ff,
                              T *__restrict__ out, ActLayout lay) {
    const int per_row = d_ff / 4;
    size_t n = (size_t)M * per_row;
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += (size_t)gridDim.x * blockDim.x) {
        // consecutive threads walk down the rows of one column group: the tiled layout is row-contiguous
        int row = (int)(idx % M);
        int f = 4 * (int)(idx / M);
        const float *pg = part + pt_index(32 * (f >> 4) + (f & 15), row, M);
        const float *pu = part + pt_index(32 * (f >> 4) + 16 + (f & 15), row, M);
        float4 g = make_float4(0.f, 0.f, 0.f, 0.f), u = g;
        for (int sp = 0; sp < S; ++sp) {
            float4 a = *(const float4 *)(pg + (size_t)sp * split_stride);
            float4 c = *(const float4 *)(pu + (size_t)sp * split_stride);
            g.x += a.x; g.y += a.y; g.z += a.z; g.w += a.w;
            u.x += c.x; u.y += c.y; u.z += c.z; u.w += c.w;
        }
        store4<T>(out + af_index(row, f, lay), g.x / (1.f + __expf(-g.x)) * u.x, g.y / (1.f + __expf(-g.y)) * u.y,
                  g.z / (1.f + __expf(-g.z)) * u.z, g.w / (1.f + __expf(-g.w)) * u.w);
    }
}

// ------------------------------------------------------------------ vocabulary argmax / Gumbel-max
// One block per (sequence, row o < n_rows) over materialised logits with Rh rows per sequence.  With few rows it is a
// chain of trips to memory, with many a stream: U pieces of W columns per thread are on their way at a time (one
// column at a time: 20 rows of 151 936 72 us, 272 rows 93 us; now 24 and 58).  W = 4: 16-byte aligned rows.
template <int W>
__global__ __launch_bounds__(1024) void argmax_rows_kernel(const float *__restrict__ logits, int Rh, int n_rows, int vocab, int n_choose,
                                   const int32_t *__restrict__ pos_rows, int pos_stride, int pos_row0, int seq_base,
                                   int sample, float temperature, uint64_t seed, float beta, int mix_base,
                                   int mix_stride, int32_t *__restrict__ y, int y_stride) {
    int b = blockIdx.x / n_rows;
    int o = blockIdx.x - b * n_rows;
    const float *lg = logits + ((size_t)b * Rh + o) * vocab;
    bool choose = o < n_choose;            // a row whose token is *taken* (causal logits)
    const float *mix = nullptr;
    if (choose && beta != 1.0f) mix = logits + ((size_t)b * Rh + mix_base + (size_t)o * mix_stride) * vocab;
    bool noisy = choose && sample;
    uint64_t key = 0;
    float inv_t = 1.f;
    if (noisy) {
        int pos_pred = pos_rows[(size_t)b * pos_stride + pos_row0 + o] + 1;      // causal rows are label shifted
        key = noise_key(seed, seq_base + b, pos_pred);
        inv_t = 1.f / temperature;
    }
    float best = -INFINITY;
    int best_i = 0x7fffffff;
    constexpr int U = 8;
    typedef float vec __attribute__((ext_vector_type(W)));
    auto take = [&](float val, float other, int v) {
        if (mix) val = beta * val + (1.f - beta) * other;
        if (noisy) val = perturbed_logit(val, inv_t, key, (uint32_t)v);
        if (val > best || (val == best && v < best_i)) { best = val; best_i = v; }
    };
    for (int v0 = W * threadIdx.x; v0 < vocab; v0 += U * W * blockDim.x) {      // vocab is a multiple of W
        vec x[U], m[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int v = min(v0 + u * W * (int)blockDim.x, vocab - W);             // clamped: always a real address
            x[u] = *(const vec *)(lg + v);
            if (mix) m[u] = *(const vec *)(mix + v);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int v = v0 + u * W * (int)blockDim.x;
            if (v >= vocab) break;
#pragma unroll
            for (int e = 0; e < W; ++e) take(x[u][e], mix ? m[u][e] : 0.f, v + e);
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        float ob = __shfl_xor(best, off);
        int oi = __shfl_xor(best_i, off);
        if (ob > best || (ob == best && oi < best_i)) { best = ob; best_i = oi; }
    }
    __shared__ float sb[16];
    __shared__ int si[16];
    if ((threadIdx.x & 63) == 0) { sb[threadIdx.x >> 6] = best; si[threadIdx.x >> 6] = best_i; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w)
            if (sb[w] > best || (sb[w] == best && si[w] < best_i)) { best = sb[w]; best_i = si[w]; }
        y[(size_t)b * y_stride + o] = best_i == 0x7fffffff ? -1 : best_i;     // a row without a single number
                                                                              // (all NaN) has no token
    }
}

// ------------------------------------------------------------------ log-probability of a label under a row of logits
// One block per row of one scoring pass over text positions [c0, c0 + nc) of a sequence of `len` tokens.  Causal row
// r is label shifted (Section 3.1): it scores token c0 + r + 1 into ar_out[c0 + r] (0 when the text ends there);
// mask row m is scored against the token it stands in for, c0 + m, into diff_out[c0 + m].
// log p = logit[label] - (max + ln sum exp(logit - max)), two passes over the row.
__global__ __launch_bounds__(1024) void score_rows_kernel(const float *__restrict__ logits, int vocab,
                                                         const int32_t *__restrict__ text, int len, int c0, int nc,
                                                         float *__restrict__ ar_out, float *__restrict__ diff_out) {
    const int r = blockIdx.x;
    const float *lg = logits + (size_t)r * vocab;
    const bool causal = r < nc;
    const int i = c0 + (causal ? r : r - nc);
    const int li = causal ? i + 1 : i;
    float *dst = (causal ? ar_out : diff_out) + i;
    if (li >= len) {                       // uniform over the block
        if (threadIdx.x == 0) *dst = 0.f;
        return;
    }
    const int label = text[li];
    if ((unsigned)label >= (unsigned)vocab) {     // uniform over the block: an id outside the vocabulary scores NaN
        if (threadIdx.x == 0) *dst = __builtin_nanf("");
        return;
    }
    __shared__ float red[16];
    __shared__ float bc;
    const int nw = blockDim.x >> 6;
    float mx = -INFINITY;
    for (int v = 4 * threadIdx.x; v < vocab; v += 4 * blockDim.x) {        // vocab is a multiple of 16
        const float4 q = *(const float4 *)(lg + v);
        mx = fmaxf(fmaxf(mx, fmaxf(q.x, q.y)), fmaxf(q.z, q.w));
    }
    mx = wave_max(mx);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        float m = red[0];
        for (int w = 1; w < nw; ++w) m = fmaxf(m, red[w]);
        bc = m;
    }
    __syncthreads();
    mx = bc;
    float sum = 0.f;
    for (int v = 4 * threadIdx.x; v < vocab; v += 4 * blockDim.x) {
        const float4 q = *(const float4 *)(lg + v);
        sum += (expf(q.x - mx) + expf(q.y - mx)) + (expf(q.z - mx) + expf(q.w - mx));
    }
    sum = wave_sum(sum);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.f;
        for (int w = 0; w < nw; ++w) t += red[w];
        *dst = lg[label] - (mx + logf(t));
    }
}

// Section 3.1 objective of one sequence from its per-token log-probabilities: both sums run over the first len-1
// entries and are divided by len-1; the causal one is weighted by alpha, the total by 1/(1+alpha).  Without a mask
// section (diff == nullptr) the result is the plain mean negative log-likelihood.  One block, fixed summation order;
// n = len - 1.
__global__ __launch_bounds__(256) void score_loss_kernel(const float *__restrict__ ar, const float *__restrict__ diff,
                                                        int n, float alpha, float *__restrict__ loss) {
    float sa = 0.f, sd = 0.f;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        sa += ar[i];
        if (diff) sd += diff[i];
    }
    sa = wave_sum(sa);
    sd = wave_sum(sd);
    __shared__ float ra[4], rd[4];
    if ((threadIdx.x & 63) == 0) { ra[threadIdx.x >> 6] = sa; rd[threadIdx.x >> 6] = sd; }
    __syncthreads();
    if (threadIdx.x == 0) {
        const float ta = ((ra[0] + ra[1]) + ra[2]) + ra[3], td = ((rd[0] + rd[1]) + rd[2]) + rd[3];
        float v = 0.f;
        if (n > 0) v = diff ? (alpha * (-ta / n) + (-td / n)) / (1.f + alpha) : -ta / n;
        *loss = v;
    }
}

// ------------------------------------------------------------------ verify / accept / commit / next-draft select
// y: [B][k(k+1)] chosen token per row (rows: c_0..c_{k-1}, blk_0[0..k), ...).  One wavefront per sequence: lane i
// holds draft i, the token its causal row chose and the answer to "is draft i what row i-1 chose"; the acceptance
// length is the position of the first lane that says no.  The same wavefront is the call's device-side checker:
// a sequence that did not fit the page table, that wrote through a page id outside the pool, that was fed a token
// id outside the vocabulary or whose needed rows chose no token (all NaN) is reported with accepted_len 0, its
// tokens -1 and its prefix length untouched (the forward stored nothing of it where the store was unsafe).
__global__ __launch_bounds__(64) void verify_step_kernel(const int32_t *__restrict__ y,
                                                         const int32_t *__restrict__ drafts, int k, int vocab,
                                                         KvView kv, int seq_base, int32_t *__restrict__ prefix_len,
                                                         int32_t *__restrict__ accepted_len,
                                                         int32_t *__restrict__ accepted_tokens,
                                                         int32_t *__restrict__ next_drafts) {
    const int b = blockIdx.x, lane = threadIdx.x;
    const int R = k * (k + 1);
    const int32_t *yb = y + (size_t)b * R;
    const int L = prefix_len[b];
    const bool fits = seq_fits(kv, L, k);
    const bool mine = lane < k;
    const int c = mine ? drafts[(size_t)b * k + lane] : 0;
    const int y_prev = (mine && lane > 0) ? yb[lane - 1] : 0;            // causal row i-1 judges draft i
    bool bad = mine && (unsigned)c >= (unsigned)vocab;
    if (mine && fits) {
        const int page = kv.page_table[(size_t)(seq_base + b) * kv.pages_per_seq + ((L + lane) >> 4)];
        bad = bad || !page_ok(kv, page);
    }
    const unsigned long long no = __ballot(mine && lane > 0 && c != y_prev) | (1ull << k);
    const int a = __ffsll((long long)no) - 1;                            // first rejected draft = tokens accepted, 1..k
    const int nxt = !mine ? 0 : lane == 0 ? yb[a - 1] : yb[k + (a - 1) * k + lane];
    bad = bad || (mine && nxt < 0);
    const bool err = !fits || __ballot(bad) != 0ull;
    if (mine) {
        accepted_tokens[(size_t)b * k + lane] = (!err && lane < a) ? c : -1;
        next_drafts[(size_t)b * k + lane] = err ? -1 : nxt;
    }
    if (lane == 0) {
        accepted_len[b] = err ? 0 : a;
        if (!err) prefix_len[b] = L + a;           // commit: rejected drafts' K/V fall behind the frontier
    }
}

__global__ __launch_bounds__(64) void finish_ar_kernel(const int32_t *__restrict__ y,
                                                       const int32_t *__restrict__ token_in, int B, int vocab,
                                                       KvView kv, int32_t *__restrict__ prefix_len,
                                                       int32_t *__restrict__ token_out) {
    int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const int L = prefix_len[b];
    bool err = !seq_fits(kv, L, 1) || (unsigned)token_in[b] >= (unsigned)vocab || y[b] < 0;
    if (!err) err = !page_ok(kv, kv.page_table[(size_t)b * kv.pages_per_seq + (L >> 4)]);
    token_out[b] = err ? -1 : y[b];
    if (!err) prefix_len[b] = L + 1;
}

// One wavefront per prefill pass over prompt positions [L, L + add_len) of sequence `seq`.  A pass that was fed a
// token id outside the vocabulary or met a page id outside the pool marks the sequence: prefix_len = -1, which
// keeps every later pass from storing anything for it, and first_drafts = -1.
__global__ __launch_bounds__(64) void finish_prefill_kernel(const int32_t *__restrict__ y,
                                                            const int32_t *__restrict__ tokens, int tok_stride, int k,
                                                            int seq0, Segs sg, int add_len, int last, int vocab,
                                                            KvView kv, int32_t *__restrict__ prefix_len,
                                                            int32_t *__restrict__ first_drafts) {
    const int lane = threadIdx.x, seq = seq0 + blockIdx.x;
    y += (size_t)blockIdx.x * (1 + k);
    tokens += (size_t)blockIdx.x * tok_stride;
    if (sg.n) add_len = sg.row0[blockIdx.x + 1] - sg.row0[blockIdx.x] - k;
    const int L = prefix_len[seq];
    bool bad = !seq_fits(kv, L, add_len);
    if (!bad) {
        for (int i = lane; i < add_len; i += 64) bad = bad || (unsigned)tokens[i] >= (unsigned)vocab;
        for (int p = (L >> 4) + lane; p <= ((L + add_len - 1) >> 4); p += 64)
            bad = bad || !page_ok(kv, kv.page_table[(size_t)seq * kv.pages_per_seq + p]);
    }
    // y rows: last prompt row, then mask slots 0..k-1; slot 0 of the block is superseded by the causal token
    int tok = 0;
    if (last && lane < k) {
        tok = (lane == 0) ? y[0] : y[1 + lane];
        bad = bad || tok < 0;
    }
    const bool err = __ballot(bad) != 0ull;
    if (lane == 0) prefix_len[seq] = err ? -1 : L + add_len;
    if ((last || err) && lane < k) first_drafts[(size_t)seq * k + lane] = err ? -1 : tok;
}

// plain row-major [M][K] -> A-fragment layout (8 elements per thread)
template <typename T>
__global__ void pack_act_kernel(const T *__restrict__ src, int M, int K, T *__restrict__ dst, ActLayout lay) {
    size_t n = (size_t)M * (K / 8);
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += (size_t)gridDim.x * blockDim.x) {
        int row = (int)(idx / (K / 8));
        int k = 8 * (int)(idx % (K / 8));
        const T *sp = src + (size_t)row * K + k;
        T *dp = dst + af_index(row, k, lay);
#pragma unroll
        for (int j = 0; j < 8; ++j) dp[j] = sp[j];
    }
}

// tiled partial sums [S][N/32][M][32] -> plain row-major [M][N]
__global__ void untile_sum_kernel(const float *__restrict__ part, int S, int M, int N, float *__restrict__ out) {
    size_t n = (size_t)M * N, stride = pt_split_stride(M, N);
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += (size_t)gridDim.x * blockDim.x) {
        int row = (int)(idx / N), col = (int)(idx % N);
        float v = 0.f;
        for (int sp = 0; sp < S; ++sp) v += part[(size_t)sp * stride + pt_index(col, row, M)];
        out[idx] = v;
    }
}

// Fold of the LM head's per-group maxima ([G][M] values, then [G][M] columns).  A block takes RB rows (a power
// of two, at most 16) and splits the groups over 1024 / RB slices; the slices are folded by a tree in LDS.  The
// order (larger value, then lower column) is total, so the result does not depend on how the fold is grouped.
__global__ __launch_bounds__(1024) void argmax_groups_kernel(const float *__restrict__ part, int M, int G, int RB,
                                                             int32_t *__restrict__ y) {
    const int r = threadIdx.x & (RB - 1), sl = threadIdx.x / RB, SL = 1024 / RB;
    const int row = blockIdx.x * RB + r;
    const float *pmax = part;
    const int *pidx = (const int *)(part + (size_t)G * M);
    float best = -INFINITY;
    int bi = 0x7fffffff;
    auto take = [&](float v, int i) {
        if (v > best || (v == best && i < bi)) {
            best = v;
            bi = i;
        }
    };
    if (row < M) {
        int g = sl;
        for (; g + 3 * SL < G; g += 4 * SL) {      // four independent loads at a time
            const float v0 = pmax[(size_t)g * M + row], v1 = pmax[(size_t)(g + SL) * M + row];
            const float v2 = pmax[(size_t)(g + 2 * SL) * M + row], v3 = pmax[(size_t)(g + 3 * SL) * M + row];
            const int i0 = pidx[(size_t)g * M + row], i1 = pidx[(size_t)(g + SL) * M + row];
            const int i2 = pidx[(size_t)(g + 2 * SL) * M + row], i3 = pidx[(size_t)(g + 3 * SL) * M + row];
            take(v0, i0);
            take(v1, i1);
            take(v2, i2);
            take(v3, i3);
        }
        for (; g < G; g += SL) take(pmax[(size_t)g * M + row], pidx[(size_t)g * M + row]);
    }
    __shared__ float sv[1024];
    __shared__ int si[1024];
    sv[threadIdx.x] = best;
    si[threadIdx.x] = bi;
    __syncthreads();
    for (int half = SL >> 1; half >= 1; half >>= 1) {
        if (sl < half) {
            take(sv[threadIdx.x + half * RB], si[threadIdx.x + half * RB]);
            sv[threadIdx.x] = best;
            si[threadIdx.x] = bi;
        }
        __syncthreads();
    }
    if (sl == 0 && row < M) y[row] = bi == 0x7fffffff ? -1 : bi;      // same rule as argmax_rows_kernel
}

__global__ void set_i32_kernel(int32_t *p, int n, int32_t v) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// ------------------------------------------------------------------ fp32 GEMM (v_mfma_f32_16x16x4_f32)
// a: A-fragment layout (fp32 elements), w: row-major [N][K], out: tiled or row-major.
// The fp32 configuration is a small model whose GEMMs are all latency, so a workgroup's four waves split K (32 at a
// time, in turn), every wave takes both operands straight into registers, eight k of one row or column per lane (a
// 16x16x4 MFMA sums one of them over the four lane groups), and the four sums meet in LDS in wave order: one trip to
// memory per 128 k instead of four with two barriers each (20 x 128 x 512 44 -> 4.2 us, 272 x 4096 x 4096 617 -> 191).  RT x CT tiles of 16 per
// workgroup: one by one while that leaves compute units idle, then 2 x 4.
// (A caller's fp32 buffers may start on any float; a 16-byte load takes any multiple of four bytes, the type says so.)
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
template <int RT, int CT>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float *__restrict__ a, const float *__restrict__ w,
                                                       float *__restrict__ out, int M, int N, int K,
                                                       int out_row_major) {
    __shared__ float part[4][RT * CT * 4][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int row0 = blockIdx.y * 16 * RT, col0 = blockIdx.x * 16 * CT;
    const ActLayout lay = act_layout(M);
    f32x4 acc[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    for (int kb = 32 * wave; kb < K; kb += 128) {
        const int k = kb + 8 * g;                  // K is a multiple of 8: a lane's eight k exist or do not
        f32x4 av[RT][2], wv[CT][2];
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            const int row = row0 + 16 * i + n;
            const bool ok = row < M && k < K;
            const float *p = a + (ok ? af_index(row, k, lay) : 0);
            av[i][0] = ok ? *(const f32x4_any *)p : zero;
            av[i][1] = ok ? *(const f32x4_any *)(p + 4) : zero;
        }
#pragma unroll
        for (int j = 0; j < CT; ++j) {
            const int col = col0 + 16 * j + n;
            const bool ok = col < N && k < K;
            const float *p = w + (ok ? (size_t)col * K + k : 0);
            wv[j][0] = ok ? *(const f32x4_any *)p : zero;
            wv[j][1] = ok ? *(const f32x4_any *)(p + 4) : zero;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int j = 0; j < CT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i][e >> 2][e & 3], wv[j][e >> 2][e & 3], acc[i][j], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) part[wave][(i * CT + j) * 4 + e][lane] = acc[i][j][e];
    __syncthreads();
    for (int x = wave; x < RT * CT * 4; x += 4) {      // register x % 4 of tile x / 4: row 4 * (lane / 16) + x % 4
        const float v = ((part[0][x][lane] + part[1][x][lane]) + part[2][x][lane]) + part[3][x][lane];
        const int t = x >> 2, m = row0 + 16 * (t / CT) + 4 * g + (x & 3), c = col0 + 16 * (t % CT) + n;
        if (m < M && c < N) out[out_row_major ? (size_t)m * N + c : pt_index(c, m, M)] = v;
    }
}

// The same GEMM with its producer and its consumer folded in, for the few-row forwards of small fp32 models, which are a chain of
// launches that cost more than their work (two layers of d = 128, 20 rows: 24 launches 89 us, with these 14 and 58):
//   * A = rmsnorm(x + the pending partial sums of the previous GEMM) * gain.  Every workgroup sums its 16 rows over all of
//     K for their mean squares (in registers: KI pieces of 128 k) and the first column block of each row tile writes the
//     updated residual stream to x_out, which must not be x;
//   * FUSE_ROPE: CT tiles are one head; Q rotated to q_out, K rotated and V into the cache pages or the scratch tiles, as
//     rope_kv_kernel stores them (a rotation pair is CT / 2 tiles apart, in the same lane and register);
//   * FUSE_SWIGLU: gate and up tile of the same 16 features, h into the A-fragment layout of the down projection;
//   * FUSE_LOGITS: row-major output of the rows a sequence sends through the head.
template <int KI, int CT, int EPI, class SG>
__global__ __launch_bounds__(256) void gemm_f32_fused_kernel(const float *__restrict__ x, const float *__restrict__ pend,
                                                             const float *__restrict__ gain, float eps,
                                                             float *__restrict__ x_out, const float *__restrict__ w,
                                                             float *__restrict__ out, int M, int N, int K, int n_rows,
                                                             int R, int M_all, RowDesc d_any, SG sg, RopeOut ro) {
    __shared__ float part[4][CT * 4][64];
    __shared__ float sums[4][16];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int row0 = blockIdx.y * 16, col0 = blockIdx.x * 16 * CT;
    // this lane's row of A: output row row0 + n, row src of the forward
    const int o_row = min(row0 + n, M - 1);
    int src = o_row;
    if (EPI == FUSE_LOGITS) {
        const int b = o_row / n_rows;
        src = (b + 1) * R;
        if constexpr (kSegs<SG>) src = sg.row0[b + 1];
        src += o_row - (b + 1) * n_rows;
    }
    f32x4 av[KI][2], wv[CT][2];
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    auto load_w = [&](int k) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < CT; ++j) {
            const int col = col0 + 16 * j + n;
            const bool ok = col < N && k < K;
            const float *p = w + (ok ? (size_t)col * K + k : 0);
            wv[j][0] = ok ? *(const f32x4_any *)p : zero;
            wv[j][1] = ok ? *(const f32x4_any *)(p + 4) : zero;
        }
    };
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < KI; ++i) {
        const int k = 128 * i + 32 * wave + 8 * g;
        av[i][0] = av[i][1] = zero;
        if (k < K) {
            const float *p = x + (size_t)src * K + k;
            av[i][0] = *(const f32x4_any *)p;
            av[i][1] = *(const f32x4_any *)(p + 4);
            if (pend) {
                const float *q = pend + pt_index(k, src, M_all);
                av[i][0] += *(const f32x4_any *)q;
                av[i][1] += *(const f32x4_any *)(q + 4);
            }
        }
    }
    load_w(32 * wave + 8 * g);
#pragma unroll
    for (int i = 0; i < KI; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) ss += av[i][e >> 2][e & 3] * av[i][e >> 2][e & 3];
    ss += __shfl_xor(ss, 16);
    ss += __shfl_xor(ss, 32);
    if (g == 0) sums[wave][n] = ss;
    __syncthreads();
    const float rs = rsqrtf((((sums[0][n] + sums[1][n]) + sums[2][n]) + sums[3][n]) / (float)K + eps);
    f32x4 acc[CT];
#pragma unroll
    for (int j = 0; j < CT; ++j) acc[j] = zero;
#pragma unroll
    for (int i = 0; i < KI; ++i) {
        const int k = 128 * i + 32 * wave + 8 * g;
        if (128 * i + 32 * wave >= K) break;           // wave-uniform
        if (i) load_w(k);
        if (EPI != FUSE_LOGITS && blockIdx.x == 0 && row0 + n < M && k < K) {
            *(f32x4_any *)(x_out + (size_t)src * K + k) = av[i][0];
            *(f32x4_any *)(x_out + (size_t)src * K + k + 4) = av[i][1];
        }
        const float *gp = gain + (k < K ? k : 0);
        const f32x4 g0 = *(const f32x4_any *)gp, g1 = *(const f32x4_any *)(gp + 4);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float a = av[i][e >> 2][e & 3] * rs * (e < 4 ? g0[e & 3] : g1[e & 3]);
#pragma unroll
            for (int j = 0; j < CT; ++j)
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, wv[j][e >> 2][e & 3], acc[j], 0, 0, 0);
        }
    }
#pragma unroll
    for (int j = 0; j < CT; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) part[wave][j * 4 + e][lane] = acc[j][e];
    __syncthreads();
    auto sum4 = [&](int i) { return ((part[0][i][lane] + part[1][i][lane]) + part[2][i][lane]) + part[3][i][lane]; };
    // register e of tile t: row 4 * (lane / 16) + e, column 16 t + lane % 16
    if constexpr (EPI == FUSE_LOGITS) {
        for (int i = wave; i < CT * 4; i += 4) {
            const int m = row0 + 4 * g + (i & 3), c = col0 + 16 * (i >> 2) + n;
            const float v = sum4(i);
            if (m < M && c < N) out[(size_t)m * N + c] = v;
        }
    } else if constexpr (EPI == FUSE_SWIGLU) {
        const ActLayout lay = act_layout(M);
        const int m = row0 + 4 * g + wave, f = (col0 >> 1) + n;
        const float gt = sum4(wave), up = sum4(4 + wave);
        if (m < M) out[af_index(m, f, lay)] = gt / (1.f + __expf(-gt)) * up;
    } else {
        const KvView &kv = ro.kv;
        const int hd = 16 * CT, half = hd / 2, head = blockIdx.x, n_q = ro.n_q;
        const int n_mtiles = (d_any.nm + 15) / 16;
#pragma unroll
        for (int t = 0; t < CT / 2; ++t) {
            const int m = row0 + 4 * g + wave, i = 16 * t + n;        // rotation pair (i, i + half) of row m
            const float lo = sum4(4 * t + wave), hi = sum4(4 * (t + CT / 2) + wave);
            if (m >= M) continue;
            const float c = ro.rope_cs[((size_t)m * half + i) * 2], s = ro.rope_cs[((size_t)m * half + i) * 2 + 1];
            const float r0 = lo * c - hi * s, r1 = hi * c + lo * s;
            if (head < n_q) {
                float *q = out + ((size_t)m * n_q + head) * hd + i;
                q[0] = r0;
                q[half] = r1;
                continue;
            }
            const int b = seq_of_row(d_any, sg, m);
            int row_base;
            const RowDesc d = seq_desc(d_any, sg, b, &row_base);
            const int r = m - row_base, h = head < n_q + kv.n_kv ? head - n_q : head - n_q - kv.n_kv;
            const bool is_k = head < n_q + kv.n_kv;
            float *dst;                          // of pair element i; the other one `half` rows or values on
            if (r < d.nc) {
                const int L_raw = ro.prefix_len[d.seq_base + b], L = clamp_prefix(kv, L_raw, d.nc), p = L + r;
                if (!seq_fits(kv, L_raw, d.nc)) continue;
                const int page = kv.page_table[(size_t)(d.seq_base + b) * kv.pages_per_seq + (p >> 4)];
                if (!page_ok(kv, page)) continue;
                dst = is_k ? (float *)kv.k_pages + k_page_offset(kv, page, h, p & 15, i)
                           : (float *)kv.v_pages + v_page_offset(kv, page, h, p & 15, i);
            } else {
                const int mm = r - d.nc;
                const size_t tile = ((size_t)b * kv.n_kv + h) * n_mtiles + (mm >> 4);
                dst = is_k ? ro.k_scr + (tile * 16 + (mm & 15)) * hd + i : ro.v_scr + (tile * hd + i) * 16 + (mm & 15);
            }
            dst[0] = is_k ? r0 : lo;
            dst[is_k ? half : half * 16] = is_k ? r1 : hi;
        }
    }
}

// ------------------------------------------------------------------ fp32 hybrid-mask attention (plain ALU)
// One workgroup per (sequence, query head, row).  Keys come in units of 16: cache pages 0 .. ceil((L + nc) / 16) - 1,
// then the mask rows' scratch tiles.  A wave takes four units at a time, one key per lane for the scores, one head
// dimension (of two halves of the units where hd <= 32) per lane for the values; the four waves take every fourth
// group of units and are folded at the end.  What bounds it is latency: page id, K row, V piece, three dependent
// trips per 64 keys (they used to be two per key: 22 -> 5.4 us at 20 rows, 64 cached tokens).
// VEC: rows of K are whole, aligned 16-byte pieces and the pages start on 16 bytes.
template <bool VEC, class SG>
__global__ __launch_bounds__(256) void attention_f32_kernel(const float *__restrict__ q, KvView kv,
                                                            const float *__restrict__ k_scr,
                                                            const float *__restrict__ v_scr,
                                                            const int32_t *__restrict__ prefix_len, RowDesc d_any,
                                                            SG sg, int n_q, float *__restrict__ out, int out_af,
                                                            ActLayout lay) {
    const int row = blockIdx.x, head = blockIdx.y;
    const int b = seq_of_row(d_any, sg, row);
    int row_base;
    const RowDesc d = seq_desc(d_any, sg, b, &row_base);
    const int r = row - row_base;
    const int hd = kv.hd, n_kv = kv.n_kv, g = head / (n_q / n_kv);
    const int L = clamp_prefix(kv, prefix_len[d.seq_base + b], d.nc);
    const RowInfo ri = row_info(d, r, L);
    const int n_cache = L + d.nc, n_mtiles = (d.nm + 15) / 16;
    const int cache_units = (n_cache + 15) / 16, units = cache_units + n_mtiles;
    const float *kp = (const float *)kv.k_pages, *vp = (const float *)kv.v_pages;
    const int32_t *pt = kv.page_table + (size_t)(d.seq_base + b) * kv.pages_per_seq;
    __shared__ __attribute__((aligned(16))) float qs[128];
    __shared__ __attribute__((aligned(16))) float ps[4][64];
    __shared__ float fold[4][2 + 128];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int i = threadIdx.x; i < hd; i += 256) qs[i] = q[((size_t)row * n_q + head) * hd + i];
    __syncthreads();
    const float scale = rsqrtf((float)hd);
    const bool split = hd <= 32;                    // 32 dimensions: the half-waves take two units each
    const int d0 = split ? lane & 31 : lane;
    float m_run = -INFINITY, l_run = 0.f;
    float o0 = 0.f, o1 = 0.f;                       // this lane's output dimensions: d0, d0 + 64
    for (int u0 = 4 * wave; u0 < units; u0 += 16) {
        const int u = u0 + (lane >> 4), slot = lane & 15;
        bool vis = false;
        const float *kt = nullptr, *vt = nullptr;   // this lane's unit (16 keys) of K and V
        if (u < cache_units) {
            const int t = 16 * u + slot;
            vis = t < L || (t < n_cache && t - L < ri.vis);
            const int page = pt[u], pg = page_ok(kv, page) ? page : 0;
            kt = kp + k_page_offset(kv, pg, g, 0, 0);
            vt = vp + v_page_offset(kv, pg, g, 0, 0);
        } else if (u < units) {
            const int m = 16 * (u - cache_units) + slot;
            vis = ri.blk >= 0 && m < d.nm && m / d.bl == ri.blk;
            const size_t tile = ((size_t)b * n_kv + g) * n_mtiles + (u - cache_units);
            kt = k_scr + tile * 16 * hd;
            vt = v_scr + tile * hd * 16;
        }
        float s = -INFINITY;
        if (vis) {
            const float *krow = kt + slot * hd;
            float acc = 0.f;
            if (VEC) {
#pragma unroll 8
                for (int i = 0; i < hd; i += 4) {
                    const float4 k4 = *(const float4 *)(krow + i), q4 = *(const float4 *)(qs + i);
                    acc = fmaf(q4.x, k4.x, acc);
                    acc = fmaf(q4.y, k4.y, acc);
                    acc = fmaf(q4.z, k4.z, acc);
                    acc = fmaf(q4.w, k4.w, acc);
                }
            } else {
                for (int i = 0; i < hd; ++i) acc = fmaf(qs[i], krow[i], acc);
            }
            s = acc * scale;
        }
        const float mx = wave_max(s);
        if (mx == -INFINITY) continue;     // nothing visible in these units (uniform across the wave)
        const float m_new = fmaxf(m_run, mx);
        const float alpha = __expf(m_run - m_new);
        const float p = vis ? __expf(s - m_new) : 0.f;
        l_run = l_run * alpha + wave_sum(p);
        o0 *= alpha;
        o1 *= alpha;
        m_run = m_new;
        __builtin_amdgcn_wave_barrier();
        ps[wave][lane] = p;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const unsigned long long any = __ballot(p != 0.f);
        // a key that carries no weight is never multiplied: its slot may hold anything
        auto take = [&](int uu, int dd, float &o) {
            const float *src = (const float *)__shfl((unsigned long long)vt, 16 * uu) + (size_t)dd * 16;
            if (!((any >> (16 * uu)) & 0xffffull) || dd >= hd) return;
            float v[16];
            if (VEC) {
#pragma unroll
                for (int x = 0; x < 4; ++x) *(float4 *)(v + 4 * x) = *(const float4 *)(src + 4 * x);
            } else {
#pragma unroll
                for (int x = 0; x < 16; ++x) v[x] = src[x];
            }
#pragma unroll
            for (int x = 0; x < 16; ++x) {
                const float pj = ps[wave][16 * uu + x];
                o = pj != 0.f ? fmaf(pj, v[x], o) : o;
            }
        };
        if (split) {
#pragma unroll
            for (int x = 0; x < 2; ++x) take(2 * x + (lane >> 5), d0, o0);
        } else {
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                take(x, d0, o0);
                if (hd > 64) take(x, d0 + 64, o1);
            }
        }
    }
    if (split) o0 += __shfl_xor(o0, 32);
    if (lane == 0) {
        fold[wave][0] = m_run;
        fold[wave][1] = l_run;
    }
    if (d0 < hd && (!split || lane < 32)) fold[wave][2 + d0] = o0;
    if (hd > 64 && d0 + 64 < hd) fold[wave][2 + d0 + 64] = o1;
    __syncthreads();
    const int dd = threadIdx.x;
    if (dd < hd) {
        const float m = fmaxf(fmaxf(fold[0][0], fold[1][0]), fmaxf(fold[2][0], fold[3][0]));
        float num = 0.f, den = 0.f;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            if (fold[x][0] == -INFINITY) continue;       // no key of this wave is visible
            const float wgt = __expf(fold[x][0] - m);
            num = fmaf(wgt, fold[x][2 + dd], num);
            den = fmaf(wgt, fold[x][1], den);
        }
        out[out_af ? af_index(row, head * hd + dd, lay) : ((size_t)row * n_q + head) * hd + dd] = num / den;
    }
}

inline int grid_for(size_t n, int block, int cap = 4096) {
    size_t g = (n + block - 1) / block;
    return (int)(g < 1 ? 1 : (g > (size_t)cap ? cap : g));
}

}  // namespace

void launch_pack_weight(int dtype, const void *src, int rows, int cols, void *dst, int dst_rows, int tile_off,
                        int tile_stride, hipStream_t st) {
    if (dtype == TIDAR_BF16) {
        size_t n = (size_t)rows * (cols / 8);
        pack_bf16_kernel<<<grid_for(n, 256, 65536), 256, 0, st>>>((const bf16_t *)src, rows, cols, (bf16_t *)dst,
                                                                   (dst_rows + 31) / 32, tile_off, tile_stride);
    } else {
        size_t n = (size_t)rows * cols;
        pack_f32_kernel<<<grid_for(n, 256, 65536), 256, 0, st>>>((const float *)src, rows, cols, (float *)dst,
                                                                  tile_off, tile_stride);
    }
}

void launch_embed_rows(int dtype, const void *embed, const int32_t *tokens, int tok_stride, const int32_t *prefix_len,
                       const RowDesc &d, const Segs &sg, int M, int d_model, int mask_id, int vocab, KvView kv,
                       float rope_base, float *x, int32_t *pos_out, int n_head, float *rope_cs, hipStream_t st) {
    auto go = [&](auto table, auto segs) {
        embed_rows_kernel<<<M, 256, 0, st>>>(table, tokens, tok_stride, prefix_len, d, segs, d_model, mask_id, vocab, kv,
                                             kv.hd, rope_base, x, pos_out, n_head, rope_cs);
    };
    auto typed = [&](auto table) {
        if (sg.n) go(table, sg);
        else go(table, NoSegs());
    };
    if (dtype == TIDAR_BF16) typed((const bf16_t *)embed);
    else typed((const float *)embed);
}

void launch_rmsnorm(int dtype, float *x, const float *part, int S, const void *gain, float eps, int B, int n_rows, int M,
                    const Segs &sg, int d_model, void *out, hipStream_t st) {
    int rows = B * n_rows, R = M / B;
    ActLayout mt_out = act_layout(rows);
    size_t stride = pt_split_stride(M, d_model);
    // from where it gains on (figures at the kernel), which is also where the GEMMs change class.  (Gains are loaded 16 bytes
    // at a time there: a caller's gain on another boundary stays with the kernel below.)
    if (dtype == TIDAR_BF16 && rows > 480 && d_model <= 4096 && ((uintptr_t)gain & 15) == 0) {
        auto go = [&](auto jp, auto segs) {
            rmsnorm_rows_kernel<decltype(jp)::value><<<(rows + 63) / 64 * 16, 256, 0, st>>>(
                x, part, S, stride, (const bf16_t *)gain, eps, n_rows, R, segs, d_model, M, rows, (bf16_t *)out, mt_out);
        };
        auto typed = [&](auto jp) {
            if (sg.n) go(jp, sg);
            else go(jp, NoSegs());
        };
        if (d_model <= 1536) typed(std::integral_constant<int, 3>());
        else if (d_model <= 2048) typed(std::integral_constant<int, 4>());
        else typed(std::integral_constant<int, 8>());
        return;
    }
    int threads = ((d_model / 4 + 63) / 64) * 64;
    threads = threads > 1024 ? 1024 : threads < 64 ? 64 : threads;
    auto go = [&](auto g, auto o, auto segs) {
        using T = std::remove_pointer_t<decltype(o)>;
        if (mt_out.wide)
            rmsnorm_kernel<T, true><<<line_rows(rows), threads, 0, st>>>(x, part, S, stride, g, eps, n_rows, R, segs, d_model, M,
                                                                         rows, o, mt_out);
        else
            rmsnorm_kernel<T, false><<<rows, threads, 0, st>>>(x, part, S, stride, g, eps, n_rows, R, segs, d_model, M, rows, o,
                                                               mt_out);
    };
    auto typed = [&](auto g, auto o) {
        if (sg.n) go(g, o, sg);
        else go(g, o, NoSegs());
    };
    if (dtype == TIDAR_BF16) typed((const bf16_t *)gain, (bf16_t *)out);
    else typed((const float *)gain, (float *)out);
}

void launch_gemm_f32(const float *a, const float *w, float *out, int M, int N, int K, int out_row_major,
                     hipStream_t st) {
    // 16 x 16 tiles until there are a few workgroups for every compute unit
    if ((size_t)((N + 15) / 16) * ((M + 15) / 16) <= 1024)
        gemm_f32_kernel<1, 1><<<dim3((N + 15) / 16, (M + 15) / 16), 256, 0, st>>>(a, w, out, M, N, K, out_row_major);
    else
        gemm_f32_kernel<2, 4><<<dim3((N + 63) / 64, (M + 31) / 32), 256, 0, st>>>(a, w, out, M, N, K, out_row_major);
}

// Every workgroup makes its own norm, so the line lies where that costs what the launch saved.  Four layers, k(k+1) rows, before ->
// with: d 128 / 20 and 240 rows 126 -> 91, 155 -> 113 us; d 256 / 20, 72 and 240 rows 148 -> 132, 162 -> 143, 214 -> 188;
// d 512 / 20 and 240 rows 189 -> 189, 356 -> 419; d 1024 / 20 rows 335 -> 442.
bool gemm_f32_fuse_ok(int M, int K, int hd) {
    return M <= kFuseF32Rows && K <= kFuseF32K && (hd == 32 || hd == 64 || hd == 128);
}

void launch_gemm_f32_fused(int epi, const float *x, const float *pend, const float *gain, float eps, float *x_out,
                           const float *w, float *out, int M, int N, int K, int n_rows, int R, int M_all, const RowDesc &d,
                           const Segs &sg, const RopeOut &ro, hipStream_t st) {
    auto go = [&](auto ki, auto ct, auto e, auto segs) {
        constexpr int KI = decltype(ki)::value, CT = decltype(ct)::value, E = decltype(e)::value;
        gemm_f32_fused_kernel<KI, CT, E><<<dim3((N + 16 * CT - 1) / (16 * CT), (M + 15) / 16), 256, 0, st>>>(
            x, pend, gain, eps, x_out, w, out, M, N, K, n_rows, R, M_all, d, segs, ro);
    };
    auto by_segs = [&](auto ki, auto ct, auto e) {
        if (sg.n) go(ki, ct, e, sg);
        else go(ki, ct, e, NoSegs());
    };
    auto by_k = [&](auto ct, auto e) {
        if (K <= 128) by_segs(std::integral_constant<int, 1>(), ct, e);
        else by_segs(std::integral_constant<int, kFuseF32K / 128>(), ct, e);
    };
    if (epi == FUSE_SWIGLU) by_k(std::integral_constant<int, 2>(), std::integral_constant<int, FUSE_SWIGLU>());
    else if (epi == FUSE_LOGITS) by_k(std::integral_constant<int, 1>(), std::integral_constant<int, FUSE_LOGITS>());
    else if (ro.kv.hd == 32) by_k(std::integral_constant<int, 2>(), std::integral_constant<int, FUSE_ROPE>());
    else if (ro.kv.hd == 64) by_k(std::integral_constant<int, 4>(), std::integral_constant<int, FUSE_ROPE>());
    else by_k(std::integral_constant<int, 8>(), std::integral_constant<int, FUSE_ROPE>());
}

void launch_pack_act(int dtype, const void *src, int M, int K, void *dst, hipStream_t st) {
    size_t n = (size_t)M * (K / 8);
    ActLayout mt = act_layout(M);
    if (dtype == TIDAR_BF16)
        pack_act_kernel<bf16_t><<<grid_for(n, 256, 8192), 256, 0, st>>>((const bf16_t *)src, M, K, (bf16_t *)dst, mt);
    else
        pack_act_kernel<float><<<grid_for(n, 256, 8192), 256, 0, st>>>((const float *)src, M, K, (float *)dst, mt);
}

void launch_untile_sum(const float *part, int S, int M, int N, float *out, hipStream_t st) {
    untile_sum_kernel<<<grid_for((size_t)M * N, 256, 8192), 256, 0, st>>>(part, S, M, N, out);
}

void launch_rope_kv(int dtype, const float *qkv_part, int S, const float *rope_cs, const int32_t *prefix_len,
                    const RowDesc &d, const Segs &sg, int B, int rows, int n_q, KvView kv, void *q_out, void *k_scr,
                    void *v_scr, hipStream_t st) {
    size_t stride = pt_split_stride(rows, (n_q + 2 * kv.n_kv) * kv.hd);
    const int per_head = kv.hd / 8;                  // items (four rotation pairs) per head
    const int gy = (n_q * per_head + 255) / 256 + (kv.n_kv * per_head + 255) / 256;
    const int v_parts = (kv.n_kv * kv.hd * 4 + gy * 256 - 1) / (gy * 256);      // see the kernel's V-tile branch
    const int v_tiles = B * ((d.nc + 15) / 16 + 1 + (d.nm + 15) / 16);
    dim3 grid(rows + v_tiles * v_parts, gy);
    auto go = [&](auto q, auto segs) {
        typedef decltype(q) out_t;
        rope_kv_kernel<<<grid, 256, 0, st>>>(qkv_part, S, stride, rope_cs, prefix_len, d, segs, n_q, rows, kv, q, (out_t)k_scr,
                                             (out_t)v_scr);
    };
    auto typed = [&](auto q) {
        if (sg.n) go(q, sg);
        else go(q, NoSegs());
    };
    if (dtype == TIDAR_BF16) typed((bf16_t *)q_out);
    else typed((float *)q_out);
}

void launch_place_kv(int dtype, const void *k_new, const void *v_new, const int32_t *prefix_len, RowDesc d, int B,
                     KvView kv, void *k_scr, void *v_scr, hipStream_t st) {
    int rows = B * d.R;
    if (dtype == TIDAR_BF16)
        place_kv_kernel<bf16_t><<<rows, 256, 0, st>>>((const bf16_t *)k_new, (const bf16_t *)v_new, prefix_len, d, kv,
                                                       (bf16_t *)k_scr, (bf16_t *)v_scr);
    else
        place_kv_kernel<float><<<rows, 256, 0, st>>>((const float *)k_new, (const float *)v_new, prefix_len, d, kv,
                                                      (float *)k_scr, (float *)v_scr);
}

void launch_attention_f32(const float *q, KvView kv, const float *k_scr, const float *v_scr,
                          const int32_t *prefix_len, const RowDesc &d, const Segs &sg, int M, int n_q, float *out,
                          int out_af, hipStream_t st) {
    dim3 grid(M, n_q);
    const bool vec = kv.hd % 4 == 0 && (((uintptr_t)kv.k_pages | (uintptr_t)kv.v_pages | (uintptr_t)k_scr | (uintptr_t)v_scr) & 15) == 0;
    auto go = [&](auto kernel, auto segs) {
        kernel<<<grid, 256, 0, st>>>(q, kv, k_scr, v_scr, prefix_len, d, segs, n_q, out, out_af, act_layout(M));
    };
    if (vec && sg.n) go(attention_f32_kernel<true, Segs>, sg);
    else if (vec) go(attention_f32_kernel<true, NoSegs>, NoSegs());
    else if (sg.n) go(attention_f32_kernel<false, Segs>, sg);
    else go(attention_f32_kernel<false, NoSegs>, NoSegs());
}

void launch_swiglu(int dtype, const float *part, int S, int M, int d_ff, void *out, hipStream_t st) {
    size_t n = (size_t)M * (d_ff / 4);
    size_t stride = pt_split_stride(M, 2 * d_ff);
    ActLayout mt = act_layout(M);
    if (dtype == TIDAR_BF16)
        swiglu_kernel<bf16_t><<<grid_for(n, 256, 8192), 256, 0, st>>>(part, S, stride, M, d_ff, (bf16_t *)out, mt);
    else
        swiglu_kernel<float><<<grid_for(n, 256, 8192), 256, 0, st>>>(part, S, stride, M, d_ff, (float *)out, mt);
}

void launch_argmax_groups(const float *part, int M, int G, int32_t *y, hipStream_t st) {
    int RB = 16;
    while (RB > 1 && RB / 2 >= M) RB /= 2;       // smallest power of two that holds the rows, at most 16
    argmax_groups_kernel<<<(M + RB - 1) / RB, 1024, 0, st>>>(part, M, G, RB, y);
}

void launch_argmax_rows(const float *logits, int B, int Rh, int n_rows, int vocab, int n_choose,
                        const int32_t *pos_rows, int pos_stride, int pos_row0, int seq_base, int sample,
                        float temperature, uint64_t seed, float beta, int mix_base, int mix_stride, int32_t *y,
                        int y_stride, hipStream_t st) {
    if (((uintptr_t)logits & 15) == 0 && vocab % 4 == 0)
        argmax_rows_kernel<4><<<B * n_rows, 1024, 0, st>>>(logits, Rh, n_rows, vocab, n_choose, pos_rows, pos_stride, pos_row0,
                                                       seq_base, sample, temperature, seed, beta, mix_base, mix_stride,
                                                       y, y_stride);
    else
        argmax_rows_kernel<1><<<B * n_rows, 1024, 0, st>>>(logits, Rh, n_rows, vocab, n_choose, pos_rows, pos_stride, pos_row0,
                                                       seq_base, sample, temperature, seed, beta, mix_base, mix_stride,
                                                       y, y_stride);
}

void launch_score_rows(const float *logits, int rows, int vocab, const int32_t *text, int len, int c0, int nc,
                       float *ar_out, float *diff_out, hipStream_t st) {
    score_rows_kernel<<<rows, 1024, 0, st>>>(logits, vocab, text, len, c0, nc, ar_out, diff_out);
}

void launch_score_loss(const float *ar, const float *diff, int n, float alpha, float *loss, hipStream_t st) {
    score_loss_kernel<<<1, 256, 0, st>>>(ar, diff, n, alpha, loss);
}

void launch_verify_step(const int32_t *y, const int32_t *drafts, int k, int B, int vocab, KvView kv, int seq_base,
                        int32_t *prefix_len, int32_t *accepted_len, int32_t *accepted_tokens, int32_t *next_drafts,
                        hipStream_t st) {
    verify_step_kernel<<<B, 64, 0, st>>>(y, drafts, k, vocab, kv, seq_base, prefix_len, accepted_len, accepted_tokens,
                                         next_drafts);
}

void launch_finish_ar(const int32_t *y, const int32_t *token_in, int B, int vocab, KvView kv, int32_t *prefix_len,
                      int32_t *token_out, hipStream_t st) {
    finish_ar_kernel<<<(B + 63) / 64, 64, 0, st>>>(y, token_in, B, vocab, kv, prefix_len, token_out);
}

void launch_finish_prefill(const int32_t *y, const int32_t *tokens, int tok_stride, int k, int seq, int B, const Segs &sg,
                           int add_len, int last, int vocab, KvView kv, int32_t *prefix_len, int32_t *first_drafts,
                           hipStream_t st) {
    finish_prefill_kernel<<<B, 64, 0, st>>>(y, tokens, tok_stride, k, seq, sg, add_len, last, vocab, kv, prefix_len,
                                            first_drafts);
}

void launch_set_i32(int32_t *p, int n, int32_t v, hipStream_t st) {
    set_i32_kernel<<<(n + 255) / 256, 256, 0, st>>>(p, n, v);
}
