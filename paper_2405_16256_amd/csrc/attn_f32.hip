// fp32 causal attention of the fp32 path, forward and backward, on the fp32 matrix instructions
// (v_mfma_f32_16x16x4_f32: fp32 operands, products and sums).  The S x S scores are never written out.
//
// A workgroup of 4 waves owns 16 queries (forward, dq) or 16 keys (dk, dv) of one head and its waves take the 16-row
// tiles of the other side in turn; their partial results are added through LDS in wave order (no atomics).  Tiles of
// 16 and not of 32 because this path serves small launches: it is bound by the longest chain of tiles one wave walks
// (64 to 128 MFMAs of 32 cycles per pair of tiles at head_dim 128), so it needs many short chains.
//
// Operands go from global memory (L2 for all but the first reader) straight to registers, in two layouts:
//   rows: lane l holds row l%16 and the channels 16j + 4(l/16) + e: 16-byte loads; as both operands of a product over
//         the channels carry the same lane -> channel map, the order in which channels are summed does not matter.
//   cols: lane l holds the rows 4(l/16) + r and the channels 64q + 4(l%16) + e: the transposed first operand of a
//         product over the tile's rows, whose second operand is then exactly the accumulator of the scores
//         (lane l: column l%16, rows 4(l/16) + r).
// The next tile of each operand is requested as soon as its registers are free.
//
// Measured on one MI355X against one wave per row with scalar dot products (us per call, 8 query heads on 2 key/value
// heads of 128, 700 tokens): forward 401 -> 27, dq 424 -> 40, dk|dv 1246 -> 51; 4 heads of 64, 128 tokens: 39.7 -> 4.9,
// dq and dk|dv in one launch 59.6 -> 8.3.
#include "common.h"
#include "kernels.h"

namespace hh {

constexpr int AW = 4;     // waves per workgroup
constexpr int AT = 16;    // rows of a tile
constexpr uint32_t A_OUT = 0xFFFFFFF0u;   // byte offset past the end of every buffer: reads as zero

template <int D> struct RowsF { f32x4 v[D / 16]; };
template <int D> struct ColsF { f32x4 v[4][D / 64]; };

__device__ __forceinline__ f32x4 load4(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
    const i32x4 u = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
    return f32x4{__int_as_float(u[0]), __int_as_float(u[1]), __int_as_float(u[2]), __int_as_float(u[3])};
}

// One operand of one head: rows [0, S) of `ld` elements each, the head's channels at the base.  Rows at or past S read
// as zero (the rows behind them may belong to the next sample).
struct Operand {
    __amdgpu_buffer_rsrc_t rs;
    uint32_t base, ld4;   // bytes
    int S;
    __device__ __forceinline__ uint32_t at(int row, int channel) const {
        return row < S ? base + (uint32_t)row * ld4 + (uint32_t)channel * 4u : A_OUT;
    }
    template <int D> __device__ __forceinline__ void rows(RowsF<D>& f, int row0) const {
        const int l = threadIdx.x & 63;
        const uint32_t o = at(row0 + (l & 15), 4 * (l >> 4));
#pragma unroll
        for (int j = 0; j < D / 16; j++) f.v[j] = load4(rs, o + (o == A_OUT ? 0u : 64u * j));
    }
    template <int D> __device__ __forceinline__ void cols(ColsF<D>& f, int row0) const {
        const int l = threadIdx.x & 63;
#pragma unroll
        for (int r = 0; r < 4; r++)
#pragma unroll
            for (int q = 0; q < D / 64; q++) f.v[r][q] = load4(rs, at(row0 + 4 * (l >> 4) + r, 64 * q + 4 * (l & 15)));
    }
};
// `origin` is the array, `elems` its extent, `first` the element of row 0, channel 0
__device__ __forceinline__ Operand operand(const float* origin, size_t elems, size_t first, int ld, int S) {
    return Operand{make_rsrc(origin, (uint32_t)(elems * 4)), (uint32_t)(first * 4), (uint32_t)ld * 4u, S};
}

// a b^T over the channels: lane l gets column l%16 (row of b), rows 4(l/16) + r (rows of a)
template <int D>
__device__ __forceinline__ f32x4 dot_tiles(const RowsF<D>& a, const RowsF<D>& b) {
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;   // two chains: one alone would wait for its own results
#pragma unroll
    for (int j = 0; j < D / 16; j += 2)
#pragma unroll
        for (int e = 0; e < 4; e++) {
            s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[j][e], b.v[j][e], s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[j + 1][e], b.v[j + 1][e], s1, 0, 0, 0);
        }
    return s0 + s1;
}

// acc[4q+e] += c^T w over the tile's rows; w as dot_tiles gives it.  Accumulator register r of block 4q+e is channel
// 64q + 16(l/16) + 4r + e of column l%16.
template <int D>
__device__ __forceinline__ void add_cols(f32x4 (&acc)[D / 16], const ColsF<D>& c, f32x4 w) {
#pragma unroll
    for (int r = 0; r < 4; r++)
#pragma unroll
        for (int q = 0; q < D / 64; q++)
#pragma unroll
            for (int e = 0; e < 4; e++) acc[4 * q + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(c.v[r][q][e], w[r], acc[4 * q + e], 0, 0, 0);
}

// On the diagonal some weights are zero because the pair is masked, and a product of such a zero with an infinity or
// NaN must not reach the sum: a tile that holds one goes through the allowed pairs alone.
template <int D>
__device__ __forceinline__ bool all_finite(const ColsF<D>& c) {
    float t = 0.f;
#pragma unroll
    for (int r = 0; r < 4; r++)
#pragma unroll
        for (int q = 0; q < D / 64; q++)
#pragma unroll
            for (int e = 0; e < 4; e++) t = fmaf(c.v[r][q][e], 0.f, t);
    return !__any(t != 0.f);
}
// rows_are_keys: pair allowed where tile row <= column; else where tile row >= column (both count from the diagonal)
template <int D, bool ROWS_ARE_KEYS>
__device__ __forceinline__ void add_cols_masked(f32x4 (&acc)[D / 16], const Operand& op, int row0, f32x4 w) {
    const int l = threadIdx.x & 63, col = l & 15, g = l >> 4;
    for (int row = 0; row < AT; row++) {
        float wr = 0.f;
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const float t = __shfl(w[r], ((row >> 2) << 4) | col, WAVE);
            if (r == (row & 3)) wr = t;
        }
        if (row0 + row >= op.S || (ROWS_ARE_KEYS ? row > col : row < col)) continue;
#pragma unroll
        for (int q = 0; q < D / 64; q++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const f32x4 v = load4(op.rs, op.at(row0 + row, 64 * q + 16 * g + 4 * r));
#pragma unroll
                for (int e = 0; e < 4; e++) acc[4 * q + e][r] = fmaf(wr, v[e], acc[4 * q + e][r]);
            }
    }
}

// Partial sums of the 4 waves: [wave][column][channel], rows padded by one 16-byte chunk against bank conflicts.
template <int D> struct Merge {
    static constexpr int PITCH = D + 4;
    static constexpr int FLOATS = AW * AT * PITCH;
    __device__ static __forceinline__ void put(float* buf, int wave, const f32x4 (&acc)[D / 16]) {
        const int l = threadIdx.x & 63;
        float* p = buf + (wave * AT + (l & 15)) * PITCH + 16 * (l >> 4);
#pragma unroll
        for (int q = 0; q < D / 64; q++)
#pragma unroll
            for (int r = 0; r < 4; r++)
                *reinterpret_cast<f32x4*>(p + 64 * q + 4 * r) = f32x4{acc[4 * q][r], acc[4 * q + 1][r], acc[4 * q + 2][r], acc[4 * q + 3][r]};
    }
    __device__ static __forceinline__ f32x4 get(const float* buf, int wave, int column, int channel) {
        return *reinterpret_cast<const f32x4*>(buf + (wave * AT + column) * PITCH + channel);
    }
    __device__ static __forceinline__ f32x4 sum(const float* buf, int column, int channel) {
        f32x4 s = get(buf, 0, column, channel);
#pragma unroll
        for (int w = 1; w < AW; w++) s += get(buf, w, column, channel);
        return s;
    }
    // the workgroup writes the sums of its 16 columns, times `scale`, to rows tok0.. of `out`; with a rotary table the
    // pairs (i, i + D/2) are rotated by minus the angle of their position on the way
    __device__ static __forceinline__ void write(const float* buf, float* out, int ld, int pos0, int S, float scale,
                                                 const float* table, int table_seq) {
        constexpr int HALF = D / 2;
        const int column = threadIdx.x >> 4, c = (threadIdx.x & 15) * 4;
        if (pos0 + column >= S || c >= HALF) return;
        f32x4 a = sum(buf, column, c) * scale, b = sum(buf, column, c + HALF) * scale;
        if (table) {
            const f32x4 cs = *reinterpret_cast<const f32x4*>(table + (size_t)(pos0 + column) * HALF + c);
            const f32x4 sn = *reinterpret_cast<const f32x4*>(table + (size_t)(table_seq + pos0 + column) * HALF + c);
            const f32x4 ra = a * cs + b * sn, rb = b * cs - a * sn;
            a = ra; b = rb;
        }
        float* p = out + (size_t)column * ld + c;
        *reinterpret_cast<f32x4*>(p) = a;
        *reinterpret_cast<f32x4*>(p + HALF) = b;
    }
};

// The shape of a launch, with the divisors that take a workgroup's index apart.
struct F32Shape {
    int B, S, nh, nkv, tiles, parts;
    Divisor heads, nh_, group;        // heads of all samples, of one; query heads of a key/value head
    Divisor kv_jobs, kv, parts_, level;   // dk | dv jobs of a key tile, of one sample; workgroups a key/value head's query heads are dealt to;
                                          // jobs of both passes of a tile
    Divisor micro;                    // micro-batches
    int turn;                         // jobs of a tile in all of them, where that is a multiple of 8, otherwise 0
    int G;                            // query heads of one of those workgroups
};

// reductions over the four lanes that share a column
__device__ __forceinline__ float col_max(float v) { v = fmaxf(v, __shfl_xor(v, 16, WAVE)); return fmaxf(v, __shfl_xor(v, 32, WAVE)); }
__device__ __forceinline__ float col_sum(float v) { v += __shfl_xor(v, 16, WAVE); return v + __shfl_xor(v, 32, WAVE); }

template <int D>
__global__ __launch_bounds__(AW* WAVE, 2) void k_attn_f32_fwd(const float* __restrict__ qkv, int ld, float* __restrict__ o,
                                                              float* __restrict__ lse, F32Shape sh, MicroStride micro) {
    qkv = micro_at(qkv, micro.saved); o = micro_at(o, micro.saved); lse = micro_at(lse, micro.saved);
    const int B = sh.B, S = sh.S, nh = sh.nh, nkv = sh.nkv;
    __shared__ __attribute__((aligned(16))) float buf[Merge<D>::FLOATS];
    __shared__ float ms[AW][AT], ls[AW][AT];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, g = lane >> 4;
    int qt = (int)blockIdx.x, b = split_off(qt, sh.heads);
    qt = sh.tiles - 1 - qt;   // longest first
    const int h = split_off(b, sh.nh_);
    const int A = nh * D, kcol = A + quotient(h, sh.group) * D;
    const size_t extent = (size_t)B * S * ld, row0 = (size_t)b * S * ld;
    const Operand oq = operand(qkv, extent, row0 + h * D, ld, S), ok = operand(qkv, extent, row0 + kcol, ld, S),
                  ov = operand(qkv, extent, row0 + kcol + nkv * D, ld, S);
    RowsF<D> qf, kf;
    ColsF<D> vf;
    oq.rows(qf, qt * AT);
    f32x4 acc[D / 16];
#pragma unroll
    for (int i = 0; i < D / 16; i++) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;
    const float scale = 1.0f / sqrtf((float)D);
    if (wave <= qt) { ok.rows(kf, wave * AT); ov.cols(vf, wave * AT); }
    for (int t = wave; t <= qt; t += AW) {
        f32x4 z = dot_tiles<D>(kf, qf) * scale;   // row = key, column = query
        if (t + AW <= qt) ok.rows(kf, (t + AW) * AT);
        if (t == qt)
#pragma unroll
            for (int r = 0; r < 4; r++)
                if (4 * g + r > (lane & 15)) z[r] = -INFINITY;
        const float mn = fmaxf(m, col_max(fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]))));
        const float ref = mn == -INFINITY ? 0.f : mn;   // no finite score yet: all weights are zero, not NaN
        const float alpha = expf(m - ref);
        f32x4 p;
#pragma unroll
        for (int r = 0; r < 4; r++) p[r] = expf(z[r] - ref);
        l = l * alpha + col_sum((p[0] + p[1]) + (p[2] + p[3]));
#pragma unroll
        for (int i = 0; i < D / 16; i++) acc[i] *= alpha;
        if (t == qt && !all_finite<D>(vf)) add_cols_masked<D, true>(acc, ov, t * AT, p);
        else add_cols<D>(acc, vf, p);
        if (t + AW <= qt) ov.cols(vf, (t + AW) * AT);
        m = mn;
    }
    Merge<D>::put(buf, wave, acc);
    if (g == 0) { ms[wave][lane] = m; ls[wave][lane] = l; }
    __syncthreads();
    const int column = threadIdx.x >> 4, s = qt * AT + column;
    if (s >= S) return;
    float M = ms[0][column], f[AW], L = 0.f;
#pragma unroll
    for (int w = 1; w < AW; w++) M = fmaxf(M, ms[w][column]);
#pragma unroll
    for (int w = 0; w < AW; w++) {
        f[w] = ms[w][column] == -INFINITY ? 0.f : expf(ms[w][column] - M);
        L += f[w] * ls[w][column];
    }
    float* orow = o + ((size_t)b * S + s) * A + h * D;
    for (int c = (threadIdx.x & 15) * 4; c < D; c += 64) {
        f32x4 v = Merge<D>::get(buf, 0, column, c) * f[0];
#pragma unroll
        for (int w = 1; w < AW; w++) v += Merge<D>::get(buf, w, column, c) * f[w];
        *reinterpret_cast<f32x4*>(orow + c) = v / L;
    }
    if ((threadIdx.x & 15) == 0) lse[((size_t)b * nh + h) * S + s] = M + logf(L);
}

// Per 16 queries (tile qt of head and sample hb): delta = <do, o>, which is also left in dvec unless that is null, and
// dq = sum_t dZ[s,t] k[t] / sqrt(d).
template <int D>
__device__ __forceinline__ void bwd_q_body(float* buf, const int qt, const int hb, const float* __restrict__ qkv, int ld, const float* __restrict__ o,
                                           const float* __restrict__ dout, const float* __restrict__ lse, float* __restrict__ dvec,
                                           float* __restrict__ dqkv, const F32Shape& sh, const float* __restrict__ table, int table_seq) {
    const int B = sh.B, S = sh.S, nh = sh.nh, nkv = sh.nkv;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, g = lane >> 4;
    int b = hb;
    const int h = split_off(b, sh.nh_);
    const int A = nh * D, kcol = A + quotient(h, sh.group) * D;
    const size_t extent = (size_t)B * S * ld, row0 = (size_t)b * S * ld;
    const size_t extent_o = (size_t)B * S * A, row0_o = (size_t)b * S * A;
    const Operand oq = operand(qkv, extent, row0 + h * D, ld, S), ok = operand(qkv, extent, row0 + kcol, ld, S),
                  ov = operand(qkv, extent, row0 + kcol + nkv * D, ld, S);
    const Operand od = operand(dout, extent_o, row0_o + h * D, A, S), oo = operand(o, extent_o, row0_o + h * D, A, S);
    RowsF<D> qf, df, kf, vf;
    ColsF<D> kc;
    od.rows(df, qt * AT);
    oo.rows(kf, qt * AT);
    oq.rows(qf, qt * AT);
    float delta = 0.f;
#pragma unroll
    for (int j = 0; j < D / 16; j++)
#pragma unroll
        for (int e = 0; e < 4; e++) delta = fmaf(df.v[j][e], kf.v[j][e], delta);
    delta = col_sum(delta);
    const int s = qt * AT + (lane & 15);
    const size_t at_s = ((size_t)b * nh + h) * S + s;
    const float L = s < S ? lse[at_s] : 0.f;
    if (dvec && wave == 0 && g == 0 && s < S) dvec[at_s] = delta;
    const float scale = 1.0f / sqrtf((float)D);
    f32x4 acc[D / 16];
#pragma unroll
    for (int i = 0; i < D / 16; i++) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (wave <= qt) { ok.rows(kf, wave * AT); ov.rows(vf, wave * AT); ok.cols(kc, wave * AT); }
    for (int t = wave; t <= qt; t += AW) {
        const f32x4 z = dot_tiles<D>(kf, qf) * scale;   // row = key, column = query
        const bool more = t + AW <= qt;
        if (more) ok.rows(kf, (t + AW) * AT);
        const f32x4 dp = dot_tiles<D>(vf, df);
        if (more) ov.rows(vf, (t + AW) * AT);
        f32x4 dz;
#pragma unroll
        for (int r = 0; r < 4; r++) dz[r] = t == qt && 4 * g + r > (lane & 15) ? 0.f : expf(z[r] - L) * (dp[r] - delta);
        if (t == qt && !all_finite<D>(kc)) add_cols_masked<D, true>(acc, ok, t * AT, dz);
        else add_cols<D>(acc, kc, dz);
        if (more) ok.cols(kc, (t + AW) * AT);
    }
    Merge<D>::put(buf, wave, acc);
    __syncthreads();
    Merge<D>::write(buf, dqkv + ((size_t)b * S + qt * AT) * ld + h * D, ld, qt * AT, S, scale, table, table_seq);
}

// Per 16 keys (tile kt) of one key/value head: dv[t] = sum over its query heads and s >= t of P[s,t] do[s]; dk[t] = the same
// sum of dZ[s,t] q[s] / sqrt(d).  With parts > 1 the query heads are dealt out to `parts` workgroups, whose sums go to
// partial[part][token][dk | dv of every key/value head] and are finished by k_attn_f32_kv_reduce.  Unless DELTA_GIVEN (in
// dvec), delta of each query tile is formed here, as the dq jobs form it.
template <int D, bool DELTA_GIVEN>
__device__ __forceinline__ void bwd_kv_body(float* buf, const int kt, const int rest, const float* __restrict__ qkv, int ld, const float* __restrict__ o,
                                            const float* __restrict__ dout, const float* __restrict__ lse, const float* __restrict__ dvec,
                                            float* __restrict__ dqkv, float* __restrict__ partial, const F32Shape& sh,
                                            const float* __restrict__ table, int table_seq) {
    const int B = sh.B, S = sh.S, nh = sh.nh, nkv = sh.nkv, parts = sh.parts, tiles = sh.tiles;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, g = lane >> 4;
    int b = rest, hk = split_off(b, sh.kv);
    const int part = split_off(hk, sh.parts_);
    const int A = nh * D, kcol = A + hk * D, heads = sh.G, h0 = hk * sh.group.d + part * heads;
    const size_t extent = (size_t)B * S * ld, row0 = (size_t)b * S * ld;
    const size_t extent_o = (size_t)B * S * A, row0_o = (size_t)b * S * A;
    Operand oq = operand(qkv, extent, row0 + (size_t)h0 * D, ld, S), od = operand(dout, extent_o, row0_o + (size_t)h0 * D, A, S);
    Operand oo = od;
    if (!DELTA_GIVEN) oo.rs = make_rsrc(o, (uint32_t)(extent_o * 4));
    const uint32_t base_q = oq.base, base_d = od.base;
    RowsF<D> kf, vf, qf, df, of;
    ColsF<D> qc, dc;
    operand(qkv, extent, row0 + kcol, ld, S).rows(kf, kt * AT);
    operand(qkv, extent, row0 + kcol + nkv * D, ld, S).rows(vf, kt * AT);
    f32x4 dk[D / 16], dv[D / 16];
#pragma unroll
    for (int i = 0; i < D / 16; i++) dk[i] = dv[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float scale = 1.0f / sqrtf((float)D);
    const int per_head = tiles - kt, n = heads * per_head;   // (head, query tile) pairs, dealt out to the waves in turn
    int head = 0, tile = wave;   // query head and tile (from kt on) of the pair that is asked for
    auto point = [&]() {         // the operands at that head; its query tile
        while (tile >= per_head) { tile -= per_head; head++; }
        oq.base = base_q + (uint32_t)(head * D) * 4u;
        oo.base = od.base = base_d + (uint32_t)(head * D) * 4u;
        return kt + tile;
    };
    if (wave < n) {
        const int t = point();
        oq.rows(qf, t * AT); od.rows(df, t * AT);
        if (!DELTA_GIVEN) oo.rows(of, t * AT);
        od.cols(dc, t * AT); oq.cols(qc, t * AT);
    }
    for (int i = wave; i < n; i += AW) {
        const int qt = kt + tile, hd = h0 + head;
        const Operand cq = oq, cd = od;
        const size_t stat = ((size_t)b * nh + hd) * S;
        float L[4], dl[4];
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int s = min(qt * AT + 4 * g + r, S - 1);
            L[r] = lse[stat + s];
            if (DELTA_GIVEN) dl[r] = dvec[stat + s];
        }
        const bool more = i + AW < n;
        tile += AW;
        const int nt = more ? point() : 0;
        if (!DELTA_GIVEN) {
            float delta = 0.f;
#pragma unroll
            for (int j = 0; j < D / 16; j++)
#pragma unroll
                for (int e = 0; e < 4; e++) delta = fmaf(df.v[j][e], of.v[j][e], delta);
            delta = col_sum(delta);   // of query lane % 16
#pragma unroll
            for (int r = 0; r < 4; r++) dl[r] = __shfl(delta, 4 * g + r, WAVE);
            if (more) oo.rows(of, nt * AT);
        }
        const f32x4 z = dot_tiles<D>(qf, kf) * scale;   // row = query, column = key
        if (more) oq.rows(qf, nt * AT);
        const f32x4 dp = dot_tiles<D>(df, vf);
        if (more) od.rows(df, nt * AT);
        f32x4 p, dz;
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const bool off = (qt == kt && 4 * g + r < (lane & 15)) || qt * AT + 4 * g + r >= S;
            p[r] = off ? 0.f : expf(z[r] - L[r]);
            dz[r] = off ? 0.f : p[r] * (dp[r] - dl[r]);
        }
        if (qt == kt && !all_finite<D>(dc)) add_cols_masked<D, false>(dv, cd, qt * AT, p);
        else add_cols<D>(dv, dc, p);
        if (more) od.cols(dc, nt * AT);
        if (qt == kt && !all_finite<D>(qc)) add_cols_masked<D, false>(dk, cq, qt * AT, dz);
        else add_cols<D>(dk, qc, dz);
        if (more) oq.cols(qc, nt * AT);
    }
    const size_t tok = (size_t)b * S + kt * AT;
    float* out = parts > 1 ? partial + ((size_t)part * B * S + tok) * (2 * nkv * D) + hk * D : dqkv + tok * ld + kcol;
    const int ldo = parts > 1 ? 2 * nkv * D : ld;
    Merge<D>::put(buf, wave, dk);
    __syncthreads();
    Merge<D>::write(buf, out, ldo, kt * AT, S, scale, parts > 1 ? nullptr : table, table_seq);
    __syncthreads();
    Merge<D>::put(buf, wave, dv);
    __syncthreads();
    Merge<D>::write(buf, out + nkv * D, ldo, kt * AT, S, 1.0f, nullptr, 0);
}

// The backward kernels deal out the jobs of several micro-batches as they do those of several samples, the longest of all of them
// first: micro-batch by micro-batch the last one's long jobs start when the others are done (8 heads of 64, 500 tokens, 8 micro-batches,
// together 156 us and 131, apart 149 and 134).
template <int D>
__global__ __launch_bounds__(AW* WAVE, 2) void k_attn_f32_bwd_q(const float* __restrict__ qkv, int ld,
                                                                const float* __restrict__ o, const float* __restrict__ dout,
                                                                const float* __restrict__ lse, float* __restrict__ dvec,
                                                                float* __restrict__ dqkv, const float* __restrict__ table, int table_seq,
                                                                F32Shape sh, MicroStride micro) {
    int qt = (int)blockIdx.x;
    const int m = split_off(qt, sh.micro);
    qkv = micro_at(qkv, micro.saved, m); o = micro_at(o, micro.saved, m); lse = micro_at(lse, micro.saved, m);
    dout = micro_at(dout, micro.ws, m); dvec = micro_at(dvec, micro.ws, m); dqkv = micro_at(dqkv, micro.ws, m);
    __shared__ __attribute__((aligned(16))) float buf[Merge<D>::FLOATS];
    const int hb = split_off(qt, sh.heads);
    bwd_q_body<D>(buf, sh.tiles - 1 - qt, hb, qkv, ld, o, dout, lse, dvec, dqkv, sh, table, table_seq);
}
template <int D>
__global__ __launch_bounds__(AW* WAVE, 1) void k_attn_f32_bwd_kv(const float* __restrict__ qkv, int ld,
                                                                 const float* __restrict__ dout, const float* __restrict__ lse,
                                                                 const float* __restrict__ dvec, float* __restrict__ dqkv,
                                                                 float* __restrict__ partial, const float* __restrict__ table, int table_seq,
                                                                 F32Shape sh, MicroStride micro) {
    int kt = (int)blockIdx.x;   // the first keys see the most queries: longest first
    const int m = split_off(kt, sh.micro);
    qkv = micro_at(qkv, micro.saved, m); lse = micro_at(lse, micro.saved, m);
    dout = micro_at(dout, micro.ws, m); dvec = micro_at(dvec, micro.ws, m); dqkv = micro_at(dqkv, micro.ws, m); partial = micro_at(partial, micro.ws, m);
    __shared__ __attribute__((aligned(16))) float buf[Merge<D>::FLOATS];
    const int rest = split_off(kt, sh.kv_jobs);
    bwd_kv_body<D, true>(buf, kt, rest, qkv, ld, nullptr, dout, lse, dvec, dqkv, partial, sh, table, table_seq);
}
// Both passes in one launch: the dk | dv jobs of key tile l and the dq jobs of query tile n-1-l, longest first.  Workgroups go to the
// 8 XCDs in turn, and in each of them to its 4 shader engines in turn.  Where the jobs of a tile are a multiple of 8, an engine would be
// given those of one pass again and again, so every 32 workgroups the passes change places: 8 heads of 64, 2000 tokens 222 -> 187 us,
// 16, 700 71 -> 61; 8 of 128, 600 tokens 69 -> 57, 500 47 -> 43.
template <int D>
__global__ __launch_bounds__(AW* WAVE, D == 64 ? 2 : 1) void k_attn_f32_bwd_both(const float* __restrict__ qkv, int ld,
                                                                const float* __restrict__ o, const float* __restrict__ dout,
                                                                const float* __restrict__ lse, float* __restrict__ dqkv,
                                                                float* __restrict__ partial, const float* __restrict__ table, int table_seq,
                                                                F32Shape sh, MicroStride micro) {
    int level = (int)blockIdx.x;
    const int m = split_off(level, sh.micro);
    qkv = micro_at(qkv, micro.saved, m); o = micro_at(o, micro.saved, m); lse = micro_at(lse, micro.saved, m);
    dout = micro_at(dout, micro.ws, m); dqkv = micro_at(dqkv, micro.ws, m); partial = micro_at(partial, micro.ws, m);
    __shared__ __attribute__((aligned(16))) float buf[Merge<D>::FLOATS];
    int r = split_off(level, sh.level);
    const int kv_jobs = sh.kv_jobs.d;
    if ((uint32_t)(level * sh.turn) >> 5 & 1u) {
        r += kv_jobs;
        if (r >= sh.level.d) r -= sh.level.d;
    }
    if (r < kv_jobs) bwd_kv_body<D, false>(buf, level, r, qkv, ld, o, dout, lse, nullptr, dqkv, partial, sh, table, table_seq);
    else bwd_q_body<D>(buf, sh.tiles - 1 - level, r - kv_jobs, qkv, ld, o, dout, lse, nullptr, dqkv, sh, table, table_seq);
}

// dk | dv of a token = the sum of its `parts` partial rows in order, dk rotated back.  A thread owns 4 channel pairs.
template <int D>
__global__ __launch_bounds__(256) void k_attn_f32_kv_reduce(const float* __restrict__ partial, int parts, float* __restrict__ dqkv, int ld,
                                                            int T, Divisor S, int nh, int nkv, Divisor per_row, const float* __restrict__ table,
                                                            int table_seq, MicroStride micro) {
    partial = micro_at(partial, micro.ws); dqkv = micro_at(dqkv, micro.ws);
    constexpr int HALF = D / 2, VPH = HALF / 4;
    int t = (int)(blockIdx.x * 256 + threadIdx.x), sample;
    const int w = split_off(t, per_row), head = w / VPH, c = (w % VPH) * 4, pos = split_off(sample = t, S);
    if (t >= T) return;
    const int width = 2 * nkv * D;
    const float* p = partial + (size_t)t * width + head * D + c;
    f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
    for (int i = 0; i < parts; i++, p += (size_t)T * width) {
        a += *reinterpret_cast<const f32x4*>(p);
        b += *reinterpret_cast<const f32x4*>(p + HALF);
    }
    if (table && head < nkv) {
        const f32x4 cs = *reinterpret_cast<const f32x4*>(table + (size_t)pos * HALF + c);
        const f32x4 sn = *reinterpret_cast<const f32x4*>(table + (size_t)(table_seq + pos) * HALF + c);
        const f32x4 ra = a * cs + b * sn, rb = b * cs - a * sn;
        a = ra; b = rb;
    }
    float* out = dqkv + (size_t)t * ld + nh * D + head * D + c;
    *reinterpret_cast<f32x4*>(out) = a;
    *reinterpret_cast<f32x4*>(out + HALF) = b;
}

static F32Shape f32_shape(int B, int S, int nh, int nkv, int parts, int micro) {
    F32Shape s;
    s.B = B; s.S = S; s.nh = nh; s.nkv = nkv; s.tiles = (S + AT - 1) / AT; s.parts = parts; s.G = nh / nkv / parts;
    s.micro = divisor(micro); s.turn = (B * (nkv * parts + nh) * micro) % 8 ? 0 : B * (nkv * parts + nh) * micro;
    s.heads = divisor(nh * B); s.nh_ = divisor(nh); s.group = divisor(nh / nkv);
    s.kv_jobs = divisor(B * nkv * parts); s.kv = divisor(nkv * parts); s.parts_ = divisor(parts); s.level = divisor(B * nkv * parts + nh * B);
    return s;
}

// The query heads that share a key/value head run one after the other in a workgroup, unless that leaves fewer than
// two workgroups per CU and the scratch holds their partial sums.  dq, dk and dv together, kept together -> dealt
// out: 8 heads of 128 on 2, 700 tokens, 202 -> 92 us; 350 tokens 101 -> 50; 16 heads of 64 on 2, 2 x 1024 tokens,
// 349 -> 261; 4 heads of 64 on 1, 128 tokens, 27 -> 30 (the reduction's launch).  A micro-batch by itself decides, so that the
// order of its sums does not depend on those beside it.
static int kv_parts(int B, int S, int nh, int nkv, size_t part_bytes, size_t scratch_bytes) {
    const int tiles = (S + AT - 1) / AT, G = nh / nkv;
    int parts = 1;
    for (int p = 2; p <= G; p++)
        if (G % p == 0 && (long)tiles * B * nkv * parts < 512 && p * part_bytes <= scratch_bytes) parts = p;
    return parts;
}

// Both passes in one launch while its jobs, those of all samples and micro-batches, are few: each pass alone is bound by its longest
// job, and the second waits for the first.  But every dk | dv job then reads o as well, and the dq jobs get the dk | dv jobs' registers,
// so that fewer of them share a CU (head_dim 64: two workgroups for three; 128: one for two).  us apart -> together, head_dim 64:
// 4 heads, 128 tokens (64 jobs) 14.2 -> 8.4; 8, 2000 (2000) 191 -> 187; 16 on 2, 2 x 1024 (2560) 257 -> 217; 32, 1000 (4032) 212 -> 209;
// 11, 2 x 1500 (4136) 300 -> 315; 24, 2000 (6000) 535 -> 554.  128: 1 head, 44 tokens 15.9 -> 8.9; 8, 500 (512) 56.5 -> 42.7; 10, 500 (640)
// 63 -> 58.  From there on it depends on the heads: 8 on 2, 700 (704) 87 -> 75, 11, 500 (704) 66 -> 68, 16, 13 x 17 (832) 21.5 -> 22.7, 8, 1000
// (1008) 126 -> 130.
static bool together(int D, long jobs) { return jobs <= (D == 64 ? 4096 : 640); }

template <int D>
static hipError_t launch_bwd(const float* qkv, int ld, const float* o, const float* dout, const float* lse, float* dvec, float* dqkv,
                             float* scratch, size_t scratch_bytes, int B, int S, int nh, int nkv, const float* table, int table_seq,
                             const MicroStride& micro, hipStream_t st) {
    const size_t part_bytes = (size_t)B * S * 2 * nkv * D * sizeof(float);
    const int parts = kv_parts(B, S, nh, nkv, part_bytes, scratch_bytes);
    const F32Shape sh = f32_shape(B, S, nh, nkv, parts, micro.n);
    const unsigned jobs_q = (unsigned)sh.tiles * B * nh * micro.n, jobs_kv = (unsigned)sh.tiles * B * nkv * parts * micro.n;
    if (together(D, (long)jobs_q + jobs_kv)) {
        k_attn_f32_bwd_both<D><<<jobs_q + jobs_kv, AW * WAVE, 0, st>>>(qkv, ld, o, dout, lse, dqkv, scratch, table, table_seq, sh, micro);
    } else {
        k_attn_f32_bwd_q<D><<<jobs_q, AW * WAVE, 0, st>>>(qkv, ld, o, dout, lse, dvec, dqkv, table, table_seq, sh, micro);
        k_attn_f32_bwd_kv<D><<<jobs_kv, AW * WAVE, 0, st>>>(qkv, ld, dout, lse, dvec, dqkv, scratch, table, table_seq, sh, micro);
    }
    if (parts > 1) {
        const long n = (long)B * S * 2 * nkv * (D / 8);
        k_attn_f32_kv_reduce<D><<<dim3((unsigned)((n + 255) / 256), micro.n), 256, 0, st>>>(scratch, parts, dqkv, ld, B * S, divisor(S), nh, nkv, divisor(2 * nkv * (D / 8)),
                                                                                            table, table_seq, micro);
    }
    return hipGetLastError();
}

hipError_t attn_f32_fwd(const void* qkv, int ld, void* o, float* lse, int B, int S, int nh, int nkv, int d, const MicroStride& micro,
                        hipStream_t st) {
    const dim3 grid((S + AT - 1) / AT * B * nh, micro.n);
    const F32Shape sh = f32_shape(B, S, nh, nkv, 1, micro.n);
    if (d == 64) k_attn_f32_fwd<64><<<grid, AW * WAVE, 0, st>>>((const float*)qkv, ld, (float*)o, lse, sh, micro);
    else if (d == 128) k_attn_f32_fwd<128><<<grid, AW * WAVE, 0, st>>>((const float*)qkv, ld, (float*)o, lse, sh, micro);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t attn_f32_bwd(const void* qkv, int ld, const void* o, const void* dout, const float* lse, float* dvec,
                        void* dqkv, float* scratch, size_t scratch_bytes, int B, int S, int nh, int nkv, int d,
                        const float* table, int table_seq, const MicroStride& micro, hipStream_t st) {
    if (d == 64) return launch_bwd<64>((const float*)qkv, ld, (const float*)o, (const float*)dout, lse, dvec, (float*)dqkv, scratch,
                                       scratch_bytes, B, S, nh, nkv, table, table_seq, micro, st);
    if (d == 128) return launch_bwd<128>((const float*)qkv, ld, (const float*)o, (const float*)dout, lse, dvec, (float*)dqkv, scratch,
                                         scratch_bytes, B, S, nh, nkv, table, table_seq, micro, st);
    return hipErrorInvalidValue;
}

}  // namespace hh

// For tests, not part of the public interface: whether the backward passes of that many micro-batches share a launch.
extern "C" int hh_internal_attn_f32_together(int B, int S, int nh, int nkv, int d, int micro) {
    using namespace hh;
    return together(d, (long)((S + AT - 1) / AT) * B * (nh + nkv * kv_parts(B, S, nh, nkv, 0, 0)) * micro);
}
