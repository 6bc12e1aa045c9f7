// HBM-bound kernels of the decoder layer: RMSNorm forward/backward (with the
// residual gradient folded in), rotary embedding, SwiGLU forward/backward and
// the column-sum reduction for the gain gradients.  All global accesses are
// 16-byte vectors along the contiguous feature dimension; math is fp32.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace hh {

constexpr int TPB = 256;
constexpr int NWAVES = TPB / WAVE;

// ------------------------------------------------------------------ RMSNorm
// A row of up to RC * TPB * V elements stays in registers between the reduction pass and the
// output pass (RC raw 16-byte vectors per thread); longer rows are re-read (from L2).
constexpr int RC = 6;

// The norms read a GEMM's product right behind it.  Where the GEMM has cut k into shares, they add the shares themselves
// (SPLIT) in place of a reduction kernel of 4 to 5 us and a pass over the product: every thread its own columns, in the order
// and with the rounding of k_ring_reduce.
__device__ __forceinline__ uint4 sum_shares(const GemmSplit& sp, int n_micro, int row, int c, const bf16_t* res) {
    const int tm = row / sp.bm, tn = c / sp.bn, tile = sp.bm * sp.bn;
    const float* p = sp.partial + ((size_t)(tm * sp.tiles_n + tn) * n_micro + blockIdx.y) * sp.ksplit * tile + (row - tm * sp.bm) * sp.bn + (c - tn * sp.bn);
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int s = 0; s < sp.ksplit; s++, p += tile) {
        const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
        v[0] += a.x; v[1] += a.y; v[2] += a.z; v[3] += a.w;
        v[4] += b.x; v[5] += b.y; v[6] += b.z; v[7] += b.w;
    }
    if (res) {
        float f[8];
        Vec<bf16_t>::load(res, f);
#pragma unroll
        for (int e = 0; e < 8; e++) v[e] += f[e];
    }
    return make_uint4(pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]), pack_bf2(v[6], v[7]));
}

template <typename T, bool SPLIT>
__device__ __forceinline__ void rmsnorm_fwd_body(T* __restrict__ x, const T* __restrict__ g, T* __restrict__ xn, float* __restrict__ r,
                                                 int H, float eps, const GemmSplit& sp, int n_micro, const T* __restrict__ res) {
    constexpr int V = Vec<T>::N;
    typedef typename Vec<T>::Raw Raw;
    __shared__ float red[NWAVES];
    const size_t base = (size_t)blockIdx.x * H;
    const bool cached = SPLIT || H <= RC * TPB * V;
    static_assert(!SPLIT || SPLIT_COLUMNS <= RC * TPB * V, "a row of shares stays in registers");
    Raw keep[RC], gain[RC];   // the gain is asked for with the row and not behind the barriers of its sum
    float ss = 0.f;
    if (cached) {
#pragma unroll
        for (int i = 0; i < RC; i++) {
            const int c = (threadIdx.x + i * TPB) * V;
            if (c < H) {
                if constexpr (SPLIT) {
                    keep[i] = sum_shares(sp, n_micro, blockIdx.x, c, res + base + c);
                    *reinterpret_cast<Raw*>(x + base + c) = keep[i];
                } else {
                    keep[i] = Vec<T>::raw(x + base + c);
                }
                gain[i] = Vec<T>::raw(g + c);
                float f[V];
                Vec<T>::widen(keep[i], f);
#pragma unroll
                for (int e = 0; e < V; e++) ss += f[e] * f[e];
            }
        }
    } else {
        for (int c = threadIdx.x * V; c < H; c += TPB * V) {
            float f[V];
            Vec<T>::load(x + base + c, f);
#pragma unroll
            for (int e = 0; e < V; e++) ss += f[e] * f[e];
        }
    }
    ss = block_sum<NWAVES>(ss, red);
    const float rs = 1.0f / sqrtf(ss / (float)H + eps);
    if (threadIdx.x == 0) r[blockIdx.x] = rs;
    if (cached) {
#pragma unroll
        for (int i = 0; i < RC; i++) {
            const int c = (threadIdx.x + i * TPB) * V;
            if (c < H) {
                float f[V], gg[V];
                Vec<T>::widen(keep[i], f);
                Vec<T>::widen(gain[i], gg);
#pragma unroll
                for (int e = 0; e < V; e++) f[e] = f[e] * rs * gg[e];
                Vec<T>::store(xn + base + c, f);
            }
        }
    } else {
        for (int c = threadIdx.x * V; c < H; c += TPB * V) {
            float f[V], gg[V];
            Vec<T>::load(x + base + c, f);
            Vec<T>::load(g + c, gg);
#pragma unroll
            for (int e = 0; e < V; e++) f[e] = f[e] * rs * gg[e];
            Vec<T>::store(xn + base + c, f);
        }
    }
}

// Micro-batches side by side: blockIdx.y.
template <int N>
static Ops<N> ops(const Each& e) {
    Ops<N> o;
    for (int m = 0; m < N; m++) o.p[m] = e.p[m];
    return o;
}
template <typename T, int N>
__global__ __launch_bounds__(TPB) void k_rmsnorm_fwd(Ops<N> x, const T* g, Ops<N> xn, Ops<N> r, int H, float eps) {
    const int m = blockIdx.y;
    rmsnorm_fwd_body<T, false>((T*)x.at(m), g, (T*)xn.at(m), (float*)r.at(m), H, eps, GemmSplit{}, 1, nullptr);
}
template <int N>
__global__ __launch_bounds__(TPB) void k_rmsnorm_fwd_split(GemmSplit sp, int n, Ops<N> res, Ops<N> x, const bf16_t* g, Ops<N> xn, Ops<N> r, int H,
                                                           float eps) {
    const int m = blockIdx.y;
    rmsnorm_fwd_body<bf16_t, true>((bf16_t*)x.at(m), g, (bf16_t*)xn.at(m), (float*)r.at(m), H, eps, sp, N == 1 ? 1 : n, (const bf16_t*)res.at(m));
}

// The operands of the backward kernels, one per micro-batch but for the gain.
template <int N>
struct NormBwd {
    Ops<N> dxn, x, r, dres, dx, partial;
    const void* g;
    int T, H, rpb, nblk, n;
    GemmSplit split;
    float* gain;      // not null: workgroups nblk .. of micro-batch 0 write its gradient, and nobody partial sums
    int accumulate;
    int gain_blocks() const { return gain ? (H + 63) / 64 : 0; }
};

// The gain's gradient straight from the rows: a workgroup covers 64 columns (16 lanes of 4) with NT / 16 row groups, the
// micro-batches one after the other, each added to those before it.  The rows are read a second time, from L2, but beside the
// workgroups that norm them, which spares the launch that sums partial rows: up to GAIN_ROWS rows a micro-batch, beyond which
// these workgroups would take longer than the others.  fp32 step of hidden 256, 128 tokens: 89.8 -> 87.9 us.
constexpr int GAIN_ROWS = 256;
constexpr int GAIN_COLUMNS = 6 * TPB * Vec<float>::N;
template <typename T> struct Quad;
template <> struct Quad<float> {
    __device__ static __forceinline__ float4 load(const float* p) { return *reinterpret_cast<const float4*>(p); }
};
template <> struct Quad<bf16_t> {
    __device__ static __forceinline__ float4 load(const bf16_t* p) {
        const uint2 w = *reinterpret_cast<const uint2*>(p);
        return make_float4(lo_bf(w.x), hi_bf(w.x), lo_bf(w.y), hi_bf(w.y));
    }
};
template <typename T, int NT, int N>
__device__ __forceinline__ void gain_columns(const NormBwd<N>& a) {
    __shared__ float4 red[2][NT / WAVE][16];
    const int H = a.H, rows = a.T, cx = threadIdx.x % 16, wave = threadIdx.x / WAVE;
    const int col = ((blockIdx.x - a.nblk) * 16 + cx) * 4;
    const bool owner = threadIdx.x < 16 && col < H;
    float4* const out = reinterpret_cast<float4*>(a.gain + col);
    float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
    if (owner && a.accumulate) sum = *out;
    for (int m = 0; m < (N == 1 ? 1 : a.n); m++) {
        const T* dxn = (const T*)a.dxn.at(m) + col;
        const T* x = (const T*)a.x.at(m) + col;
        const float* r = (const float*)a.r.at(m);
        float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
        if (col < H) {
#pragma unroll 4
            for (int t = threadIdx.x / 16; t < rows; t += NT / 16) {
                const float4 d = Quad<T>::load(dxn + (size_t)t * H), xx = Quad<T>::load(x + (size_t)t * H);
                const float rs = r[t];
                s.x = fmaf(d.x, xx.x * rs, s.x); s.y = fmaf(d.y, xx.y * rs, s.y);
                s.z = fmaf(d.z, xx.z * rs, s.z); s.w = fmaf(d.w, xx.w * rs, s.w);
            }
        }
#pragma unroll
        for (int o = 16; o < WAVE; o *= 2) {
            s.x += __shfl_xor(s.x, o, WAVE); s.y += __shfl_xor(s.y, o, WAVE);
            s.z += __shfl_xor(s.z, o, WAVE); s.w += __shfl_xor(s.w, o, WAVE);
        }
        if ((threadIdx.x & (WAVE - 1)) < 16) red[m & 1][wave][cx] = s;
        __syncthreads();   // red[m & 1] is written again two barriers after its readers
        if (owner) {
            float4 t = red[m & 1][0][cx];
#pragma unroll
            for (int i = 1; i < NT / WAVE; i++) {
                const float4 v = red[m & 1][i][cx];
                t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w;
            }
            if (a.accumulate || m) { sum.x = t.x + sum.x; sum.y = t.y + sum.y; sum.z = t.z + sum.z; sum.w = t.w + sum.w; }
            else sum = t;
        }
    }
    if (owner) *out = sum;
}

// RMSNorm backward, rows too long for registers: one workgroup walks `rpb` consecutive rows and reads each twice.
// Column j is always handled by the same thread, so the per-column sums of dxn*u live in LDS without atomics.
template <typename T>
__device__ __forceinline__ void rmsnorm_bwd_body(const T* __restrict__ dxn, const T* __restrict__ x, const float* __restrict__ r, const T* __restrict__ g,
                                                 const T* __restrict__ dres, T* __restrict__ dx, float* __restrict__ partial,
                                                 int T_rows, int H, int rpb) {
    constexpr int V = Vec<T>::N;
    extern __shared__ float colacc[];  // [H]
    __shared__ float red[NWAVES];
    for (int c = threadIdx.x * V; c < H; c += TPB * V)
#pragma unroll
        for (int e = 0; e < V; e++) colacc[c + e] = 0.f;
    const int row0 = blockIdx.x * rpb;
    const int row1 = min(T_rows, row0 + rpb);
    const float invH = 1.0f / (float)H;
    for (int row = row0; row < row1; row++) {
        const size_t base = (size_t)row * H;
        const float rs = r[row];
        float s = 0.f;
        for (int c = threadIdx.x * V; c < H; c += TPB * V) {
            float d[V], xx[V], gg[V];
            Vec<T>::load(dxn + base + c, d);
            Vec<T>::load(x + base + c, xx);
            Vec<T>::load(g + c, gg);
#pragma unroll
            for (int e = 0; e < V; e++) s += d[e] * gg[e] * xx[e];
        }
        const float c1 = block_sum<NWAVES>(s, red) * rs * invH;  // mean_j(w_j u_j)
        for (int c = threadIdx.x * V; c < H; c += TPB * V) {
            float d[V], xx[V], gg[V], rr[V], o[V];
            Vec<T>::load(dxn + base + c, d);
            Vec<T>::load(x + base + c, xx);
            Vec<T>::load(g + c, gg);
            Vec<T>::load(dres + base + c, rr);
#pragma unroll
            for (int e = 0; e < V; e++) {
                const float u = xx[e] * rs;
                colacc[c + e] += d[e] * u;
                o[e] = rr[e] + rs * (d[e] * gg[e] - u * c1);
            }
            Vec<T>::store(dx + base + c, o);
        }
    }
    float* out = partial + (size_t)blockIdx.x * H;
    for (int c = threadIdx.x * V; c < H; c += TPB * V)
#pragma unroll
        for (int e = 0; e < V; e++) out[c + e] = colacc[c + e];
}

template <typename T, int N>
__global__ __launch_bounds__(TPB) void k_rmsnorm_bwd(NormBwd<N> a) {
    const int m = blockIdx.y;
    rmsnorm_bwd_body<T>((const T*)a.dxn.at(m), (const T*)a.x.at(m), (const float*)a.r.at(m), (const T*)a.g, (const T*)a.dres.at(m),
                        (T*)a.dx.at(m), (float*)a.partial.at(m), a.T, a.H, a.rpb);
}

// RMSNorm backward, short rows (at most NV * 64 * V elements): one wave per row, no barrier until the end; a lane's
// columns are the same in every row, so their sums stay in registers and the waves' sums meet in LDS once, in a fixed
// order.  Bound by latency: one row at a time per workgroup of 256 threads, most of them idle, took 9.6-11.3 us for
// 128 rows of 256 and 20.8 us for 2200 rows of 512 (bf16); this kernel with one to nine rows a workgroup takes
// 3.0-4.2 and 4.8 us.
constexpr int RW = 8;   // waves per workgroup
template <typename T, int NV, bool SPLIT>
__device__ __forceinline__ void rmsnorm_bwd_wave_body(const T* __restrict__ dxn, const T* __restrict__ x, const float* __restrict__ r, const T* __restrict__ g,
                                                      const T* __restrict__ dres, T* __restrict__ dx, float* __restrict__ partial,
                                                      int T_rows, int H, int rpb,
                                                      const GemmSplit& sp, int n_micro) {
    constexpr int V = Vec<T>::N;
    extern __shared__ float colsum[];  // [RW][H]
    const int wave = threadIdx.x / WAVE, lane = threadIdx.x & (WAVE - 1);
    const int row0 = blockIdx.x * rpb, row1 = min(T_rows, row0 + rpb);
    const float invH = 1.0f / (float)H;
    float gg[NV][V], acc[NV][V];
#pragma unroll
    for (int i = 0; i < NV; i++) {
        const int c = (lane + i * WAVE) * V;
        if (c < H) Vec<T>::load(g + c, gg[i]);
#pragma unroll
        for (int e = 0; e < V; e++) acc[i][e] = 0.f;
    }
    for (int row = row0 + wave; row < row1; row += RW) {
        const size_t base = (size_t)row * H;
        const float rs = r[row];
        float d[NV][V], xx[NV][V], rr[NV][V];
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < NV; i++) {
            const int c = (lane + i * WAVE) * V;
            if (c < H) {
                if constexpr (SPLIT) Vec<T>::widen(sum_shares(sp, n_micro, row, c, nullptr), d[i]);
                else Vec<T>::load(dxn + base + c, d[i]);
                Vec<T>::load(x + base + c, xx[i]);
                Vec<T>::load(dres + base + c, rr[i]);
#pragma unroll
                for (int e = 0; e < V; e++) s += d[i][e] * gg[i][e] * xx[i][e];
            }
        }
        const float c1 = wave_sum(s) * rs * invH;  // mean_j(w_j u_j)
#pragma unroll
        for (int i = 0; i < NV; i++) {
            const int c = (lane + i * WAVE) * V;
            if (c < H) {
                float o[V];
#pragma unroll
                for (int e = 0; e < V; e++) {
                    const float u = xx[i][e] * rs;
                    acc[i][e] += d[i][e] * u;
                    o[e] = rr[i][e] + rs * (d[i][e] * gg[i][e] - u * c1);
                }
                Vec<T>::store(dx + base + c, o);
            }
        }
    }
    if (!partial) return;
#pragma unroll
    for (int i = 0; i < NV; i++) {
        const int c = (lane + i * WAVE) * V;
        if (c < H)
#pragma unroll
            for (int e = 0; e < V; e += 4)
                *reinterpret_cast<float4*>(colsum + wave * H + c + e) = make_float4(acc[i][e], acc[i][e + 1], acc[i][e + 2], acc[i][e + 3]);
    }
    __syncthreads();
    const int waves = min(RW, row1 - row0);   // waves that had a row
    for (int c = threadIdx.x; c < H; c += RW * WAVE) {
        float s = 0.f;
        for (int w = 0; w < waves; w++) s += colsum[w * H + c];
        partial[(size_t)blockIdx.x * H + c] = s;
    }
}

template <typename T, int NV, int N, bool SPLIT>
__global__ __launch_bounds__(RW * WAVE) void k_rmsnorm_bwd_wave(NormBwd<N> a) {
    const int m = blockIdx.y;
    if (a.gain && (int)blockIdx.x >= a.nblk) {
        if constexpr (!SPLIT)
            if (m == 0) gain_columns<T, RW * WAVE, N>(a);
        return;
    }
    rmsnorm_bwd_wave_body<T, NV, SPLIT>((const T*)a.dxn.at(m), (const T*)a.x.at(m), (const float*)a.r.at(m), (const T*)a.g, (const T*)a.dres.at(m),
                                 (T*)a.dx.at(m), a.gain ? nullptr : (float*)a.partial.at(m), a.T, a.H, a.rpb, a.split, N == 1 ? 1 : a.n);
}

// out[j] (=|+=) sum_b partial[b][j] of one or two gain gradients (blockIdx.y).  A workgroup covers 64 columns (a float4
// per lane, 16 lanes a row) with 64 row groups, combined by shuffles and through LDS in a fixed order: at most 256
// partial rows are then one batch of loads per thread, and a row of 4096 is spread over 64 CUs.  Both sums at 256 x 12288
// and at 254 x 4096: 12.8 and 11.8 us as two launches of 256 columns a workgroup, 7.6 and 6.0 us as this one.
constexpr int CSW = 16;   // waves of a workgroup
template <int N>
struct ColSums {
    struct { Ops<N> partial; int rows; float* out; } j[2];
};
template <int N>
__global__ __launch_bounds__(CSW * WAVE) void k_colsum_reduce(ColSums<N> sums, int n, int H, int accumulate) {
    __shared__ float4 red[2][CSW][16];
    const auto& j = sums.j[blockIdx.y];
    const int cx = threadIdx.x % 16, wave = threadIdx.x / WAVE;
    const int col = (blockIdx.x * 16 + cx) * 4;
    const bool owner = threadIdx.x < 16 && col < H;
    float4* const out = reinterpret_cast<float4*>(j.out + col);
    float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
    if (owner && accumulate) sum = *out;
    // A thread's first rows of the next micro-batch, all of them with up to 256 rows, are asked for before this one's are combined: a round
    // trip to memory less for each (2 layers of hidden 512, three micro-batches of 2200 tokens 714 -> 707 us; 4 of hidden 256 1181 -> 1172).
    constexpr int GROUPS = CSW * WAVE / 16, AHEAD = 4;
    float4 next[AHEAD];
    auto ask = [&](int m) {
        const float* p = (const float*)j.partial.at(m) + col;
#pragma unroll
        for (int q = 0; q < AHEAD; q++) {
            const int i = threadIdx.x / 16 + q * GROUPS;
            next[q] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (col < H && i < j.rows) next[q] = *reinterpret_cast<const float4*>(p + (size_t)i * H);
        }
    };
    ask(0);
    for (int m = 0; m < (N == 1 ? 1 : n); m++) {   // each micro-batch's sum is added to those before it, as n calls would
        float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int q = 0; q < AHEAD; q++) { s.x += next[q].x; s.y += next[q].y; s.z += next[q].z; s.w += next[q].w; }
        if (col < H) {
            const float* p = (const float*)j.partial.at(m) + col;
            for (int i = threadIdx.x / 16 + AHEAD * GROUPS; i < j.rows; i += GROUPS) {
                const float4 v = *reinterpret_cast<const float4*>(p + (size_t)i * H);
                s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
            }
        }
        if (N > 1 && m + 1 < n) ask(m + 1);
#pragma unroll
        for (int o = 16; o < WAVE; o *= 2) {
            s.x += __shfl_xor(s.x, o, WAVE); s.y += __shfl_xor(s.y, o, WAVE);
            s.z += __shfl_xor(s.z, o, WAVE); s.w += __shfl_xor(s.w, o, WAVE);
        }
        if ((threadIdx.x & (WAVE - 1)) < 16) red[m & 1][wave][cx] = s;
        lds_barrier();   // red[m & 1] is written again two barriers after its readers
        if (owner) {
            float4 t = red[m & 1][0][cx];
#pragma unroll
            for (int i = 1; i < CSW; i++) {
                const float4 v = red[m & 1][i][cx];
                t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w;
            }
            if (accumulate || m) { sum.x = t.x + sum.x; sum.y = t.y + sum.y; sum.z = t.z + sum.z; sum.w = t.w + sum.w; }
            else sum = t;
        }
    }
    if (owner) *out = sum;
}

// --------------------------------------------------------------------- RoPE
// One thread rotates V pairs (i, i + d/2) of one of the nrot heads that start at column 0 of a token's row
// (the query heads followed by the key heads).
template <typename T, int N>
__global__ __launch_bounds__(TPB) void k_rope(Ops<N> qkv, int ld, int Ttok, Divisor S, Divisor nrot, int d, Divisor vph,   // vph: vectors of a head-half
                                              const float* __restrict__ table, int table_seq) {
    constexpr int V = Vec<T>::N;
    const int half = d / 2;
    int t = (int)(blockIdx.x * TPB + threadIdx.x);
    const int iv = split_off(t, vph), head = split_off(t, nrot);
    if (t >= Ttok) return;
    int sample = t;
    const int pos = split_off(sample, S);
    T* p = (T*)qkv.at(blockIdx.y) + (size_t)t * ld + (size_t)head * d + iv * V;
    const float* cs = table + ((size_t)pos * half + iv * V);
    const float* sn = cs + (size_t)table_seq * half;
    float a[V], b[V];
    Vec<T>::load(p, a);
    Vec<T>::load(p + half, b);
#pragma unroll
    for (int e = 0; e < V; e++) rotate_pair(a[e], b[e], cs[e], sn[e]);
    Vec<T>::store(p, a);
    Vec<T>::store(p + half, b);
}

// ------------------------------------------------------------------- SwiGLU
template <typename T, int N>
__global__ __launch_bounds__(TPB) void k_swiglu_fwd(Ops<N> gu_, Ops<N> m_, int Ttok, int F, Divisor vpr) {
    constexpr int V = Vec<T>::N;
    const T* gu = (const T*)gu_.at(blockIdx.y);
    T* m = (T*)m_.at(blockIdx.y);
    int t = (int)(blockIdx.x * TPB + threadIdx.x);
    const int c = split_off(t, vpr) * V;
    if (t >= Ttok) return;
    float gt[V], u[V], o[V];
    Vec<T>::load(gu + (size_t)t * 2 * F + c, gt);
    Vec<T>::load(gu + (size_t)t * 2 * F + F + c, u);
#pragma unroll
    for (int e = 0; e < V; e++) o[e] = swiglu(gt[e], u[e]);
    Vec<T>::store(m + (size_t)t * F + c, o);
}

template <typename T, int N>
__global__ __launch_bounds__(TPB) void k_swiglu_bwd(Ops<N> dm_, Ops<N> gu_, Ops<N> dgu_, Ops<N> m_, int Ttok, int F, Divisor vpr) {
    constexpr int V = Vec<T>::N;
    const T *dm = (const T*)dm_.at(blockIdx.y), *gu = (const T*)gu_.at(blockIdx.y);
    T *dgu = (T*)dgu_.at(blockIdx.y), *m = (T*)m_.at(blockIdx.y);
    int t = (int)(blockIdx.x * TPB + threadIdx.x);
    const int c = split_off(t, vpr) * V;
    if (t >= Ttok) return;
    float gt[V], u[V], d[V], og[V], ou[V], om[V];
    Vec<T>::load(gu + (size_t)t * 2 * F + c, gt);
    Vec<T>::load(gu + (size_t)t * 2 * F + F + c, u);
    Vec<T>::load(dm + (size_t)t * F + c, d);
#pragma unroll
    for (int e = 0; e < V; e++) swiglu_grad(gt[e], u[e], d[e], og[e], ou[e], om[e]);
    Vec<T>::store(dgu + (size_t)t * 2 * F + c, og);
    Vec<T>::store(dgu + (size_t)t * 2 * F + F + c, ou);
    Vec<T>::store(m + (size_t)t * F + c, om);
}

// ---------------------------------------------------------------- launchers
static inline unsigned nblocks(long n) { return (unsigned)((n + TPB - 1) / TPB); }

template <typename T>
static void rmsnorm_fwd_t(const Each& x, const void* g, const Each& xn, const Each& r, int n, int T_, int H, float eps, hipStream_t st) {
    if (n == 1) k_rmsnorm_fwd<T, 1><<<T_, TPB, 0, st>>>(ops<1>(x), (const T*)g, ops<1>(xn), ops<1>(r), H, eps);
    else
        k_rmsnorm_fwd<T, MICRO_MAX><<<dim3(T_, n), TPB, 0, st>>>(ops<MICRO_MAX>(x), (const T*)g, ops<MICRO_MAX>(xn), ops<MICRO_MAX>(r), H, eps);
}
template <int N>
static void rmsnorm_fwd_split(const GemmSplit& sp, const Each& res, const Each& x, const void* g, const Each& xn, const Each& r, int n, int T, int H,
                              float eps, hipStream_t st) {
    k_rmsnorm_fwd_split<N><<<dim3(T, n), TPB, 0, st>>>(sp, n, ops<N>(res), ops<N>(x), (const bf16_t*)g, ops<N>(xn), ops<N>(r), H, eps);
}
hipError_t rmsnorm_fwd(int dtype, const Each& x, const void* g, const Each& xn, const Each& r, int n, int T, int H, float eps,
                       hipStream_t st, const GemmSplit* split, const Each* res) {
    if (split) {
        if (dtype != DT_BF16 || !res || H > SPLIT_COLUMNS) return hipErrorInvalidValue;
        if (n == 1) rmsnorm_fwd_split<1>(*split, *res, x, g, xn, r, n, T, H, eps, st);
        else rmsnorm_fwd_split<MICRO_MAX>(*split, *res, x, g, xn, r, n, T, H, eps, st);
        return hipGetLastError();
    }
    if (dtype == DT_BF16) rmsnorm_fwd_t<bf16_t>(x, g, xn, r, n, T, H, eps, st);
    else rmsnorm_fwd_t<float>(x, g, xn, r, n, T, H, eps, st);
    return hipGetLastError();
}

// Rows of up to NV * TPB * V elements (exactly that many unless GUARD): the three input rows of row r + 1 are requested before row r is
// reduced and written, each in its own registers, so the memory queue never drains between rows.  The one
// barrier per row waits for LDS only (a full workgroup fence would also wait for the loads in flight).
__device__ __forceinline__ void keep_raw(uint4& v) { asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w)); }
__device__ __forceinline__ void keep_raw(float4& v) { asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w)); }

template <typename T, int NV, bool GUARD, bool SPLIT>
__device__ __forceinline__ void rmsnorm_bwd_rows_body(const T* __restrict__ dxn, const T* __restrict__ x, const float* __restrict__ r, const T* __restrict__ g,
                                                      const T* __restrict__ dres, T* __restrict__ dx, float* __restrict__ partial,
                                                      int T_rows, int H_, int rpb,
                                                      const GemmSplit& sp, int n_micro) {
    constexpr int V = Vec<T>::N;
    const int H = GUARD ? H_ : NV * TPB * V;
    typedef typename Vec<T>::Raw Raw;
    extern __shared__ float colacc[];  // [H]
    __shared__ float red[2][NWAVES];
    struct Row { Raw d[NV], x[NV], res[NV]; float rs; };
    auto fetch = [&](Row& w, int row) {
        const size_t base = (size_t)row * H;
#pragma unroll
        for (int i = 0; i < NV; i++) {
            const int c = (threadIdx.x + i * TPB) * V;
            if (GUARD && c >= H) break;
            if constexpr (SPLIT) w.d[i] = sum_shares(sp, n_micro, row, c, nullptr);
            else w.d[i] = Vec<T>::raw(dxn + base + c);
            w.x[i] = Vec<T>::raw(x + base + c);
            w.res[i] = Vec<T>::raw(dres + base + c);
        }
        w.rs = r[row];
    };
    Raw gain[NV];
#pragma unroll
    for (int i = 0; i < NV; i++) {
        const int c = (threadIdx.x + i * TPB) * V;
        if (GUARD && c >= H) break;
        gain[i] = Vec<T>::raw(g + c);
#pragma unroll
        for (int e = 0; e < V; e++) colacc[c + e] = 0.f;   // only this thread ever touches these columns
    }
    const int row0 = blockIdx.x * rpb;
    const int row1 = min(T_rows, row0 + rpb);
    const float invH = 1.0f / (float)H;
    const int wave = threadIdx.x / WAVE, lane = threadIdx.x & (WAVE - 1);
    auto finish = [&](Row& w, int row) {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < NV; i++) {
            if (GUARD && (threadIdx.x + i * TPB) * V >= H) break;
            float d[V], xx[V], gg[V];
            Vec<T>::widen(w.d[i], d);
            Vec<T>::widen(w.x[i], xx);
            Vec<T>::widen(gain[i], gg);
#pragma unroll
            for (int e = 0; e < V; e++) s += d[e] * gg[e] * xx[e];
        }
        s = wave_sum(s);
        float* rd = red[row & 1];      // the other parity's readers are a barrier behind at most
        if (lane == 0) rd[wave] = s;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        float tot = 0.f;
#pragma unroll
        for (int i = 0; i < NWAVES; i++) tot += rd[i];
        // the raw rows are unpacked a second time below: keeping the fp32 copies of the first pass alive
        // across the barrier would double the registers a row takes
#pragma unroll
        for (int i = 0; i < NV; i++) { keep_raw(w.d[i]); keep_raw(w.x[i]); }
        const float rs = w.rs;
        const float c1 = tot * rs * invH;  // mean_j(w_j u_j)
        const size_t base = (size_t)row * H;
#pragma unroll
        for (int i = 0; i < NV; i++) {
            const int c = (threadIdx.x + i * TPB) * V;
            if (GUARD && c >= H) break;
            float d[V], xx[V], gg[V], rr[V], o[V];
            Vec<T>::widen(w.d[i], d);
            Vec<T>::widen(w.x[i], xx);
            Vec<T>::widen(gain[i], gg);
            Vec<T>::widen(w.res[i], rr);
#pragma unroll
            for (int e = 0; e < V; e++) {
                const float u = xx[e] * rs;
                colacc[c + e] += d[e] * u;
                o[e] = rr[e] + rs * (d[e] * gg[e] - u * c1);
            }
            Vec<T>::store(dx + base + c, o);
        }
    };
    if (row0 >= row1) return;
    // fetches past the block's last row re-read that row (in bounds, unused): no branch around a request
    const int last = row1 - 1;
    Row a, b;
    fetch(a, row0);
    for (int row = row0; row < row1; row += 2) {
        fetch(b, min(row + 1, last));
        finish(a, row);
        fetch(a, min(row + 2, last));
        if (row + 1 < row1) finish(b, row + 1);
    }
    if (!partial) return;
#pragma unroll
    for (int i = 0; i < NV; i++) {
        const int c = (threadIdx.x + i * TPB) * V;
        if (GUARD && c >= H) break;
#pragma unroll
        for (int e = 0; e < V; e++) partial[(size_t)blockIdx.x * H + c + e] = colacc[c + e];
    }
}

template <typename T, int NV, bool GUARD, int N, bool SPLIT>
__global__ __launch_bounds__(TPB, 2) void k_rmsnorm_bwd_rows(NormBwd<N> a) {
    const int m = blockIdx.y;
    if (a.gain && (int)blockIdx.x >= a.nblk) {
        if constexpr (!SPLIT)
            if (m == 0) gain_columns<T, TPB, N>(a);
        return;
    }
    rmsnorm_bwd_rows_body<T, NV, GUARD, SPLIT>((const T*)a.dxn.at(m), (const T*)a.x.at(m), (const float*)a.r.at(m), (const T*)a.g, (const T*)a.dres.at(m),
                                        (T*)a.dx.at(m), a.gain ? nullptr : (float*)a.partial.at(m), a.T, a.H, a.rpb, a.split, N == 1 ? 1 : a.n);
}

// One micro-batch, partial sums, no shares: the large launches.  Pointers as arguments of their own, of which the compiler knows
// that they do not overlap: 4096 rows of 8192 58.8 us, 61.5 with the pointers in a struct.
template <typename T, int NV, bool GUARD>
__global__ __launch_bounds__(TPB, 2) void k_rmsnorm_bwd_rows_one(const T* __restrict__ dxn, const T* __restrict__ x, const float* __restrict__ r,
                                                                 const T* __restrict__ g, const T* __restrict__ dres, T* __restrict__ dx,
                                                                 float* __restrict__ partial, int T_rows, int H, int rpb) {
    rmsnorm_bwd_rows_body<T, NV, GUARD, false>(dxn, x, r, g, dres, dx, partial, T_rows, H, rpb, GemmSplit{}, 1);
}

template <typename T, int NV, bool GUARD, int N>
static hipError_t launch_rows(const NormBwd<N>& a, hipStream_t st) {
    const int lds = a.H * (int)sizeof(float);   // at most 48 KB
    constexpr int FEWER = (NV - 1) * TPB * Vec<T>::N;   // columns, and rows have more than that
    if constexpr (sizeof(T) == 2 && FEWER < SPLIT_COLUMNS)
        if (a.split.partial) {
            k_rmsnorm_bwd_rows<T, NV, GUARD, N, true><<<dim3(a.nblk, a.n), TPB, lds, st>>>(a);
            return hipGetLastError();
        }
    if constexpr (N == 1)
        if (!a.gain) {
            k_rmsnorm_bwd_rows_one<T, NV, GUARD><<<a.nblk, TPB, lds, st>>>((const T*)a.dxn.p[0], (const T*)a.x.p[0], (const float*)a.r.p[0], (const T*)a.g,
                                                                           (const T*)a.dres.p[0], (T*)a.dx.p[0], (float*)a.partial.p[0], a.T, a.H, a.rpb);
            return hipGetLastError();
        }
    if constexpr (N > 1 || FEWER < GAIN_COLUMNS) k_rmsnorm_bwd_rows<T, NV, GUARD, N, false><<<dim3(a.nblk + a.gain_blocks(), a.n), TPB, lds, st>>>(a);
    return hipGetLastError();
}
template <typename T, int NV, int N>
static hipError_t launch_wave(const NormBwd<N>& a, hipStream_t st) {
    const int lds = RW * a.H * (int)sizeof(float);   // at most 64 KB
    constexpr int MOST = RW * NV * WAVE * Vec<T>::N * (int)sizeof(float);
    static std::atomic<uint64_t> lds_ok[2];
    if constexpr (sizeof(T) == 2)
        if (a.split.partial) {
            const hipError_t e = allow_lds((const void*)k_rmsnorm_bwd_wave<T, NV, N, true>, MOST, lds_ok[1]);
            if (e != hipSuccess) return e;
            k_rmsnorm_bwd_wave<T, NV, N, true><<<dim3(a.nblk, a.n), RW * WAVE, lds, st>>>(a);
            return hipGetLastError();
        }
    const hipError_t e = allow_lds((const void*)k_rmsnorm_bwd_wave<T, NV, N, false>, MOST, lds_ok[0]);
    if (e != hipSuccess) return e;
    k_rmsnorm_bwd_wave<T, NV, N, false><<<dim3(a.nblk + a.gain_blocks(), a.n), RW * WAVE, lds, st>>>(a);
    return hipGetLastError();
}

// Workgroups (= rows of `partial`) of rmsnorm_bwd: as few rows each as 256 of them leave, so that neither a short
// batch nor a ragged one idles CUs (700 rows: 234 workgroups of 3, 3300 rows: 254 of 13), and no more of them than
// `partial` has room for.
static inline int rms_rows_per_block(int T, int H, size_t partial_bytes) {
    const size_t room = partial_bytes / ((size_t)H * sizeof(float));
    const int most = (int)std::max<size_t>(1, std::min<size_t>(256, room));
    return (T + most - 1) / most;
}
int rmsnorm_bwd_blocks(int T, int H, size_t partial_bytes) {
    const int rpb = rms_rows_per_block(T, H, partial_bytes);
    return (T + rpb - 1) / rpb;
}

template <typename T, int N>
static hipError_t rmsnorm_bwd_t(const NormBwd<N>& a, hipStream_t st) {
    constexpr int V = Vec<T>::N;
    // A wave per row up to two vectors a lane, a workgroup per row beyond (four times the threads at work on a row), whose rows
    // are pipelined; but up to four vectors a lane still a wave per row where a workgroup's row is not whole (a guard around
    // every request): 3820 rows of 1984 20.0 -> 15.1 us, 333 rows of 1280 in 42 workgroups 9.8 -> 6.8, 700 of 1536 in 234 6.2 and
    // 6.4; 2048 rows of 2048, whole, 9.9 and 11.1.
    if (a.H <= WAVE * V) return launch_wave<T, 1>(a, st);
    if (a.H <= 2 * WAVE * V) return launch_wave<T, 2>(a, st);
    const bool whole = a.H % (TPB * V) == 0;   // row length as a compile-time multiple of the workgroup's 16-byte vectors
    switch ((a.H + TPB * V - 1) / (TPB * V)) {
        case 1: return whole ? launch_rows<T, 1, false>(a, st) : a.H <= 3 * WAVE * V ? launch_wave<T, 3>(a, st) : launch_wave<T, 4>(a, st);
        case 2: return whole ? launch_rows<T, 2, false>(a, st) : launch_rows<T, 2, true>(a, st);
        case 3: return whole ? launch_rows<T, 3, false>(a, st) : launch_rows<T, 3, true>(a, st);
        case 4: return whole ? launch_rows<T, 4, false>(a, st) : launch_rows<T, 4, true>(a, st);
        case 5: return whole ? launch_rows<T, 5, false>(a, st) : launch_rows<T, 5, true>(a, st);
        case 6: return whole ? launch_rows<T, 6, false>(a, st) : launch_rows<T, 6, true>(a, st);
    }
    const int lds = a.H * (int)sizeof(float);
    static std::atomic<uint64_t> lds_ok{0};
    const hipError_t e = allow_lds((const void*)k_rmsnorm_bwd<T, N>, 32768 * (int)sizeof(float), lds_ok);
    if (e != hipSuccess) return e;
    k_rmsnorm_bwd<T, N><<<dim3(a.nblk, a.n), TPB, lds, st>>>(a);
    return hipGetLastError();
}

// Not from shares: the columns' workgroups would have to add them up as well.
bool rmsnorm_bwd_sums_gain(int T, int H, const GemmSplit* split) { return T <= GAIN_ROWS && H <= GAIN_COLUMNS && !split; }

template <int N>
static hipError_t rmsnorm_bwd_n(int dtype, const Each& dxn, const Each& x, const Each& r, const void* g, const Each& dres,
                                const Each& dx, const Each& partial, size_t partial_bytes, int n, int T, int H, hipStream_t st,
                                const GemmSplit* split, float* gain, int accumulate) {
    NormBwd<N> a{ops<N>(dxn), ops<N>(x), ops<N>(r), ops<N>(dres), ops<N>(dx), ops<N>(partial), g, T, H, rms_rows_per_block(T, H, partial_bytes),
                 0, n, split ? *split : GemmSplit{}, gain, accumulate};
    a.nblk = (T + a.rpb - 1) / a.rpb;
    return dtype == DT_BF16 ? rmsnorm_bwd_t<bf16_t>(a, st) : rmsnorm_bwd_t<float>(a, st);
}
hipError_t rmsnorm_bwd(int dtype, const Each& dxn, const Each& x, const Each& r, const void* g, const Each& dres,
                       const Each& dx, const Each& partial, size_t partial_bytes, int n, int T, int H, hipStream_t st, const GemmSplit* split, float* gain, int accumulate) {
    if (split && (gain || dtype != DT_BF16 || H > SPLIT_COLUMNS)) return hipErrorInvalidValue;
    if (gain && H > GAIN_COLUMNS) return hipErrorInvalidValue;
    return n == 1 ? rmsnorm_bwd_n<1>(dtype, dxn, x, r, g, dres, dx, partial, partial_bytes, n, T, H, st, split, gain, accumulate)
                  : rmsnorm_bwd_n<MICRO_MAX>(dtype, dxn, x, r, g, dres, dx, partial, partial_bytes, n, T, H, st, split, gain, accumulate);
}

template <int N>
static void colsum_n(const ColSum* jobs, int n_jobs, int n, int H, int accumulate, hipStream_t st) {
    ColSums<N> s;
    for (int i = 0; i < 2; i++) {
        const ColSum& q = jobs[std::min(i, n_jobs - 1)];
        s.j[i] = {ops<N>(q.partial), q.rows, q.out};
    }
    k_colsum_reduce<N><<<dim3((H + 63) / 64, n_jobs), CSW * WAVE, 0, st>>>(s, n, H, accumulate);
}
hipError_t colsum_reduce(const ColSum* jobs, int n_jobs, int n, int H, int accumulate, hipStream_t st) {
    if (n == 1) colsum_n<1>(jobs, n_jobs, n, H, accumulate, st);
    else colsum_n<MICRO_MAX>(jobs, n_jobs, n, H, accumulate, st);
    return hipGetLastError();
}

template <typename T, int N>
static void rope_t(const Each& qkv, int ld, int n, int Ttok, int S, int nrot, int d, const float* table, int table_seq, hipStream_t st) {
    const long vecs = (long)Ttok * nrot * (d / 2 / Vec<T>::N);
    k_rope<T, N><<<dim3(nblocks(vecs), n), TPB, 0, st>>>(ops<N>(qkv), ld, Ttok, divisor(S), divisor(nrot), d, divisor(d / 2 / Vec<T>::N), table,
                                                           table_seq);
}
hipError_t rope(int dtype, const Each& qkv, int ld, int n, int T, int S, int nrot, int d, const float* table, int table_seq,
                hipStream_t st) {
    if (dtype != DT_BF16 && n == 1) rope_t<float, 1>(qkv, ld, n, T, S, nrot, d, table, table_seq, st);
    else if (dtype != DT_BF16) rope_t<float, MICRO_MAX>(qkv, ld, n, T, S, nrot, d, table, table_seq, st);
    else if (n == 1) rope_t<bf16_t, 1>(qkv, ld, n, T, S, nrot, d, table, table_seq, st);
    else rope_t<bf16_t, MICRO_MAX>(qkv, ld, n, T, S, nrot, d, table, table_seq, st);
    return hipGetLastError();
}

template <typename T, int N>
static void swiglu_fwd_t(const Each& gu, const Each& m, int n, int Ttok, int F, hipStream_t st) {
    k_swiglu_fwd<T, N><<<dim3(nblocks((long)Ttok * (F / Vec<T>::N)), n), TPB, 0, st>>>(ops<N>(gu), ops<N>(m), Ttok, F, divisor(F / Vec<T>::N));
}
hipError_t swiglu_fwd(int dtype, const Each& gu, const Each& m, int n, int T, int F, hipStream_t st) {
    if (dtype != DT_BF16 && n == 1) swiglu_fwd_t<float, 1>(gu, m, n, T, F, st);
    else if (dtype != DT_BF16) swiglu_fwd_t<float, MICRO_MAX>(gu, m, n, T, F, st);
    else if (n == 1) swiglu_fwd_t<bf16_t, 1>(gu, m, n, T, F, st);
    else swiglu_fwd_t<bf16_t, MICRO_MAX>(gu, m, n, T, F, st);
    return hipGetLastError();
}

template <typename T, int N>
static void swiglu_bwd_t(const Each& dm, const Each& gu, const Each& dgu, const Each& m, int n, int Ttok, int F, hipStream_t st) {
    k_swiglu_bwd<T, N><<<dim3(nblocks((long)Ttok * (F / Vec<T>::N)), n), TPB, 0, st>>>(ops<N>(dm), ops<N>(gu), ops<N>(dgu), ops<N>(m), Ttok, F,
                                                                                         divisor(F / Vec<T>::N));
}
hipError_t swiglu_bwd(int dtype, const Each& dm, const Each& gu, const Each& dgu, const Each& m, int n, int T, int F, hipStream_t st) {
    if (dtype != DT_BF16 && n == 1) swiglu_bwd_t<float, 1>(dm, gu, dgu, m, n, T, F, st);
    else if (dtype != DT_BF16) swiglu_bwd_t<float, MICRO_MAX>(dm, gu, dgu, m, n, T, F, st);
    else if (n == 1) swiglu_bwd_t<bf16_t, 1>(dm, gu, dgu, m, n, T, F, st);
    else swiglu_bwd_t<bf16_t, MICRO_MAX>(dm, gu, dgu, m, n, T, F, st);
    return hipGetLastError();
}

}  // namespace hh
