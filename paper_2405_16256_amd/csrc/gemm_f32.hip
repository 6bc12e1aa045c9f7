// fp32 GEMM of the fp32 path on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 operands, products and sums), any
// sizes that are multiples of 8 in N and in a contiguous K.
//
//   NT  C[M,N] = A[M,K] B[N,K]^T     NN  C[M,N] = A[M,K] B[K,N]     TN  C[M,N] = A[K,M]^T B[K,N]
//
// A workgroup of 4 waves computes a BM x BN tile; k advances FK = 32 at a time through a ring of NS LDS stages filled
// straight from global memory.  Tile 64x64: each wave a 32x32 block over the whole stage.  Tile 32x32: all four waves
// on the one block, each taking 8 of the stage's 32 k values, their sums added through LDS in wave order.
//
// What bounds it: one wave needs 16 MFMAs of 64 cycles per 32x32 block and stage, so the small problems of this path
// (a few dozen blocks, k up to a few thousand) are bound by how many waves share that chain: the 32x32 tile spreads a
// problem over 16 times the waves of a 64x64 one at twice the LDS traffic, and is taken until 64x64 tiles fill the
// chip.  Measured against the 64x64 FMA tile kernel with scalar loads before it, per call: 128x256x1376 NN 189 -> 12.7
// us, 700x1024x1536 NN 285 -> 27 us (82 TFLOP/s), 1024x2048x700 TN 98 -> 30 us, 2048x8192x1024 NT 536 -> 270 us (127).
// Rings of two stages on full launches, so that ten workgroups of 32x32 (five of 64x64) share a CU and their barriers and loads overlap:
// 700x1536x1024 NT 30.0 us with four stages, 27.7 with two; 2048x8192x1024 329 and 270; eight are slower still.
#include <algorithm>
#include <climits>
#include <utility>

#include "gemm_tile.h"
#include "kernels.h"

namespace hh {

constexpr int FK = 32;   // k values per stage

// One operand's tile of ROWS rows of C's dimension x FK values of k.
//   KC (k contiguous): LDS [row][k], 128 bytes a row, 16-byte chunks XOR-swizzled by the row index.
//   otherwise:         LDS [k][row], bit 7 of the byte address flipped for k rows with bit 2 set, so that the two half
//                      waves of a fragment read (k and k + 4) fall into different banks.
template <bool KC, int ROWS>
struct FTile {
    static constexpr int BYTES = ROWS * FK * 4;
    static constexpr int PER_WAVE = BYTES / 1024 / 4;
    static constexpr int PITCH = ROWS * 4;
    struct Src { uint32_t off; int k; };   // byte offset at k tile 0; first k value the lane fetches there
    __device__ static __forceinline__ Src src(int wave, int i, int row0, int ld) {
        const int idx = wave * PER_WAVE + i, L = threadIdx.x & 63;
        if (KC) {
            const int r = 8 * idx + (L >> 3), c = (L & 7) ^ ((r >> 1) & 7);
            return {((uint32_t)(row0 + r) * (uint32_t)ld + (uint32_t)(4 * c)) * 4u, 4 * c};
        }
        const int p = idx * 1024 + L * 16;
        const int lb = p ^ ((((p / PITCH) >> 2) & 1) << 7);
        const int k = lb / PITCH;
        return {((uint32_t)k * (uint32_t)ld + (uint32_t)row0) * 4u + (uint32_t)(lb % PITCH), k};
    }
    __device__ static __forceinline__ uint32_t kstep_bytes(int ld) { return KC ? FK * 4u : (uint32_t)FK * (uint32_t)ld * 4u; }
    // the lane's 4 values of k step kk (8 k values): row rb + lane%32, k = 8kk + 4(lane/32) + e
    __device__ static __forceinline__ f32x4 frag(const char* lds, int rb, int kk) {
        const int l = threadIdx.x & 63, r = rb + (l & 31), hf = l >> 5;
        if (KC) return *reinterpret_cast<const f32x4*>(lds + r * 128 + (((2 * kk + hf) ^ ((r >> 1) & 7)) << 4));
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const int k = 8 * kk + 4 * hf + e;
            v[e] = *reinterpret_cast<const float*>(lds + ((k * PITCH + r * 4) ^ (hf << 7)));   // (k >> 2) & 1 == hf
        }
        return v;
    }
};

// A launch takes a group of up to F32_MAX independent problems (weight gradients beside an input gradient, projections
// with separate weights), each owning the workgroups first .. first + tiles - 1: alone they are bound by their chain of
// k stages on a few dozen workgroups.  dWdown | dWgate|up | d(hn) of hidden 256, ffn 688 and 128 tokens in three launches
// 22.3 us, in one 15.5; of hidden 1024, ffn 2048 and 700 tokens 171 -> 137; dWo | da there 39.5 -> 32.
constexpr int F32_MAX = 4;
// F: the launch does what GemmFuse says on its way out (an instantiation of its own, as in gemm_ring.h).  A step of hidden 256,
// ffn 688 and 128 tokens is 19 launches of 3 to 16 us, three of which are spared: 95.6 -> 89.8 us; of hidden 1024, ffn 2048 and
// 700 tokens 507 -> 499.
template <bool F>
struct F32Fuse {};
template <>
struct F32Fuse<true> {
    GemmFuse fuse;
    int shift;
    Divisor tokens;   // of a sample
};
// MB: 1 or MICRO_MAX micro-batches, as in gemm_ring.h: NT and NN problems own that many times the workgroups, a workgroup of a TN
// one adds the products of all of them, in order, to the gradient it reads and writes once.
template <bool F, int MB>
struct F32Problem : F32Fuse<F> {
    Ops<MB> A, B, C, R, X, Y;
    uint32_t a_bytes, b_bytes;
    int kind, lda, ldb, ldc, ldr, M, N, K, accumulate, first, micro;
    TileMap map;
    Divisor tiles;   // of a micro-batch
};
template <bool F, int MB>
struct F32Group {
    int n;
    F32Problem<F, MB> p[F32_MAX];
};

template <int KIND, int BT, int NS, bool F, int MB>
__device__ __forceinline__ void f32_body(const F32Problem<F, MB>& g, int item) {   // item: workgroup of the problem
    constexpr bool A_KC = KIND != GEMM_TN, B_KC = KIND == GEMM_NT;
    using TA = FTile<A_KC, BT>;
    using TB = FTile<B_KC, BT>;
    constexpr int KG = BT == 32 ? 4 : 1;                  // waves that share a block along k
    constexpr int STAGE = TA::BYTES + TB::BYTES, PW = TA::PER_WAVE + TB::PER_WAVE;
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int M = g.M, N = g.N, K = g.K, lda = g.lda, ldb = g.ldb, ldc = g.ldc, ldr = g.ldr, accumulate = g.accumulate;
    const uint32_t a_bytes = g.a_bytes, b_bytes = g.b_bytes;
    int micro = 0;
    if (MB > 1) { micro = item; item = split_off(micro, g.tiles); }
    const int seq = KIND == GEMM_TN && MB > 1 ? g.micro : 1;   // products summed here
    const float* const R = (const float*)g.R.at(micro);
    float* const C = (float*)g.C.at(micro);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, hf = lane >> 5;
    int tm, tn;
    g.map.tile(item, tm, tn);
    const int m0 = tm * BT, n0 = tn * BT;
    const int wm = KG == 1 ? (wave >> 1) * 32 : 0, wn = KG == 1 ? (wave & 1) * 32 : 0;
    const int nk = (K + FK - 1) / FK;

    float4 sum[4 / KG];
    for (int mi = 0; mi < seq; mi++) {
        const uint64_t pa = (uint64_t)g.A.at(micro + mi), pb = (uint64_t)g.B.at(micro + mi);
        const i32x4 rsA = {(int)(uint32_t)pa, (int)(uint32_t)(pa >> 32), (int)a_bytes, 0x00020000};
        const i32x4 rsB = {(int)(uint32_t)pb, (int)(uint32_t)(pb >> 32), (int)b_bytes, 0x00020000};
        const uint32_t stepA = TA::kstep_bytes(lda), stepB = TB::kstep_bytes(ldb);
        typename TA::Src sa[TA::PER_WAVE];
        typename TB::Src sb[TB::PER_WAVE];
#pragma unroll
        for (int i = 0; i < TA::PER_WAVE; i++) sa[i] = TA::src(wave, i, m0, lda);
#pragma unroll
        for (int i = 0; i < TB::PER_WAVE; i++) {
            int row0 = n0;
            if constexpr (KIND == GEMM_NT && F) {   // src adds the lane's row of the tile
                const int r = 8 * (wave * TB::PER_WAVE + i) + (lane >> 3);
                row0 = pair_column(n0 + r, g.fuse.period, g.shift, N) - r;
            }
            sb[i] = TB::src(wave, i, row0, ldb);
        }
        const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem);
        auto issue = [&](int slot, int kt) {
            const uint32_t base = lds0 + slot * STAGE;
            // k values at or past K read as zero: they lie past the end of a k-strided operand by themselves, in a
            // k-contiguous one (4 values per lane, K a multiple of 8) the lane's offset is put out of range
            const int k0 = kt * FK;
#pragma unroll
            for (int i = 0; i < TA::PER_WAVE; i++) {
                const uint32_t off = sa[i].off + (uint32_t)kt * stepA;
                dma16(base + (wave * TA::PER_WAVE + i) * 1024, A_KC && k0 + sa[i].k >= K ? a_bytes : off, rsA);
            }
#pragma unroll
            for (int i = 0; i < TB::PER_WAVE; i++) {
                const uint32_t off = sb[i].off + (uint32_t)kt * stepB;
                dma16(base + TA::BYTES + (wave * TB::PER_WAVE + i) * 1024, B_KC && k0 + sb[i].k >= K ? b_bytes : off, rsB);
            }
        };
#pragma unroll
        for (int s = 0; s < NS - 1; s++)
            if (s < nk) issue(s, s);

        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; r++) acc[r] = 0.f;
        int slot = 0, fill = NS - 1;
        for (int kt = 0; kt < nk; kt++) {
            // k tile kt has landed, and everyone has read k tile kt - 1, whose slot is filled next
            if (nk - 1 - kt >= NS - 2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NS - 2) * PW) : "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (kt + NS - 1 < nk) issue(fill, kt + NS - 1);
            const char* cA = smem + slot * STAGE;
            const char* cB = cA + TA::BYTES;
#pragma unroll
            for (int q = 0; q < 4 / KG; q++) {
                const int kk = KG == 1 ? q : wave;
                const f32x4 fa = TA::frag(cA, wm, kk), fb = TB::frag(cB, wn, kk);
#pragma unroll
                for (int e = 0; e < 4; e++) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[e], fa[e], acc, 0, 0, 0);
            }
            slot = slot + 1 == NS ? 0 : slot + 1;
            fill = fill + 1 == NS ? 0 : fill + 1;
        }
        __syncthreads();   // nobody reads the ring any more
        // A lane owns row lane%32 of its block and runs of 4 columns 8g + 4hf; through an LDS patch of 4 KB per block the
        // stores cover 128-byte row segments.  With KG = 4 the patches of the waves that share a block are its partial sums.
        char* const patch = smem + wave * 4096;
        const int r_w = lane & 31;
#pragma unroll
        for (int g = 0; g < 4; g++)
            *reinterpret_cast<float4*>(patch + r_w * 128 + (((2 * g + hf) ^ ((r_w >> 1) & 7)) << 4)) =
                make_float4(acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]);
        if (KG > 1) __syncthreads();
        const int r_r = lane >> 3, c_r = lane & 7;
#pragma unroll
        for (int t = 0; t < 4 / KG; t++) {
            const int rr = 8 * (KG == 1 ? t : wave) + r_r;
            const int at = rr * 128 + ((c_r ^ ((rr >> 1) & 7)) << 4);
            float4 v = *reinterpret_cast<const float4*>((KG == 1 ? patch : smem) + at);
#pragma unroll
            for (int q = 1; q < KG; q++) {
                const float4 u = *reinterpret_cast<const float4*>(smem + q * 4096 + at);
                v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
            }
            const int m = m0 + wm + rr;
            int n = n0 + wn + 4 * c_r;
            if constexpr (KIND == GEMM_NT && F) {
                // the partners are 16 columns on, four lanes: lanes 0..3 of a row hold the first half's columns
                const float4 u = make_float4(__shfl_xor(v.x, 4, WAVE), __shfl_xor(v.y, 4, WAVE), __shfl_xor(v.z, 4, WAVE), __shfl_xor(v.w, 4, WAVE));
                if (m >= M || n >= N) continue;
                const bool second = c_r & 4;
                const int block = n0 + wn, half = g.fuse.period / 2, col = pair_column(block, g.fuse.period, g.shift, N) + 4 * (c_r & 3);
                float a[4] = {v.x, v.y, v.z, v.w}, b[4] = {u.x, u.y, u.z, u.w};
                if (g.fuse.kind == FUSE_SWIGLU) {
                    if (!second)
                        *reinterpret_cast<float4*>((float*)g.X.at(micro) + (size_t)m * half + col) =
                            make_float4(swiglu(a[0], b[0]), swiglu(a[1], b[1]), swiglu(a[2], b[2]), swiglu(a[3], b[3]));
                } else if (block < g.fuse.rot) {
                    int sample = m;
                    const float* cs = g.fuse.table + (size_t)split_off(sample, g.tokens) * half + (col & (g.fuse.period - 1));
                    const float4 c4 = *reinterpret_cast<const float4*>(cs), s4 = *reinterpret_cast<const float4*>(cs + (size_t)g.fuse.table_seq * half);
                    const float c[4] = {c4.x, c4.y, c4.z, c4.w}, sn[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        float x = second ? b[e] : a[e], y = second ? a[e] : b[e];
                        rotate_pair(x, y, c[e], sn[e]);
                        a[e] = second ? y : x;
                    }
                    v = make_float4(a[0], a[1], a[2], a[3]);
                }
                n = col + (second ? half : 0);
            }
            if (m >= M || n >= N) continue;
            if constexpr (KIND == GEMM_NN && F) {   // v: dm
                const float* gu = (const float*)g.X.at(micro) + (size_t)m * 2 * N + n;
                float* dgu = (float*)g.Y.at(micro) + (size_t)m * 2 * N + n;
                const float4 g4 = *reinterpret_cast<const float4*>(gu), u4 = *reinterpret_cast<const float4*>(gu + N);
                float4 dg, du, mm;
                swiglu_grad(g4.x, u4.x, v.x, dg.x, du.x, mm.x);
                swiglu_grad(g4.y, u4.y, v.y, dg.y, du.y, mm.y);
                swiglu_grad(g4.z, u4.z, v.z, dg.z, du.z, mm.z);
                swiglu_grad(g4.w, u4.w, v.w, dg.w, du.w, mm.w);
                *reinterpret_cast<float4*>(dgu) = dg;
                *reinterpret_cast<float4*>(dgu + N) = du;
                v = mm;
            }
            if (R) {
                const float4 u = *reinterpret_cast<const float4*>(R + (size_t)m * ldr + n);
                v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
            }
            float4* c = reinterpret_cast<float4*>(C + (size_t)m * ldc + n);
            if (accumulate || mi) {
                const float4 u = mi ? sum[t] : *c;
                v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
            }
            if (mi + 1 < seq) sum[t] = v;
            else *c = v;
        }
        if (mi + 1 < seq) __syncthreads();   // the patches become the ring again
    }
}

// BWD: NN and TN problems (bit i of `tn`: problem i is TN), otherwise NT
template <bool BWD, int BT, int NS, bool F, int MB>
__global__ __launch_bounds__(256) void k_gemm_f32(int second, int third, int fourth, int tn, F32Group<F, MB> grp) {
    const int i = own_problem(Firsts{second, third, fourth}), item = (int)blockIdx.x - grp.p[i].first;
    const F32Problem<F, MB>& g = grp.p[i];
    if (!BWD) f32_body<GEMM_NT, BT, NS, F, MB>(g, item);
    else if (F || !(tn >> i & 1)) f32_body<GEMM_NN, BT, NS, F, MB>(g, item);
    else f32_body<GEMM_TN, BT, NS, F, MB>(g, item);
}

template <bool BWD, int BT, int NS, bool F, int MB>
static hipError_t launch(F32Group<F, MB>& grp, hipStream_t st) {
    constexpr int LDS = NS * 2 * BT * FK * 4;
    static_assert(LDS >= 4 * 4096, "the epilogue patches reuse the ring");
    static_assert(LDS <= 48 * 1024, "no raised LDS limit");
    int first = 0, tn = 0, starts[F32_MAX];
    for (int i = 0; i < F32_MAX; i++) starts[i] = INT_MAX;
    for (int i = 0; i < grp.n; i++) {
        F32Problem<F, MB>& p = grp.p[i];
        p.map = tile_map(p.M, p.N, BT, BT);
        p.tiles = divisor(p.map.tiles());
        starts[i] = p.first = first;
        tn |= (p.kind == GEMM_TN) << i;
        first += p.map.tiles() * (p.kind == GEMM_TN ? 1 : p.micro);
    }
    k_gemm_f32<BWD, BT, NS, F, MB><<<first, 256, LDS, st>>>(starts[1], starts[2], starts[3], tn, grp);
    return hipGetLastError();
}

// 64x64 tiles (half the loads per product) once two of them per CU are kept busy to the end: their k stages, dealt to 512
// places, have to last a quarter longer than the longest tile.  700x4096x1024 NT, 704 tiles: 53.6 us against 55.3 with
// 32x32 tiles; 2048x8192x1024: 270 against 302; 700x1536x1024, 264 of them: 39.0 against 27.7; dWdown | dWgate|up | d(hn)
// of hidden 1024, 700 tokens, 1712 tiles of which 176 six times as long as the others: 149 against 137.
template <bool BWD, bool F, int MB>
static hipError_t pick(F32Group<F, MB>& grp, hipStream_t st) {
    long stages = 0, longest = 0, small = 0;
    for (int i = 0; i < grp.n; i++) {
        const F32Problem<F, MB>& p = grp.p[i];
        const long nk = (p.K + FK - 1) / FK;
        stages += (long)((p.M + 63) / 64) * ((p.N + 63) / 64) * nk;
        longest = std::max(longest, nk);
        small += (long)((p.M + 31) / 32) * ((p.N + 31) / 32);
    }
    // longest k loop first: the launch then ends with the short ones
    for (int i = 1; i < grp.n; i++)
        for (int j = i; j > 0 && grp.p[j].K > grp.p[j - 1].K; j--) std::swap(grp.p[j], grp.p[j - 1]);
    if (stages >= 640 * longest) return launch<BWD, 64, 2, F, MB>(grp, st);
    // Up to three 32x32 tiles per CU: six stages, because few workgroups hide little of the latency of operands that
    // another kernel has just written.  128x256x688 NT of a step of hidden 256
    // and 128 tokens: 11.3 us with two stages, 8.0 with six (704 tiles: alike).
    if (small <= 768) return launch<BWD, 32, 6, F, MB>(grp, st);
    return launch<BWD, 32, 2, F, MB>(grp, st);
}

template <bool F, int MB>
static hipError_t gemm_f32_f(const GemmDesc* d, int n, hipStream_t st) {
    F32Group<F, MB> grp{};
    grp.n = n;
    for (int i = 0; i < n; i++) {
        const GemmDesc& g = d[i];
        if (g.M <= 0 || g.N <= 0 || g.K <= 0 || g.k1 || (g.kind == GEMM_NT) != (d[0].kind == GEMM_NT)) return hipErrorInvalidValue;
        const long a_rows = (g.kind == GEMM_TN) ? g.K : g.M, a_cols = (g.kind == GEMM_TN) ? g.M : g.K;
        const long b_rows = (g.kind == GEMM_NT) ? g.N : g.K, b_cols = (g.kind == GEMM_NT) ? g.K : g.N;
        const long a_bytes = ((a_rows - 1) * g.lda + a_cols) * 4, b_bytes = ((b_rows - 1) * g.ldb + b_cols) * 4;
        // 32-bit byte offsets with room for a tile of rows, past the end
        if (a_bytes >= (1L << 32) - (1L << 25) || b_bytes >= (1L << 32) - (1L << 25)) return hipErrorInvalidValue;
        if (g.lda > 65535 || g.ldb > 65535 || g.N % 4 != 0) return hipErrorInvalidValue;
        if (g.kind != GEMM_TN && g.K % 4 != 0) return hipErrorInvalidValue;
        F32Problem<F, MB>& p = grp.p[i];
        if (g.micro < 1 || g.micro > MB || g.micro != d[0].micro || (MB > 1 && !g.each)) return hipErrorInvalidValue;
        for (int m = 0; m < MB; m++) {
            p.A.p[m] = MB == 1 ? const_cast<void*>(g.A) : g.each->A.p[m]; p.B.p[m] = MB == 1 ? const_cast<void*>(g.B) : g.each->B.p[m];
            p.C.p[m] = MB == 1 ? g.C : g.each->C.p[m]; p.R.p[m] = MB == 1 ? const_cast<void*>(g.R) : g.each->R.p[m];
            p.X.p[m] = MB == 1 ? g.fuse.X : g.each->X.p[m]; p.Y.p[m] = MB == 1 ? g.fuse.Y : g.each->Y.p[m];
        }
        p.micro = g.micro;
        p.a_bytes = (uint32_t)a_bytes; p.b_bytes = (uint32_t)b_bytes;
        p.kind = g.kind; p.lda = g.lda; p.ldb = g.ldb; p.ldc = g.ldc; p.ldr = g.ldr; p.M = g.M; p.N = g.N; p.K = g.K;
        p.accumulate = g.accumulate;
        if constexpr (F) {
            // whole heads, or a whole gate|up row of two whole 16-column pieces and more; a whole dm row; nothing is added
            const GemmFuse& f = g.fuse;
            if (g.R || g.accumulate || f.kind != d[0].fuse.kind) return hipErrorInvalidValue;
            if (f.kind == FUSE_ROPE && (g.kind != GEMM_NT || (f.period != 64 && f.period != 128) || g.N % f.period || f.rot % f.period ||
                                        !f.table || f.seq <= 0 || f.table_seq < f.seq)) return hipErrorInvalidValue;
            if (f.kind == FUSE_SWIGLU && (g.kind != GEMM_NT || f.period != g.N || g.N % 32 || !f.X)) return hipErrorInvalidValue;
            if (f.kind == FUSE_SWIGLU_BWD && (g.kind != GEMM_NN || n != 1 || !f.X || !f.Y)) return hipErrorInvalidValue;
            p.fuse = f;
            p.tokens = divisor(f.seq > 0 ? f.seq : 1);
            p.shift = f.kind == FUSE_ROPE ? (f.period == 128 ? 7 : 6) : 31;
        }
    }
    return d[0].kind == GEMM_NT ? pick<false, F, MB>(grp, st) : pick<true, F, MB>(grp, st);
}
hipError_t gemm_f32(const GemmDesc* d, int n, hipStream_t st) {
    if (n < 1 || n > F32_MAX) return hipErrorInvalidValue;
    if (d[0].micro > 1) return d[0].fuse.kind ? gemm_f32_f<true, MICRO_MAX>(d, n, st) : gemm_f32_f<false, MICRO_MAX>(d, n, st);
    return d[0].fuse.kind ? gemm_f32_f<true, 1>(d, n, st) : gemm_f32_f<false, 1>(d, n, st);
}

}  // namespace hh
