// k_gemm_ring: bf16 GEMM for problems on which 256x256 tiles would leave most of the chip idle.
//
// One workgroup computes one BM x BN tile of C, or one share of its k range, through a ring of NS LDS stages of
// DK = 64 k values that are filled straight from global memory.  WM x WN waves, each a (BM/WM) x (BN/WN) block of
// 32x32x16 MFMAs.  One barrier per stage, placed before its last k step: by then every wave holds its last fragments
// of the stage, so its slot can be refilled (NS stages of lookahead) and the first fragments of the next stage are
// fetched in the shadow of the last MFMAs.
#pragma once
#include <type_traits>

#include "gemm_tile.h"
#include "kernels.h"

namespace hh {

// A launch takes a group of up to RING_MAX independent problems, each with its own operands, kind and k split: the
// weight gradients of a layer's backward pass beside the input gradient that uses the same operand, or projections
// whose weights are separate allocations.  Problem p owns the workgroups first .. first + tiles * ksplit - 1.
//
// Why groups: alone, each of these problems leaves most of the chip idle and costs a launch.  Measured: dWdown | dWgate |
// dWup | d(hn) of hidden 512, ffn 768 and 2200 tokens in five launches 52 us, in one 23 us; dWo | da of hidden 4096,
// width 1024 and 3300 tokens 101 -> 77 us; a 4-layer, 8 micro-batch stage of hidden 256 and 128 tokens 3.22 -> 2.88 ms.
//
// A problem may stand for the same product in `micro` micro-batches.  NT, NN and split TN ones then own that many times the
// workgroups; a workgroup of an unsplit TN problem walks the k loops of all of them, in order, and adds each product to the
// sum of those before it (`seq` of them), so that the gradient is read and written once; or each product has a workgroup of its
// own (seq 1) and the reduction adds them in that order.  Tile and split are those of a micro-batch by itself, so every result is
// what a launch per micro-batch gives, bit for bit.  Bound as before by one workgroup's chain and by launch latency, of which
// there are fewer: a 4-layer stage of hidden 256, 128 tokens and 8 micro-batches, two at a time, 2671 -> 1485 us; 2 layers of
// hidden 512, 2200 tokens, 3 micro-batches, 1092 -> 744 us (1172 and 665 to 707 by run, with what came after).
//
// Fused problems (GemmFuse): the workgroup's columns come in pair_column's order, so that an accumulator lane owns a column
// and its partner, 4q + e and 4(q + 2) + e of a block.  C is written back in its own order, in runs of 16 columns.  Bound by launch
// latency, of which two launches of nine forward and one of ten backward go: forward of hidden 1024, 700 tokens 67.6 -> 65.9 us,
// of hidden 512, 48 tokens 35.6 -> 34.1.
constexpr int RING_MAX = 4;
// rounded to bf16
__device__ __forceinline__ float as_bf(float v) { return lo_bf(pack_bf2(v, 0.f)); }
// A launch that fuses is an instantiation of its own (F): its arguments and code in the others cost each of them 0.5 us.
template <int MB, bool F>
struct RingFuse {};
template <int MB>
struct RingFuse<MB, true> {
    Ops<MB> X, Y;
    int fuse, period, shift, rot, table_seq;
    Divisor tokens;            // of a sample
    const float* table;
};
template <int MB, bool F>     // MB: how many micro-batches a launch may stand for, 1 or MICRO_MAX
struct RingProblem : RingFuse<MB, F> {
    Ops<MB> A, B, C, R;
    const bf16_t* Bseg[2];     // NN: where the rows of B from k tile kseg[0] (kseg[1]) on are; INT_MAX: no such segment
    float* partial;            // k shares: [tile][micro-batch][share][BM*BN] fp32 sums
    uint32_t a_bytes, b_bytes; // extent of A, and of B up to the first segment's end
    int kseg[2];
    int lda, ldb, ldc, ldr, M, N, K, accumulate, first, micro, seq, nk;   // nk: k tiles
    TileMap map;
    Divisor items, tiles, ksplit;   // workgroups of a micro-batch, of a share; shares
};
// NP: how many problems a launch may have, RING_MAX or 1 where MB is: what a launch costs the host grows with its arguments.
template <int MB, bool F, int NP>
struct RingGroup {
    RingProblem<MB, F> p[NP];
};

// A launch whose problems (NT, one A) norm the rows of A on the way in: A holds x, and the product is that of xn = x * r * gain.
template <int MB>
struct RingNorm {
    Ops<MB> xn, r;
    const bf16_t* gain;
    float eps;
    int writer;   // the problem whose first column of tiles writes xn and r
};

// v of the lane N before it of its 16, in a circle
template <int N>
__device__ __forceinline__ float rotated(float v) { return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x120 + N, 0xf, 0xf, true)); }

// NORM (K up to NORM_K): the tile's rows of x come into registers, are normed as k_rmsnorm_fwd norms them, to the same bits, and lie in
// LDS for all of k; only B goes through the ring.  Bound by latency: the launch before it (3.6 us with the gap behind it, of rows of 256)
// goes, and the workgroups get 1.2 to 1.9 us longer, for about 500 instructions between x and its place in LDS and because what waits for
// x and the gain, which the compiler counts, waits for the requests of B behind them too.
template <int KIND, int MB, bool F, int BM, int BN, int WM, int WN, int NS, bool NORM = false>
__device__ __forceinline__ void ring_body(const RingProblem<MB, F>& g, const RingNorm<MB>* norm = nullptr, bool writer = false) {
    if constexpr (NORM) asm volatile("" ::"s"(norm->gain), "s"(norm->eps), "s"(g.K), "s"(g.M), "s"(g.N));
    // what the first operand requests need, loaded at once
    asm volatile("" ::"s"(g.A.p[0]), "s"(g.B.p[0]), "s"(g.a_bytes), "s"(g.b_bytes), "s"(g.lda), "s"(g.ldb), "s"(g.first), "s"(g.nk),
                 "s"(g.map.tiles_m), "s"(g.map.tiles_n), "s"(g.map.width.d), "s"(g.map.width.mul), "s"(g.map.width.shift), "s"(g.map.last.d),
                 "s"(g.map.last.mul), "s"(g.map.last.shift), "s"(g.tiles.d), "s"(g.tiles.mul), "s"(g.tiles.shift), "s"(g.ksplit.mul), "s"(g.ksplit.shift));
    constexpr bool OUT_F32 = KIND == GEMM_TN;
    constexpr int NW = WM * WN;
    using DA = DmaTile<(KIND != GEMM_TN), BM, NW>;
    using DB = DmaTile<(KIND == GEMM_NT), BN, NW>;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr bool FUSES = F && KIND != GEMM_TN;
    constexpr int STAGE = (NORM ? 0 : DA::BYTES) + DB::BYTES;
    constexpr int PW = (NORM ? 0 : DA::PER_WAVE) + DB::PER_WAVE;       // DMA instructions per wave and stage
    static_assert(!NORM || (KIND == GEMM_NT && BM / NW % 4 == 0 && BM * BN == 64 * 64), "16 lanes a row, one MFMA a k step");
    static_assert(NS * STAGE >= NW * 4096, "the epilogue patches reuse the ring");
    extern __shared__ __attribute__((aligned(1024))) char smem[];   // [stage][A | B]
    const int M = g.M, N = g.N, K = g.K, lda = g.lda, ldb = g.ldb, ldc = g.ldc, ldr = g.ldr, ksplit = g.ksplit.d;
    bool accumulate = g.accumulate != 0;

    int micro = 0, share = (int)blockIdx.x - g.first, tix = share;
    if (MB > 1) { micro = share; tix = share = split_off(micro, g.items); }
    tix = split_off(share, g.tiles);
    const bf16_t* const R = (const bf16_t*)g.R.at(micro);
    void* const Cv = g.C.at(micro);
    constexpr bool SUMS = KIND == GEMM_TN && MB > 1;
    const int seq = SUMS ? g.seq : 1;   // products summed here
    const int tiles_n = g.map.tiles_n;
    int tm, tn;
    g.map.tile(tix, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const int nk_all = g.nk;
    const int kbeg = quotient(share * nk_all, g.ksplit), nk = quotient((share + 1) * nk_all, g.ksplit) - kbeg;
    const int nt = nk * seq;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, hf = lane >> 5;
    const int wm = (wave / WN) * (BM / WM), wn = (wave % WN) * (BN / WN);

    auto rsrc_a = [&](int m) {
        const uint64_t pa = (uint64_t)g.A.at(m);
        return i32x4{(int)(uint32_t)pa, (int)(uint32_t)(pa >> 32), (int)g.a_bytes, 0x00020000};
    };
    i32x4 rsA = rsrc_a(micro);
    const uint32_t stepA = DA::kstep_bytes(lda), stepB = DB::kstep_bytes(ldb);
    // B's rows may lie in up to three allocations.  Offsets run on over the segments: segment s is addressed from a base
    // moved back by the rows before it, and its last row ends its extent.
    auto rsrc_b = [&](int m, int kt) {
        uint64_t pb = (uint64_t)g.B.at(m);
        uint32_t bytes = g.b_bytes;
        if (KIND == GEMM_NN && kt >= g.kseg[0]) {
            const int s = kt >= g.kseg[1] ? 1 : 0;
            pb = (uint64_t)g.Bseg[s] - (uint64_t)(uint32_t)g.kseg[s] * stepB;
            const int end = s == 0 && g.kseg[1] < nk_all ? g.kseg[1] * DK : K;
            bytes = ((uint32_t)(end - 1) * (uint32_t)ldb + (uint32_t)N) * 2u;
        }
        return i32x4{(int)(uint32_t)pb, (int)(uint32_t)(pb >> 32), (int)bytes, 0x00020000};
    };
    i32x4 rsB = rsrc_b(micro, kbeg);
    uint32_t voA[DA::PER_WAVE], voB[DB::PER_WAVE];
#pragma unroll
    for (int i = 0; i < DA::PER_WAVE; i++) voA[i] = DA::voff(wave, i, m0, lda) + kbeg * stepA;
#pragma unroll
    for (int i = 0; i < DB::PER_WAVE; i++) {
        int row0 = n0;
        if constexpr (KIND == GEMM_NT && FUSES) {   // voff adds the lane's row of the tile
            const int r = DB::row(wave, i);
            row0 = pair_column(n0 + r, g.period, g.shift, N) - r;
        }
        voB[i] = DB::voff(wave, i, row0, ldb) + kbeg * stepB;
    }
    const int ring = NORM ? nk_all * DA::BYTES : 0;   // LDS: x's k tiles, then the ring
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem + ring);
    const int kseg0 = g.kseg[0], kseg1 = g.kseg[1];
    int kissue = kbeg, missue = micro;   // k tile and micro-batch that `issue` fetches next
    auto next_tile = [&]() {
        if (KIND == GEMM_NN && (kissue == kseg0 || kissue == kseg1)) rsB = rsrc_b(micro, kissue);
        if (SUMS && kissue == kbeg + nk) {   // the next micro-batch's product
            kissue = kbeg;
            missue++;
            rsA = rsrc_a(missue);
            rsB = rsrc_b(missue, kbeg);
#pragma unroll
            for (int i = 0; i < DA::PER_WAVE; i++) voA[i] -= (uint32_t)nk * stepA;
#pragma unroll
            for (int i = 0; i < DB::PER_WAVE; i++) voB[i] -= (uint32_t)nk * stepB;
        }
        kissue++;
    };
    // quarter Q of the DMA instructions that fetch a k tile (-1: all of them)
    auto issue_part = [&](int slot, auto quarter) {
        constexpr int Q = decltype(quarter)::value;
        const uint32_t base = lds0 + slot * STAGE;
#pragma unroll
        for (int i = 0; i < (NORM ? 0 : DA::PER_WAVE); i++)
            if (Q < 0 || i * 4 / PW == Q) { dma16(base + (wave * DA::PER_WAVE + i) * 1024, voA[i], rsA); voA[i] += stepA; }
#pragma unroll
        for (int i = 0; i < DB::PER_WAVE; i++)
            if (Q < 0 || (DA::PER_WAVE + i) * 4 / PW == Q) {
                dma16(base + (NORM ? 0 : DA::BYTES) + (wave * DB::PER_WAVE + i) * 1024, voB[i], rsB);
                voB[i] += stepB;
            }
    };
    auto issue = [&](int slot) {
        next_tile();
        issue_part(slot, std::integral_constant<int, -1>{});
    };
    // The memory pipe takes 16 cycles over a DMA instruction of 1 KB, and a wave whose instruction has to wait for it issues
    // no MFMA and no fragment read meanwhile.  So the requests that refill a slot come behind the next k tile's first fragment
    // reads and the MFMAs that need no others (64x64 tiles: behind the third of four): in front of them, 700x1024x1024 took 7.0 us
    // (NN) and 7.2 (NT with residual) where it takes 6.4 and 6.8, 333x4096x4096 NN 25.7 (24.6), 200x2048x2048 10.2 (9.7).
    // With two stages they stay in front: the tile is waited for at the end of the next k tile, and the reads they hold up are the
    // other workgroup's time to multiply (steps of hidden 4224, four layers of two micro-batches of 439 tokens: 7628 us behind, 7510 in
    // front; hidden 10816, two of 621 tokens, 9013 and 8863).
    // NT problems on the larger tiles spread the instructions that refill a slot over the four k steps
    // that follow its release, a quarter behind each step's MFMAs: 333x22016x4096 (192x192 tiles) 81 -> 72 us, 333x12288x4096
    // (192x128) 52 -> 50, 333x4096x4096 (128x128) 24.2 -> 23.1.  Not with two stages, where the tile would be waited for right
    // after its last quarter (3300x8192x4096, 192x256 tiles: 87 -> 106), not on the smallest tiles, whose loops are short
    // chains (nine launches of a 700-token forward pass 67.4 -> 69.3), and not beside the transposing fragment reads of NN
    // and TN (backward of hidden 448, 3348 tokens: 176 -> 182).
    constexpr bool SPREAD = KIND == GEMM_NT && NS > 2 && BM * BN >= 128 * 128;
    // NORM: lane `sub` of 16 has the 16-byte pieces sub, sub + 16, .. of four of the wave's rows
    constexpr int ROWS = NORM ? BM / NW / 4 : 1, PIECES = NORM ? NORM_K / 128 : 1;
    i32x4 row[ROWS][PIECES], gain[PIECES];
    float rstd[ROWS];
    const int sub = lane & 15, row0 = wave * (BM / NW) + (lane >> 4);
    if constexpr (NORM) {
        // past a row's or the gain's end: an offset that is out of range
        const __amdgpu_buffer_rsrc_t rsX = make_rsrc(g.A.at(micro), g.a_bytes), rsG = make_rsrc(norm->gain, (uint32_t)K * 2u);
#pragma unroll
        for (int p = 0; p < PIECES; p++) {
            const int col = 128 * p + 8 * sub;
#pragma unroll
            for (int q = 0; q < ROWS; q++)
                row[q][p] = __builtin_amdgcn_raw_buffer_load_b128(
                    rsX, col < K ? ((uint32_t)(m0 + row0 + 4 * q) * (uint32_t)lda + (uint32_t)col) * 2u : 0x80000000u, 0, 0);
            gain[p] = __builtin_amdgcn_raw_buffer_load_b128(rsG, (uint32_t)col * 2u, 0, 0);
        }
    }
#pragma unroll
    for (int s = 0; s < NS; s++)
        if (s < nt) issue(s);

    constexpr uint32_t CES = OUT_F32 ? 4u : 2u;
    constexpr uint32_t OUT_OF_RANGE = 0x80000000u;
    const __amdgpu_buffer_rsrc_t rsC = make_rsrc(Cv, (uint32_t)(((size_t)(M - 1) * ldc + N) * CES));
    const __amdgpu_buffer_rsrc_t rsR = make_rsrc(R ? (const void*)R : (const void*)Cv, R ? (uint32_t)(((size_t)(M - 1) * ldr + N) * 2u) : 0u);
    const int r_w = lane & 31;                       // row written, chunks 2g + hf
    const int r_r = lane >> 3, c_r = lane & 7;       // row (+ 8t) and chunk read back
    const int fuse = [&] { if constexpr (FUSES) return g.fuse; else return (int)FUSE_NONE; }();
    // NN: gate|up beside dm and dgate|dup; NT: silu(gate) * up
    const bool gates = FUSES && fuse > FUSE_ROPE;
    __amdgpu_buffer_rsrc_t rsX = rsC, rsY = rsC;
    if constexpr (FUSES) {
        const uint32_t row = (KIND == GEMM_NN ? 4u : 1u) * (uint32_t)N;   // bytes
        if (gates) rsX = make_rsrc(g.X.at(micro), (uint32_t)M * row);
        if (KIND == GEMM_NN) rsY = make_rsrc(g.Y.at(micro), (uint32_t)M * row);
    }
    // What the epilogue reads beside the product of block (i, j): the residual, the sum so far or gate|up, and the angles of the
    // rotary embedding.
    struct Beside { i32x2 res[KIND == GEMM_TN ? 1 : 4], up[KIND == GEMM_NN && FUSES ? 4 : 1]; i32x4 sum[OUT_F32 ? 4 : 1]; float4 cs[2], sn[2]; };
    auto ask = [&](int i, int j, Beside& s) {
        const int block = n0 + wn + 32 * j, col = block + 4 * c_r;
        if constexpr (KIND == GEMM_NT && FUSES) {
            if (fuse == FUSE_ROPE && block < g.rot) {
                int sample = m0 + wm + 32 * i + r_w;
                const int pos = split_off(sample, g.tokens), half = g.period / 2, base = pair_column(block, g.period, g.shift, N);
                const float* t = g.table + (size_t)pos * half + (base & (g.period - 1)) + 4 * hf;
#pragma unroll
                for (int q = 0; q < 2; q++) {
                    s.cs[q] = *reinterpret_cast<const float4*>(t + 8 * q);
                    s.sn[q] = *reinterpret_cast<const float4*>(t + 8 * q + (size_t)g.table_seq * half);
                }
            }
            return;
        }
#pragma unroll
        for (int t = 0; t < 4; t++) {
            const uint32_t row = (uint32_t)(m0 + wm + 32 * i + r_r + 8 * t);
            if constexpr (OUT_F32) {
                if (accumulate) s.sum[t] = __builtin_amdgcn_raw_buffer_load_b128(rsC, col < N ? (row * (uint32_t)ldc + (uint32_t)col) * CES : OUT_OF_RANGE, 0, 0);
            } else if constexpr (FUSES) {
                const uint32_t at = (row * (uint32_t)(2 * N) + (uint32_t)col) * 2u;
                s.res[t] = __builtin_amdgcn_raw_buffer_load_b64(rsX, col < N ? at : OUT_OF_RANGE, 0, 0);
                s.up[t] = __builtin_amdgcn_raw_buffer_load_b64(rsX, col < N ? at + (uint32_t)N * 2u : OUT_OF_RANGE, 0, 0);
            } else if (R) {
                s.res[t] = __builtin_amdgcn_raw_buffer_load_b64(rsR, col < N ? (row * (uint32_t)ldr + (uint32_t)col) * 2u : OUT_OF_RANGE, 0, 0);
            }
        }
    };
    if constexpr (NORM) {
        auto widen = [](const i32x4& v, float (&f)[8]) {
#pragma unroll
            for (int e = 0; e < 4; e++) { f[2 * e] = lo_bf((uint32_t)v[e]); f[2 * e + 1] = hi_bf((uint32_t)v[e]); }
        };
        float ss[ROWS];
#pragma unroll
        for (int q = 0; q < ROWS; q++) {
            float sum[PIECES];
#pragma unroll
            for (int p = 0; p < PIECES; p++) {
                float f[8];
                widen(row[q][p], f);
                sum[p] = 0.f;
#pragma unroll
                for (int e = 0; e < 8; e++) sum[p] += f[e] * f[e];
            }
            static_assert(PIECES == 2, "added up as a wave's lanes with a piece each do it");
            ss[q] = sum[0] + sum[1];
        }
#pragma unroll
        for (int q = 0; q < ROWS; q++) { ss[q] += rotated<8>(ss[q]); ss[q] += rotated<4>(ss[q]); ss[q] += rotated<2>(ss[q]); ss[q] += rotated<1>(ss[q]); }
        static_assert(ROWS == 4, "a lane of every four forms the factor of one of the four rows");
        const float mine = (sub & 2) ? ((sub & 1) ? ss[3] : ss[2]) : ((sub & 1) ? ss[1] : ss[0]);
        const int factor = __float_as_int(1.0f / sqrtf(mine / (float)K + norm->eps));
        rstd[0] = __int_as_float(__builtin_amdgcn_mov_dpp(factor, 0x00, 0xf, 0xf, true));   // lane 0 of its four, 1, 2, 3
        rstd[1] = __int_as_float(__builtin_amdgcn_mov_dpp(factor, 0x55, 0xf, 0xf, true));
        rstd[2] = __int_as_float(__builtin_amdgcn_mov_dpp(factor, 0xaa, 0xf, 0xf, true));
        rstd[3] = __int_as_float(__builtin_amdgcn_mov_dpp(factor, 0xff, 0xf, 0xf, true));
#pragma unroll
        for (int p = 0; p < PIECES; p++) {
            float gg[8];
            widen(gain[p], gg);
#pragma unroll
            for (int q = 0; q < ROWS; q++) {
                float f[8];
                widen(row[q][p], f);
#pragma unroll
                for (int e = 0; e < 8; e++) f[e] = f[e] * rstd[q] * gg[e];
                row[q][p] = i32x4{(int)pack_bf2(f[0], f[1]), (int)pack_bf2(f[2], f[3]), (int)pack_bf2(f[4], f[5]), (int)pack_bf2(f[6], f[7])};
            }
            if (128 * p + 8 * sub < K) {   // DmaTile's place of row r, piece sub % 8 of k tile 2p + sub / 8
#pragma unroll
                for (int q = 0; q < ROWS; q++) {
                    const int r = row0 + 4 * q;
                    *reinterpret_cast<i32x4*>(smem + (2 * p + (sub >> 3)) * DA::BYTES + r * 128 + (((sub & 7) ^ ((r >> 1) & 7)) << 4)) = row[q][p];
                }
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    // Asked for behind the requests of the first k tiles on the smaller tiles, whose epilogue would otherwise be a round trip to
    // memory: 128x768x256 with rotary embedding 4.2 -> 4.0 us, 700x1536x1024 10.6 -> 10.1, 128x256x256 with residual 3.33 -> 3.30.
    // Of three or four blocks a wave, 64 registers, it costs more than it gives (1100x3072x3072 with residual 27.4 -> 28.2), and
    // gate|up, two tiles as large as the product, hold up the k tiles behind them (700x2048x1024 12.2 -> 12.6).  The wait for k tile 0
    // leaves as many requests on their way as the later tiles have, so it covers as many of those as are asked for here.
    constexpr bool EARLY = TM * TN <= 2 && !(KIND == GEMM_NN && FUSES);
    Beside beside[EARLY ? TM : 1][EARLY ? TN : 1];
    if (EARLY && ksplit == 1 && !SUMS) {
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
            for (int j = 0; j < TN; j++) ask(i, j, beside[EARLY ? i : 0][EARLY ? j : 0]);
    }

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[i][j][r] = 0.f;

    // The sum of the products of the micro-batches before the one at work; a lane owns 4 consecutive columns of a row.
    constexpr int RM = SUMS ? TM : 1, RN = SUMS ? TN : 1;
    f32x16 sum[RM][RN];
    int left = nk;   // k tiles up to the end of the product at work
    bool first = true;
    if (SUMS && seq > 1 && accumulate) {
        const __amdgpu_buffer_rsrc_t rsC = make_rsrc(Cv, (uint32_t)(((size_t)(M - 1) * ldc + N) * 4u));
#pragma unroll
        for (int i = 0; i < RM; i++)
#pragma unroll
            for (int j = 0; j < RN; j++)
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const uint32_t row = (uint32_t)(m0 + wm + 32 * i + (lane & 31)), col = (uint32_t)(n0 + wn + 32 * j + 8 * q + 4 * hf);
                    const i32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsC, (int)col < N ? (row * (uint32_t)ldc + col) * 4u : 0x80000000u, 0, 0);
#pragma unroll
                    for (int e = 0; e < 4; e++) sum[i][j][4 * q + e] = __int_as_float(v[e]);
                }
        // the loads end here, as far as the compiler's wait counters go: the loop must not wait for them
#pragma unroll
        for (int i = 0; i < RM; i++)
#pragma unroll
            for (int j = 0; j < RN; j++) asm volatile("" : "+v"(sum[i][j]));
        first = false;
    }
    auto fold = [&]() {
        if (!SUMS || seq == 1 || --left) return;
        left = nk;
#pragma unroll
        for (int i = 0; i < RM; i++)
#pragma unroll
            for (int j = 0; j < RN; j++)
#pragma unroll
                for (int r = 0; r < 16; r++) {
                    sum[i][j][r] = first ? acc[i][j][r] : acc[i][j][r] + sum[i][j][r];
                    acc[i][j][r] = 0.f;
                }
        first = false;
    };

    // k tile 0 has landed
    if (nt >= NS) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * PW) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if constexpr (TM * TN == 1) {
        // One MFMA per k step: a whole k tile of fragments ahead, so that LDS latency is met once per stage and not once
        // per k step (128x256x1408 NN, eight tiles: 12.3 -> 9.0 us; 700x1024x1024 NT 7.5 -> 7.2).  With more MFMAs per k
        // step the loop is bound by its loads from L2 and the registers of a second k tile only cost (64x128 tiles 3 %
        // slower, 192x192 ones 20 %).
        bf16x8 fa[2][4][TM], fb[2][4][TN];
        auto fetch = [&](int set, int slot, int kt, int kk) {
            const char* cA = smem + (NORM ? kt * DA::BYTES : slot * STAGE);
            const char* cB = NORM ? smem + ring + slot * STAGE : cA + DA::BYTES;
#pragma unroll
            for (int i = 0; i < TM; i++) fa[set][kk][i] = DA::frag(cA, wm + 32 * i, kk);
#pragma unroll
            for (int j = 0; j < TN; j++) fb[set][kk][j] = DB::frag(cB, wn + 32 * j, kk);
        };
        int slot = 0;
        auto step = [&](auto parity, int kt) {
            constexpr int P = decltype(parity)::value, Q = P ^ 1;
            const int next = slot + 1 == NS ? 0 : slot + 1;
            // Every wave holds its fragments of k tile kt, so its slot is free once all waves are here; k tile kt + 1 must
            // have landed for everyone, the NS - 2 tiles after it may still be on their way.
            if (kt + NS <= nt) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NS - 2) * PW) : "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            const bool more = kt + 1 < nt;
            if (more) {
#pragma unroll
                for (int kk = 0; kk < 4; kk++) fetch(Q, next, kt + 1, kk);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kk = 0; kk < 4; kk++) {
                if (kk == 3 && kt + NS < nt) issue(slot);
#pragma unroll
                for (int i = 0; i < TM; i++)
#pragma unroll
                    for (int j = 0; j < TN; j++)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[P][kk][j], fa[P][kk][i], acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            fold();
            slot = next;
        };
#pragma unroll
        for (int kk = 0; kk < 4; kk++) fetch(0, 0, 0, kk);
        for (int kt = 0; kt < nt; kt += 2) {
            step(std::integral_constant<int, 0>{}, kt);
            if (kt + 1 < nt) step(std::integral_constant<int, 1>{}, kt + 1);
        }
    } else {
        bf16x8 fa[2][TM], fb[2][TN];
        auto fetch = [&](int set, int slot, int kk) {
            const char* cA = smem + slot * STAGE;
            const char* cB = cA + DA::BYTES;
#pragma unroll
            for (int i = 0; i < TM; i++) fa[set][i] = DA::frag(cA, wm + 32 * i, kk);
#pragma unroll
            for (int j = 0; j < TN; j++) fb[set][j] = DB::frag(cB, wn + 32 * j, kk);
        };
        auto mma = [&](int set) {
#pragma unroll
            for (int i = 0; i < TM; i++)
#pragma unroll
                for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[set][j], fa[set][i], acc[i][j], 0, 0, 0);
        };
        fetch(0, 0, 0);
        int slot = 0, freed = 0;
        bool refill = false;   // the slot freed last is still being refilled
        for (int kt = 0; kt < nt; kt++) {
            const int next = slot + 1 == NS ? 0 : slot + 1;
            auto step = [&](auto k) {
                constexpr int kk = decltype(k)::value;
                fetch((kk + 1) & 1, slot, kk + 1);
                mma(kk & 1);
                if (SPREAD && refill) issue_part(freed, std::integral_constant<int, kk + 1>{});
                __builtin_amdgcn_sched_barrier(0);
            };
            step(std::integral_constant<int, 0>{});
            step(std::integral_constant<int, 1>{});
            step(std::integral_constant<int, 2>{});
            // Every wave holds its last fragments of k tile kt, so its slot is free once all waves are here; k tile kt + 1
            // must have landed for everyone, the NS - 2 tiles after it may still be on their way.
            if (kt + NS <= nt) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NS - 2) * PW) : "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            refill = kt + NS < nt;
            if (refill) next_tile();
            if (NS == 2 && refill) issue_part(slot, std::integral_constant<int, -1>{});
            if (kt + 1 < nt) fetch(0, next, 0);
            __builtin_amdgcn_sched_barrier(0);
            mma(1);
            __builtin_amdgcn_sched_barrier(0);
            if (NS > 2 && !SPREAD && refill) issue_part(slot, std::integral_constant<int, -1>{});
            if (SPREAD && refill) issue_part(slot, std::integral_constant<int, 0>{});
            __builtin_amdgcn_sched_barrier(0);
            fold();
            freed = slot;
            slot = next;
        }
    }

    if constexpr (NORM) {
        if (writer && tn == 0) {
            bf16_t* const xn = (bf16_t*)norm->xn.at(micro);
            float* const rr = (float*)norm->r.at(micro);
#pragma unroll
            for (int q = 0; q < ROWS; q++) {
                const int r = m0 + row0 + 4 * q;
                if (r < M) {
                    if (sub == 0) rr[r] = rstd[q];
#pragma unroll
                    for (int p = 0; p < PIECES; p++)
                        if (128 * p + 8 * sub < K) *reinterpret_cast<i32x4*>(xn + (size_t)r * K + 128 * p + 8 * sub) = row[q][p];
                }
            }
        }
    }

    // a share of the k range, or one micro-batch's product of several: raw fp32 sums, finished by k_ring_reduce
    if (ksplit > 1 || (SUMS && seq == 1)) {
        float* pt = g.partial + (((size_t)(tm * tiles_n + tn) * (MB == 1 ? 1 : g.micro) + micro) * ksplit + share) * (BM * BN);
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
            for (int j = 0; j < TN; j++)
#pragma unroll
                for (int q = 0; q < 4; q++)
                    *reinterpret_cast<float4*>(pt + (wm + 32 * i + (lane & 31)) * BN + wn + 32 * j + 8 * q + 4 * hf) =
                        make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
        return;
    }

    if (SUMS && seq > 1) {
#pragma unroll
        for (int i = 0; i < RM; i++)
#pragma unroll
            for (int j = 0; j < RN; j++) acc[i][j] = sum[i][j];
        accumulate = false;   // what the buffer held is in the sum
    }

    // Epilogue as in k_gemm_dma: every 32x32 block goes through a wave-private LDS patch, so that loads of what is
    // added and stores cover whole row segments.
    __syncthreads();   // nobody reads the ring any more: each wave takes 4 KB of it as its patch
    char* const patch = smem + wave * 4096;
#pragma unroll
    for (int i = 0; i < TM; i++) {
#pragma unroll
        for (int j = 0; j < TN; j++) {
            const int block = n0 + wn + 32 * j;
            int col = block + 4 * c_r;
            Beside& b = beside[EARLY ? i : 0][EARLY ? j : 0];
            if (!EARLY) ask(i, j, b);
            if constexpr (KIND == GEMM_NT && FUSES) {
                const int half = g.period / 2, base = pair_column(block, g.period, g.shift, N);
                col = block >= N ? block : base + (c_r < 4 ? 4 * c_r : half + 4 * (c_r - 4));
                if (fuse == FUSE_SWIGLU || block < g.rot) {
#pragma unroll
                    for (int q = 0; q < 2; q++) {
                        float o[4];
                        const float c[4] = {b.cs[q].x, b.cs[q].y, b.cs[q].z, b.cs[q].w}, sv[4] = {b.sn[q].x, b.sn[q].y, b.sn[q].z, b.sn[q].w};
#pragma unroll
                        for (int e = 0; e < 4; e++) {
                            float u = as_bf(acc[i][j][4 * q + e]), v = as_bf(acc[i][j][4 * (q + 2) + e]);
                            if (fuse == FUSE_SWIGLU) {
                                o[e] = swiglu(u, v);
                            } else {
                                rotate_pair(u, v, c[e], sv[e]);
                                acc[i][j][4 * q + e] = u;
                                acc[i][j][4 * (q + 2) + e] = v;
                            }
                        }
                        if (fuse == FUSE_SWIGLU) {
                            const uint32_t row = (uint32_t)(m0 + wm + 32 * i + r_w);
                            const uint32_t off = block < N ? (row * (uint32_t)half + (uint32_t)(base + 8 * q + 4 * hf)) * 2u : OUT_OF_RANGE;
                            __builtin_amdgcn_raw_buffer_store_b64(i32x2{(int)pack_bf2(o[0], o[1]), (int)pack_bf2(o[2], o[3])}, rsX, off, 0, 0);
                        }
                    }
                }
            }
            float4 add[4];
            uint32_t off_c[4];
#pragma unroll
            for (int t = 0; t < 4; t++) {
                const uint32_t row = (uint32_t)(m0 + wm + 32 * i + r_r + 8 * t);
                off_c[t] = col < N ? (row * (uint32_t)ldc + (uint32_t)col) * CES : OUT_OF_RANGE;
                add[t] = make_float4(0.f, 0.f, 0.f, 0.f);
                if constexpr (OUT_F32) {
                    if (accumulate) add[t] = make_float4(__int_as_float(b.sum[t][0]), __int_as_float(b.sum[t][1]), __int_as_float(b.sum[t][2]), __int_as_float(b.sum[t][3]));
                } else if (!FUSES && R) {
                    add[t] = make_float4(lo_bf((uint32_t)b.res[t][0]), hi_bf((uint32_t)b.res[t][0]), lo_bf((uint32_t)b.res[t][1]), hi_bf((uint32_t)b.res[t][1]));
                }
            }
#pragma unroll
            for (int q = 0; q < 4; q++)
                *reinterpret_cast<float4*>(patch + r_w * 128 + (((2 * q + hf) ^ ((r_w >> 1) & 7)) << 4)) =
                    make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
#pragma unroll
            for (int t = 0; t < 4; t++) {
                const int rr = 8 * t + r_r;
                float4 v = *reinterpret_cast<const float4*>(patch + rr * 128 + ((c_r ^ ((rr >> 1) & 7)) << 4));
                v.x += add[t].x; v.y += add[t].y; v.z += add[t].z; v.w += add[t].w;
                if constexpr (KIND == GEMM_NN && FUSES) {   // v: dm
                    const uint32_t row = (uint32_t)(m0 + wm + 32 * i + r_r + 8 * t);
                    const uint32_t off_g = col < N ? (row * (uint32_t)(2 * N) + (uint32_t)col) * 2u : OUT_OF_RANGE;
                    const uint32_t off_u = col < N ? off_g + (uint32_t)N * 2u : OUT_OF_RANGE;
                    const float gt[4] = {lo_bf((uint32_t)b.res[t][0]), hi_bf((uint32_t)b.res[t][0]), lo_bf((uint32_t)b.res[t][1]), hi_bf((uint32_t)b.res[t][1])};
                    const float uu[4] = {lo_bf((uint32_t)b.up[t][0]), hi_bf((uint32_t)b.up[t][0]), lo_bf((uint32_t)b.up[t][1]), hi_bf((uint32_t)b.up[t][1])};
                    const float dm[4] = {v.x, v.y, v.z, v.w};
                    float dg[4], du[4], mm[4];
#pragma unroll
                    for (int e = 0; e < 4; e++) swiglu_grad(gt[e], uu[e], as_bf(dm[e]), dg[e], du[e], mm[e]);
                    __builtin_amdgcn_raw_buffer_store_b64(i32x2{(int)pack_bf2(dg[0], dg[1]), (int)pack_bf2(dg[2], dg[3])}, rsY, off_g, 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b64(i32x2{(int)pack_bf2(du[0], du[1]), (int)pack_bf2(du[2], du[3])}, rsY, off_u, 0, 0);
                    v = make_float4(mm[0], mm[1], mm[2], mm[3]);
                }
                if (OUT_F32) {
                    const i32x4 o = {__float_as_int(v.x), __float_as_int(v.y), __float_as_int(v.z), __float_as_int(v.w)};
                    __builtin_amdgcn_raw_buffer_store_b128(o, rsC, off_c[t], 0, 0);
                } else {
                    const i32x2 o = {(int)pack_bf2(v.x, v.y), (int)pack_bf2(v.z, v.w)};
                    __builtin_amdgcn_raw_buffer_store_b64(o, rsC, off_c[t], 0, 0);
                }
            }
        }
    }
}

// BWD: NN and TN problems (bit i of `tn`: problem i is TN), otherwise NT
template <bool BWD, int MB, bool F, int NP, int BM, int BN, int WM, int WN, int NS>
__global__ __launch_bounds__(WM * WN * 64, BM * BN / (WM * WN) > 64 * 128 ? 1 : 2) void k_gemm_ring(int second, int third, int fourth, int tn,
                                                                                                RingGroup<MB, F, NP> grp) {
    const int i = NP == 1 ? 0 : own_problem(Firsts{second, third, fourth});
    const RingProblem<MB, F>& g = grp.p[i];
    if (!BWD) ring_body<GEMM_NT, MB, F, BM, BN, WM, WN, NS>(g);
    else if (F || !(tn >> i & 1)) ring_body<GEMM_NN, MB, F, BM, BN, WM, WN, NS>(g);
    else ring_body<GEMM_TN, MB, F, BM, BN, WM, WN, NS>(g);
}

// NT problems that norm the rows of A, which they share
template <int MB, bool F, int NP, int BM, int BN, int WM, int WN, int NS>
__global__ __launch_bounds__(WM * WN * 64, 2) void k_gemm_ring_norm(int second, int third, int fourth, RingNorm<MB> norm, RingGroup<MB, F, NP> grp) {
    const int i = NP == 1 ? 0 : own_problem(Firsts{second, third, fourth});
    ring_body<GEMM_NT, MB, F, BM, BN, WM, WN, NS, true>(grp.p[i], &norm, i == norm.writer);
}

// Sums the ksplit fp32 shares of every BM x BN tile of the group's split problems in a fixed order and applies the
// epilogue.  A thread owns 4 consecutive columns of one row of C: of one micro-batch's (NT, NN), or of the gradient, to
// which it adds the micro-batches' products one after the other.
template <int MB, bool F, int NP>
struct RingReduce {
    struct Job : RingFuse<MB, F> {
        Ops<MB> C, R;
        const float* partial;
        int ksplit, ldc, ldr, M, N, accumulate, out_f32, micro, tiles_n, first;
        Divisor blocks, vectors;   // workgroups of one micro-batch; threads of a row
    } j[NP];
    Divisor bm, bn;
};
template <int MB, bool F, int NP>
__global__ __launch_bounds__(256) void k_ring_reduce(int second, int third, int fourth, RingReduce<MB, F, NP> grp) {
    const int i = NP == 1 ? 0 : own_problem(Firsts{second, third, fourth});
    const typename RingReduce<MB, F, NP>::Job& j = grp.j[i];
    const int fuse = [&] { if constexpr (F) return j.fuse; else return (int)FUSE_NONE; }();
    const bool pairs = fuse == FUSE_ROPE || fuse == FUSE_SWIGLU;   // 4 columns and their 4 partners, 16 further in the tiles
    const int bm = grp.bm.d, bn = grp.bn.d;
    const int micros = MB == 1 ? 1 : j.micro;
    int micro = 0, m = (int)blockIdx.x - j.first;
    if (MB > 1) { micro = m; m = split_off(micro, j.blocks); }
    m = m * 256 + (int)threadIdx.x;   // below 2^31: M rows of up to 65535 columns are checked to be under 2 GB
    const int v4 = split_off(m, j.vectors);
    if (m >= j.M) return;
    const int n = pairs ? (v4 >> 2) * 32 + (v4 & 3) * 4 : v4 * 4;
    int tm = m, tn = n;
    const int row = split_off(tm, grp.bm), col_in = split_off(tn, grp.bn);
    const float* p = j.partial + ((size_t)(tm * j.tiles_n + tn) * micros + micro) * j.ksplit * (bm * bn) + row * bn + col_in;
    auto shares = [&](float (&v)[4]) {   // the next ksplit shares
        for (int c = 0; c < j.ksplit; c++, p += bm * bn) {
            const float4 t = *reinterpret_cast<const float4*>(p);
            v[0] += t.x; v[1] += t.y; v[2] += t.z; v[3] += t.w;
        }
    };
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (j.out_f32) {
        float* c = reinterpret_cast<float*>(j.C.at(0)) + (size_t)m * j.ldc + n;
        float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
        if (j.accumulate) sum = *reinterpret_cast<const float4*>(c);
        for (int k = 0; k < micros; k++) {
            v[0] = v[1] = v[2] = v[3] = 0.f;
            shares(v);
            if (j.accumulate || k) { v[0] += sum.x; v[1] += sum.y; v[2] += sum.z; v[3] += sum.w; }
            sum = make_float4(v[0], v[1], v[2], v[3]);
        }
        *reinterpret_cast<float4*>(c) = sum;
    } else {
        if constexpr (F) if (pairs) {
            const float* const p0 = p;
            shares(v);
            p = p0 + 16;
            float u[4] = {0.f, 0.f, 0.f, 0.f};
            shares(u);
            const int half = j.period / 2, col = pair_column(n, j.period, j.shift, j.N);
#pragma unroll
            for (int e = 0; e < 4; e++) { v[e] = as_bf(v[e]); u[e] = as_bf(u[e]); }
            if (fuse == FUSE_SWIGLU) {
                uint2 o;
                o.x = pack_bf2(swiglu(v[0], u[0]), swiglu(v[1], u[1]));
                o.y = pack_bf2(swiglu(v[2], u[2]), swiglu(v[3], u[3]));
                *reinterpret_cast<uint2*>(reinterpret_cast<bf16_t*>(j.X.at(micro)) + (size_t)m * half + col) = o;
            } else if (n < j.rot) {
                int sample = m;
                const float* cs = j.table + (size_t)split_off(sample, j.tokens) * half + (col & (j.period - 1));
                const float* sn = cs + (size_t)j.table_seq * half;
#pragma unroll
                for (int e = 0; e < 4; e++) rotate_pair(v[e], u[e], cs[e], sn[e]);
            }
            bf16_t* const c = reinterpret_cast<bf16_t*>(j.C.at(micro)) + (size_t)m * j.ldc + col;
            *reinterpret_cast<uint2*>(c) = make_uint2(pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]));
            *reinterpret_cast<uint2*>(c + half) = make_uint2(pack_bf2(u[0], u[1]), pack_bf2(u[2], u[3]));
            return;
        }
        shares(v);
        if constexpr (F)
            if (fuse == FUSE_SWIGLU_BWD) {
                const bf16_t* gu = (const bf16_t*)j.X.at(micro) + (size_t)m * 2 * j.N + n;
                bf16_t* dgu = (bf16_t*)j.Y.at(micro) + (size_t)m * 2 * j.N + n;
                const uint2 gw = *reinterpret_cast<const uint2*>(gu), uw = *reinterpret_cast<const uint2*>(gu + j.N);
                const float gt[4] = {lo_bf(gw.x), hi_bf(gw.x), lo_bf(gw.y), hi_bf(gw.y)}, up[4] = {lo_bf(uw.x), hi_bf(uw.x), lo_bf(uw.y), hi_bf(uw.y)};
                float dg[4], du[4];
#pragma unroll
                for (int e = 0; e < 4; e++) swiglu_grad(gt[e], up[e], as_bf(v[e]), dg[e], du[e], v[e]);
                *reinterpret_cast<uint2*>(dgu) = make_uint2(pack_bf2(dg[0], dg[1]), pack_bf2(dg[2], dg[3]));
                *reinterpret_cast<uint2*>(dgu + j.N) = make_uint2(pack_bf2(du[0], du[1]), pack_bf2(du[2], du[3]));
            }
        const bf16_t* R = (const bf16_t*)j.R.at(micro);
        if (R) {
            const uint2 rr = *reinterpret_cast<const uint2*>(R + (size_t)m * j.ldr + n);
            v[0] += lo_bf(rr.x); v[1] += hi_bf(rr.x); v[2] += lo_bf(rr.y); v[3] += hi_bf(rr.y);
        }
        uint2 o;
        o.x = pack_bf2(v[0], v[1]);
        o.y = pack_bf2(v[2], v[3]);
        *reinterpret_cast<uint2*>(reinterpret_cast<bf16_t*>(j.C.at(micro)) + (size_t)m * j.ldc + n) = o;
    }
}

}  // namespace hh
