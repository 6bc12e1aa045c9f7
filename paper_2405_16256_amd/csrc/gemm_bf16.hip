// bf16 x bf16 -> fp32 GEMMs on the gfx950 matrix cores for the projections of the
// decoder layer and their input / weight gradients.
//
//   NT  C[M,N] = A[M,K] B[N,K]^T      forward  y  = x W^T
//   NN  C[M,N] = A[M,K] B[K,N]        backward dX = dY W
//   TN  C[M,N] = A[K,M]^T B[K,N]      backward dW = dY^T X   (fp32 output, optional +=)
//
// Two kernels, both on v_mfma_f32_32x32x16_bf16:
//   * k_gemm_dma: 256x256 tile of C per workgroup of 8 waves (2 per SIMD, each a 128x64
//     sub-tile), k advancing 64 at a time through two LDS stages that are filled straight
//     from global memory (buffer_load ... lds), so a k-contiguous operand row is fetched as
//     one whole 128-byte line per stage.  The loop is laid out by hand: MFMAs of one k step
//     interleaved with the LDS fragment reads of the next, one barrier per stage placed
//     before its last k step, after which the other stage's first fragments and the DMA of
//     the stage after that are issued.  TN problems have the same tile with another loop (k_gemm_dma_tn).
//   * k_gemm_ring (gemm_ring.h): tiles of 64x64 to 192x256 with rings of 2 to 4 stages, for
//     problems that 256x256 tiles would leave most of the chip idle on.
// plan() picks kernel, tile and k split, and whether problems share a launch, by a cost model fitted to measured times.
//
// Operand tiles in LDS keep the layout they have in memory, so global->LDS traffic is
// 16 bytes per lane with no transposition:
//   * k contiguous in memory  -> LDS [row][k], 16-byte chunks XOR-swizzled by the row
//     index; fragments come out with ds_read_b128.
//   * k strided in memory     -> LDS [k][rows], 64-byte slots XOR-swizzled by the k
//     index; fragments come out with the transposing ds_read_b64_tr_b16.
// Either way lane l of a fragment holds row (l % 32), k = 16*step + 8*(l/32) .. +7.
// Rows past the end of a tensor read as zero (buffer bounds), so ragged token counts
// need no special path.
//
// The MFMA takes the B-side fragment as its first operand, so each accumulator lane owns
// one row m of C and runs of 4 consecutive columns n: stores are 8-byte (bf16) or 16-byte
// (fp32) vectors along the contiguous dimension of C.
#include <algorithm>
#include <climits>
#include <cstdio>
#include <cstring>

#include "gemm_ring.h"
#include "gemm_tile.h"
#include "kernels.h"

namespace hh {

// ---------------------------------------------------------------------------
// Large-tile kernel: 256x256 tile of C, k advances 64 at a time through TWO LDS
// stages that are filled straight from global memory (buffer_load ... lds: no
// VGPR staging, no ds_write).  A k-contiguous operand row is 128 bytes per stage,
// i.e. one full cache line per request.
constexpr int DSTAGES = 2;
constexpr int DTILE = 256, DHALF = 128;
constexpr int DSTAGE_BYTES = DTILE * DK * 2;   // one operand, one stage: 32 KB
// Of the 8 DMA instructions a wave issues per stage, the last DMA_LATE wait until k step 0 of the next stage
// (their buffer is free from the barrier on and the data is not needed before the next barrier): spreading the
// requests measured 1.2 % faster on a whole layer than issuing all 8 during k step 3; more, or later, was slower.
constexpr int DMA_LATE = 3;

// A launch takes one problem or up to DMA_MAX of one kind and one k (the weight gradients of a layer): their tiles are
// numbered on, problem p from `first` on.
constexpr int DMA_MAX = 8;
struct DmaProblem {
    const bf16_t* A;
    const bf16_t* B;
    void* C;
    const bf16_t* R;
    uint32_t a_bytes, b_bytes;
    int lda, ldb, ldc, ldr, M, N, accumulate;
    TileMap map;
};
struct DmaGroup {
    int first[DMA_MAX];   // first tile of each problem, INT_MAX behind the last one
    int K;
    Divisor ksplit;       // k shares of a tile of the last round
    DmaProblem p[DMA_MAX];
    __device__ __forceinline__ int problem_of(int tile) const {
        int i = 0;
#pragma unroll
        for (int q = 1; q < DMA_MAX; q++) i += tile >= first[q];
        return i;
    }
};

// Instructions are fetched 32 bytes at a time, and where an 8-byte MFMA or the target of a branch lies in its 32 bytes decides whether
// the two waves of a SIMD are fed in time: the same k loop takes up to 2.4 % longer 16 bytes further on (NT 4096x8192x12288 by 4-byte
// steps from a 32-byte line: 627 627 630 622 636 628 629 623 us).  So the loops don't begin where the code before them happens to end
// but WORDS instructions behind such a line.  NT, NN and TN have a number each, the best of the eight for the loop as it stands or within
// 0.5 % of it, with a residual as without (NT with one 4096x8192x12288: 638 640 640 635 649 643 639 635); another compiler's may be others.
template <int WORDS>
__device__ __forceinline__ void place_loop() {
    asm volatile(".p2align 5\n\t.fill %0, 4, 0xbf800000" ::"n"(WORDS));   // s_nop
}

// NT or NN; RES: a problem has a residual, which is added to C.  A kernel of its own: what it holds costs the others registers.
template <int KIND, bool RES>
__global__ __launch_bounds__(512) void k_gemm_dma(DmaGroup grp, int full, int n_items, float* __restrict__ partial) {
    // The workgroup walks work items blockIdx.x, + gridDim.x, ... < n_items.  Items below `full` are whole tiles
    // (all of k, written out through the epilogue).  Item full + q is the (q % ksplit)-th share of the k range of
    // tile full + q / ksplit; its fp32 sums go to partial[q][256][256] and k_splitk_reduce finishes those tiles.
    // The first DMA stages of the next item are issued before the current one is written out.
    using DA = DmaTile<true, DTILE, 8>;
    using DB = DmaTile<(KIND == GEMM_NT), DTILE, 8>;
    constexpr int TM = 4, TN = 2;
    extern __shared__ __attribute__((aligned(1024))) char smem[];   // [stage][A 32 KB | B 32 KB]

    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, hf = lane >> 5;
    const int wm = (wave >> 2) * 128, wn = (wave & 3) * 64;
    const int nk_all = (grp.K + DK - 1) / DK;
    // work item -> problem, first row and column of its tile, first k tile, number of k tiles, slot in `partial` (-1: whole tile)
    int prob, m0, n0, kbeg, nk, slot;
    i32x4 rsA, rsB;
    uint32_t stepA, stepB;
    auto decode = [&](int item) {
        int tix;
        if (item < full) { tix = item; kbeg = 0; nk = nk_all; slot = -1; }
        else {
            int tile = slot = item - full;
            const int chunk = split_off(tile, grp.ksplit);
            tix = full + tile;
            kbeg = quotient(chunk * nk_all, grp.ksplit);
            nk = quotient((chunk + 1) * nk_all, grp.ksplit) - kbeg;
        }
        prob = grp.problem_of(tix);
        const DmaProblem& g = grp.p[prob];
        int tm, tn;
        g.map.tile(tix - grp.first[prob], tm, tn);
        m0 = tm * DTILE; n0 = tn * DTILE;
        const uint64_t pa = (uint64_t)g.A, pb = (uint64_t)g.B;
        rsA = i32x4{(int)(uint32_t)pa, (int)(uint32_t)(pa >> 32), (int)g.a_bytes, 0x00020000};
        rsB = i32x4{(int)(uint32_t)pb, (int)(uint32_t)(pb >> 32), (int)g.b_bytes, 0x00020000};
        stepA = DA::kstep_bytes(g.lda); stepB = DB::kstep_bytes(g.ldb);
    };
    int item = (int)blockIdx.x;
    decode(item);

    uint32_t voA[4], voB[4];
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;   // LDS byte address of the dynamic segment
    const uint32_t wave_lds = __builtin_amdgcn_readfirstlane(lds0 + wave * 4096);

    constexpr uint32_t OUT_OF_RANGE = 0x80000000u;

#define SB() __builtin_amdgcn_sched_barrier(0)
    // one DMA instruction of the k tile being issued (i < 4: A part i, else B part i-4) into stage st
    auto dma_part = [&](int st, int i) {
        const uint32_t base = wave_lds + st * (2 * DSTAGE_BYTES);
        if (i < 4) { dma16(base + i * 1024, voA[i], rsA); voA[i] += stepA; }
        else { dma16(base + DSTAGE_BYTES + (i - 4) * 1024, voB[i - 4], rsB); voB[i - 4] += stepB; }
    };
    // point the DMA offsets at the decoded tile and put its first two k tiles on their way
    auto start_tile = [&]() {
        const int lda = grp.p[prob].lda, ldb = grp.p[prob].ldb;
#pragma unroll
        for (int i = 0; i < 4; i++) { voA[i] = DA::voff(wave, i, m0, lda) + kbeg * stepA; voB[i] = DB::voff(wave, i, n0, ldb) + kbeg * stepB; }
#pragma unroll
        for (int s = 0; s < 2; s++)
            if (s < nk) {
#pragma unroll
                for (int i = 0; i < 8; i++) dma_part(s, i);
            }
    };

    start_tile();
    bool fresh = true;   // no stores of an earlier tile are in flight behind the DMAs

    for (;;) {
        f32x16 acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
            for (int j = 0; j < TN; j++)
#pragma unroll
                for (int r = 0; r < 16; r++) acc[i][j][r] = 0.f;

        // k tile 0 landed.  After an epilogue its stores sit behind the DMAs in the memory queue, so the
        // count-based wait only applies to a fresh start.
        if (fresh && nk > 1) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        bf16x8 a0[TM], b0[TN], a1[TM], b1[TN];
#pragma unroll
        for (int i = 0; i < TM; i++) a0[i] = DA::frag(smem, wm + 32 * i, 0);
#pragma unroll
        for (int j = 0; j < TN; j++) b0[j] = DB::frag(smem + DSTAGE_BYTES, wn + 32 * j, 0);

        place_loop<KIND == GEMM_NT ? 3 : 7>();
        for (int kt = 0; kt < nk; kt++) {
            const char* cA = smem + (kt & 1) * (2 * DSTAGE_BYTES);
            const char* cB = cA + DSTAGE_BYTES;
            const char* nA = smem + ((kt + 1) & 1) * (2 * DSTAGE_BYTES);
            const char* nB = nA + DSTAGE_BYTES;
            const bool more = kt + 2 < nk;
            const bool late = kt >= 1 && kt + 1 < nk;   // k tile kt+1's last DMA instructions are still to be issued
            SB();
            // k steps 0..2 of tile kt: MFMAs on one fragment set while the next one is fetched
#pragma unroll
            for (int kk = 0; kk < 3; kk++) {
                bf16x8 (&ca)[TM] = (kk & 1) ? a1 : a0;
                bf16x8 (&cb)[TN] = (kk & 1) ? b1 : b0;
                bf16x8 (&na)[TM] = (kk & 1) ? a0 : a1;
                bf16x8 (&nb)[TN] = (kk & 1) ? b0 : b1;
#pragma unroll
                for (int i = 0; i < TM; i++) {
#pragma unroll
                    for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cb[j], ca[i], acc[i][j], 0, 0, 0);
                    if (i == 0) { na[0] = DA::frag(cA, wm, kk + 1); nb[0] = DB::frag(cB, wn, kk + 1); nb[1] = DB::frag(cB, wn + 32, kk + 1); }
                    if (i == 1) { na[1] = DA::frag(cA, wm + 32, kk + 1); na[2] = DA::frag(cA, wm + 64, kk + 1); }
                    if (i == 2) { na[3] = DA::frag(cA, wm + 96, kk + 1); }
                    if (kk == 0 && i < DMA_LATE && late) dma_part((kt + 1) & 1, 8 - DMA_LATE + i);
                    SB();
                }
            }
            // Every wave now holds its last fragments of tile kt, so the stage of tile kt is free once all
            // waves are here; tile kt+1 (issued one tile ago) must have landed for everyone.
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            SB();
            // k step 3: MFMAs on (a1, b1); meanwhile fetch the first fragments of tile kt+1 and issue most of tile kt+2
#pragma unroll
            for (int i = 0; i < TM; i++) {
#pragma unroll
                for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b1[j], a1[i], acc[i][j], 0, 0, 0);
                if (i == 0) { a0[0] = DA::frag(nA, wm, 0); b0[0] = DB::frag(nB, wn, 0); b0[1] = DB::frag(nB, wn + 32, 0); }
                if (i == 1) { a0[1] = DA::frag(nA, wm + 32, 0); a0[2] = DA::frag(nA, wm + 64, 0); }
                if (i == 2) { a0[3] = DA::frag(nA, wm + 96, 0); }
                if (more) {
#pragma unroll
                    for (int q = 0; q < 8 - DMA_LATE; q++)
                        if (q * 4 / (8 - DMA_LATE) == i) dma_part(kt & 1, q);
                }
                SB();
            }
        }

        // next piece of work of this workgroup: start its loads before writing this one out
        const int cm0 = m0, cn0 = n0, cslot = slot, cprob = prob;
        item += (int)gridDim.x;
        const bool has_next = item < n_items;
        const bf16_t* const R = RES && cslot < 0 ? grp.p[cprob].R : nullptr;
        if (has_next) {
            decode(item);
            __syncthreads();   // every wave has finished reading the LDS stages
            if (!RES || !R) start_tile();
            fresh = false;
        }

        if (cslot >= 0) {   // a share of the k range: raw fp32 sums, finished by the reduction kernel
            float* pt = partial + (size_t)cslot * (DTILE * DTILE);
#pragma unroll
            for (int i = 0; i < TM; i++)
#pragma unroll
                for (int j = 0; j < TN; j++)
#pragma unroll
                    for (int g = 0; g < 4; g++)
                        *reinterpret_cast<float4*>(pt + (wm + 32 * i + (lane & 31)) * DTILE + wn + 32 * j + 8 * g + 4 * hf) =
                            make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
            if (!has_next) return;
            continue;
        }

        // Epilogue.  In the accumulators a lane owns one row and 4-column pieces of it, which would make every
        // store instruction touch 32 rows with 16 bytes each.  Each 32x32 block therefore goes through a
        // wave-private 4 KB LDS patch (fp32, 16-byte chunks XOR-swizzled by the row) and comes back with 8
        // lanes per row: loads of the residual and stores then cover whole 64-byte row segments.  C and R are reached
        // through bounds-checked buffers: rows past M fall behind the buffer's end, columns past N get an
        // out-of-range offset.
        // The residual is asked for AHEAD blocks ahead, STEP at a time, and ahead of the next tile's DMA, which it would wait behind:
        // block row by block row behind the DMA it was four round trips (NT 4096x16384xK: K 1024 187 -> 162 us, 4096 507 -> 485; NN
        // 8192x8192x512 105 -> 98).  NN, whose fragment reads keep more addresses, has registers for three: with four, ten
        // of them went to scratch memory, and NN 8192x8192x512 took 103.
        {
            const DmaProblem& g = grp.p[cprob];
            const int M = g.M, N = g.N, ldc = g.ldc, ldr = g.ldr;
            const __amdgpu_buffer_rsrc_t rsC = make_rsrc(g.C, (uint32_t)(((size_t)(M - 1) * ldc + N) * 2u));
            const __amdgpu_buffer_rsrc_t rsR = make_rsrc(R ? (const void*)R : g.C, R ? (uint32_t)(((size_t)(M - 1) * ldr + N) * 2u) : 0u);
            char* const patch = smem + DSTAGES * 2 * DSTAGE_BYTES + wave * 4096;
            const int r_w = lane & 31;                       // row written, chunks 2g + hf
            const int r_r = lane >> 3, c_r = lane & 7;       // row (+ 8t) and chunk read back
            const uint32_t row0 = (uint32_t)(cm0 + wm + r_r);
            constexpr int AHEAD = KIND == GEMM_NT ? 2 * TN : 3, STEP = KIND == GEMM_NT ? TN : 1;
            i32x2 res[AHEAD][4];
            auto ask = [&](int from, int to) {   // blocks, row by row
#pragma unroll
                for (int b = from; b < to; b++) {
                    const int col = cn0 + wn + 32 * (b % TN) + 4 * c_r;
#pragma unroll
                    for (int t = 0; t < 4; t++)
                        res[b % AHEAD][t] = __builtin_amdgcn_raw_buffer_load_b64(
                            rsR, col < N ? ((row0 + 32 * (b / TN) + 8 * t) * (uint32_t)ldr + (uint32_t)col) * 2u : OUT_OF_RANGE, 0, 0);
                }
            };
            if (RES && R) ask(0, AHEAD);
#pragma unroll
            for (int i = 0; i < TM; i++) {
#pragma unroll
                for (int j = 0; j < TN; j++) {
                    const int col = cn0 + wn + 32 * j + 4 * c_r;
#pragma unroll
                    for (int q = 0; q < 4; q++)
                        *reinterpret_cast<float4*>(patch + r_w * 128 + (((2 * q + hf) ^ ((r_w >> 1) & 7)) << 4)) =
                            make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
#pragma unroll
                    for (int t = 0; t < 4; t++) {
                        const int rr = 8 * t + r_r;
                        float4 v = *reinterpret_cast<const float4*>(patch + rr * 128 + ((c_r ^ ((rr >> 1) & 7)) << 4));
                        if (RES && R) {
                            const i32x2 u = res[(TN * i + j) % AHEAD][t];
                            v.x += lo_bf((uint32_t)u[0]); v.y += hi_bf((uint32_t)u[0]); v.z += lo_bf((uint32_t)u[1]); v.w += hi_bf((uint32_t)u[1]);
                        }
                        const i32x2 o = {(int)pack_bf2(v.x, v.y), (int)pack_bf2(v.z, v.w)};
                        __builtin_amdgcn_raw_buffer_store_b64(
                            o, rsC, col < N ? ((row0 + 32 * i + 8 * t) * (uint32_t)ldc + (uint32_t)col) * 2u : OUT_OF_RANGE, 0, 0);
                    }
                    const int asked = TN * i + j + 1 + AHEAD;   // up to here when this block's step is done
                    if (RES && R && (j + 1) % STEP == 0 && asked <= TM * TN) {
                        ask(asked - STEP, asked);
                        if (asked == TM * TN && has_next) start_tile();
                    }
                }
            }
        }
        if (!has_next) return;
    }
#undef SB
}

// The same for TN problems (fp32 C, optional +=), with another k loop.  The tile is worked off as 2x2 quadrants of 128x128, of which
// a wave has 64x32 each, one quadrant after the other over all k of a stage, so that each half of an operand's tile is read in one go
// and its place refilled from then on: a request is on its way for 1.25 to 1.5 stages where k_gemm_dma leaves it 0.5 to 1, for a
// second barrier per stage.  Half the fragments of both operands stay in registers (96).  4096x16384xK, four rounds of tiles,
// k_gemm_dma's loop -> this one, the halves written in order: K 2048 315 -> 296 us, 4096 502 -> 479, 8192 908 -> 897; 57344x8192x4096
// 3508 -> 3456.  NT and NN gain 1 to 2.5 % where the loop is long and the chip full, and lose as much or more elsewhere (NN
// 3300x4096x8192, 208 tiles, 175 -> 183): they are at the power limit or bound by barriers.  Four waves of 128x128 (a third fewer LDS
// reads) take the same.
// Every workgroup writes its tile's halves of 128 rows one after the other, all at about the same time, and where a row of C is a power
// of two bytes, rows 64 apart lie in the same memory channels.  So in every other row of tiles A's halves change places.  += with K 17,
// k_gemm_dma's loop -> halves in order -> in turn: 16384x2048 51 -> 61 -> 44 us, 8192x4096 67 -> 58 -> 49, 12288x4096 71 -> 75 -> 64;
// 16384x2112 48 -> 49 -> 49.  K 700 6144x16384 253 -> 246 -> 229.  What the longer prologue costs shows where the sums are short
// and there is one round of tiles: 4096x4096 by 64 14.6 -> 15.2, by 512 24.4 -> 25.1.
__global__ __launch_bounds__(512) void k_gemm_dma_tn(DmaGroup grp, int full, int n_items, float* __restrict__ partial) {
    using DT = DmaTile<false, DHALF, 8>;
    constexpr int TM = 4, TN = 2, PW = DT::PER_WAVE, HALF_BYTES = DT::BYTES;   // 2 instructions a wave, 16 KB
    constexpr int B_LDS = DSTAGES * DSTAGE_BYTES;
    extern __shared__ __attribute__((aligned(1024))) char smem[];   // A [stage][half] | B [stage][half] | patches

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = (wave >> 2) * 64, wn = (wave & 3) * 32;          // in each half
    const int nk_all = (grp.K + DK - 1) / DK;
    int prob, m0, n0, kbeg, nk, slot;                               // of a work item, as in k_gemm_dma
    int turn;                                                       // A's halves change places
    auto decode = [&](int item) {
        int tix;
        if (item < full) { tix = item; kbeg = 0; nk = nk_all; slot = -1; }
        else {
            int tile = slot = item - full;
            const int chunk = split_off(tile, grp.ksplit);
            tix = full + tile;
            kbeg = quotient(chunk * nk_all, grp.ksplit);
            nk = quotient((chunk + 1) * nk_all, grp.ksplit) - kbeg;
        }
        prob = grp.problem_of(tix);
        int tm, tn;
        grp.p[prob].map.tile(tix - grp.first[prob], tm, tn);
        m0 = tm * DTILE; n0 = tn * DTILE; turn = tm & 1;
    };
    int item = (int)blockIdx.x;
    decode(item);

    constexpr uint32_t OUT_OF_RANGE = 0x80000000u;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem) + wave * (PW * 1024);
    // A half's buffer begins at its first byte of the k tile asked for next, so that a lane's offset is the same in every k tile.
    struct Half { uint64_t at; int left; };   // left: elements up to the operand's end
    Half hA[2], hB[2];
    uint32_t voA[PW], voB[PW], stepA, stepB;
    // instruction p of a half; the last one moves on to the next k tile
    auto dma_half = [&](Half& h, const uint32_t (&vo)[PW], uint32_t step, int lds, int p) {
        const i32x4 rs = {(int)(uint32_t)h.at, (int)(uint32_t)(h.at >> 32), max(h.left, 0) << 1, 0x00020000};
        dma16(lds0 + lds + p * 1024, vo[p], rs);
        if (p == PW - 1) {
            h.at += step;
            h.left -= (int)(step >> 1);
        }
    };
    auto dma_a = [&](int st, int half, int p) { dma_half(hA[half], voA, stepA, st * DSTAGE_BYTES + half * HALF_BYTES, p); };
    auto dma_b = [&](int st, int half, int p) { dma_half(hB[half], voB, stepB, B_LDS + st * DSTAGE_BYTES + half * HALF_BYTES, p); };
    // point the DMA at the decoded tile and put its first two k tiles on their way
    auto start_tile = [&]() {
        const DmaProblem& g = grp.p[prob];
        stepA = DT::kstep_bytes(g.lda); stepB = DT::kstep_bytes(g.ldb);
#pragma unroll
        for (int i = 0; i < PW; i++) { voA[i] = DT::voff(wave, i, 0, g.lda); voB[i] = DT::voff(wave, i, 0, g.ldb); }
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const uint32_t skip_a = (uint32_t)(m0 + (h ^ turn) * DHALF) * 2u + (uint32_t)kbeg * stepA;
            const uint32_t skip_b = (uint32_t)(n0 + h * DHALF) * 2u + (uint32_t)kbeg * stepB;
            hA[h] = Half{(uint64_t)g.A + skip_a, (int)(g.a_bytes >> 1) - (int)(skip_a >> 1)};
            hB[h] = Half{(uint64_t)g.B + skip_b, (int)(g.b_bytes >> 1) - (int)(skip_b >> 1)};
        }
#pragma unroll
        for (int s = 0; s < 2; s++)
            if (s < nk) {
#pragma unroll
                for (int p = 0; p < PW; p++) dma_a(s, 0, p);
#pragma unroll
                for (int p = 0; p < PW; p++) dma_b(s, 0, p);
#pragma unroll
                for (int p = 0; p < PW; p++) dma_b(s, 1, p);
#pragma unroll
                for (int p = 0; p < PW; p++) dma_a(s, 1, p);
            }
    };
#define SB() __builtin_amdgcn_sched_barrier(0)
    auto sync = [&]() {
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        SB();
    };
    start_tile();
    bool fresh = true;   // no stores of an earlier tile are in flight behind the DMAs

    for (;;) {
        f32x16 acc[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
            for (int j = 0; j < TN; j++)
#pragma unroll
                for (int r = 0; r < 16; r++) acc[i][j][r] = 0.f;

        // k tile 0 has landed, as in k_gemm_dma
        if (fresh && nk > 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * PW) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        sync();
        bf16x8 a[2][2][4], b[2][4];   // A: half, row block, k step; B: register set, k step
        // fragment f of a half, in the order in which the MFMAs take them
        auto read_a = [&](int st, int half, int f) {
            a[half][f & 1][f >> 1] = DT::frag(smem + st * DSTAGE_BYTES + half * HALF_BYTES, wm + 32 * (f & 1), f >> 1);
        };
        auto read_b = [&](int set, int st, int half, int f) { b[set][f] = DT::frag(smem + B_LDS + st * DSTAGE_BYTES + half * HALF_BYTES, wn, f); };
#pragma unroll
        for (int f = 0; f < 8; f++) read_a(0, 0, f);
#pragma unroll
        for (int f = 0; f < 4; f++) read_b(0, 0, 0, f);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        sync();

        // The 8 MFMAs of quadrant (ha, hb), B from register set `set`; meanwhile the fragments of a half that is needed later are read
        // and the two DMA instructions of one whose place is free are issued.
        auto quadrant = [&](int ha, int hb, int set, auto read, int n_reads, auto dma, bool more) {
#pragma unroll
            for (int q = 0; q < 8; q++) {
                f32x16& c = acc[2 * ha + (q & 1)][hb];
                c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[set][q >> 1], a[ha][q & 1][q >> 1], c, 0, 0, 0);
#pragma unroll
                for (int f = 0; f < 8; f++)
                    if (f < n_reads && f * 4 / n_reads == q) read(f);
#pragma unroll
                for (int p = 0; p < PW; p++)
                    if (q == 4 * p + 2 && more) dma(p);
                SB();
            }
        };
        // Stage S of k tile kt: the fragments of A half 0 and B half 0 (in register set S) are there, those of B half 1 and A half 1
        // are read in the first two quadrants, the next k tile's A half 0 and B half 0 in the last two.  The waits leave the DMA
        // instructions behind the halves that are read next on their way.
        auto stage = [&](auto parity, int kt) {
            constexpr int S = decltype(parity)::value, O = S ^ 1;
            const bool more = kt + 2 < nk;
            quadrant(0, 0, S, [&](int f) { read_b(O, S, 1, f); }, 4, [&](int p) { dma_a(S, 0, p); }, more);
            quadrant(0, 1, O, [&](int f) { read_a(S, 1, f); }, 8, [&](int p) { dma_b(S, 0, p); }, more);
            if (more) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(4 * PW) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(2 * PW) : "memory");
            sync();
            quadrant(1, 1, O, [&](int f) { read_a(O, 0, f); }, 8, [&](int p) { dma_b(S, 1, p); }, more);
            quadrant(1, 0, S, [&](int f) { read_b(O, O, 0, f); }, 4, [&](int p) { dma_a(S, 1, p); }, more);
            if (more) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(4 * PW) : "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            sync();
        };
        place_loop<4>();
        for (int kt = 0; kt < nk; kt += 2) {
            stage(std::integral_constant<int, 0>{}, kt);
            if (kt + 1 < nk) stage(std::integral_constant<int, 1>{}, kt + 1);
        }

        // next piece of work of this workgroup: start its loads before writing this one out (the stages have been read)
        const int cm0 = m0, cn0 = n0, cslot = slot, cprob = prob, cturn = turn;
        item += (int)gridDim.x;
        const bool has_next = item < n_items;
        if (has_next) {
            decode(item);
            start_tile();
            fresh = false;
        }
        // formed here, out of the compiler's sight: it would keep what it derives from them through the k loop
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        const int hf = lane >> 5, r_w = lane & 31;
        auto block_row = [&](int i) { return DHALF * ((i >> 1) ^ cturn) + wm + 32 * (i & 1); };
        if (cslot >= 0) {   // a share of the k range
            float* pt = partial + (size_t)cslot * (DTILE * DTILE);
#pragma unroll
            for (int i = 0; i < TM; i++)
#pragma unroll
                for (int j = 0; j < TN; j++)
#pragma unroll
                    for (int q = 0; q < 4; q++)
                        *reinterpret_cast<float4*>(pt + (block_row(i) + r_w) * DTILE + DHALF * j + wn + 8 * q + 4 * hf) =
                            make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
            if (!has_next) return;
            continue;
        }
        // epilogue as in k_gemm_dma
        const DmaProblem& g = grp.p[cprob];
        const int M = g.M, N = g.N, ldc = g.ldc;
        const bool cacc = g.accumulate != 0;
        const __amdgpu_buffer_rsrc_t rsC = make_rsrc(g.C, (uint32_t)(((size_t)(M - 1) * ldc + N) * 4u));
        char* const patch = smem + DSTAGES * 2 * DSTAGE_BYTES + wave * 4096;
        const int r_r = lane >> 3, c_r = lane & 7;
#pragma unroll
        for (int i = 0; i < TM; i++) {
            const uint32_t row_base = (uint32_t)(cm0 + block_row(i) + r_r);
            float4 add[TN][4];
            uint32_t off_c[TN][4];
#pragma unroll
            for (int j = 0; j < TN; j++) {
                const int col = cn0 + DHALF * j + wn + 4 * c_r;
#pragma unroll
                for (int t = 0; t < 4; t++) {
                    off_c[j][t] = col < N ? ((row_base + 8 * t) * (uint32_t)ldc + (uint32_t)col) * 4u : OUT_OF_RANGE;
                    add[j][t] = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (cacc) {
                        const i32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsC, off_c[j][t], 0, 0);
                        add[j][t] = make_float4(__int_as_float(v[0]), __int_as_float(v[1]), __int_as_float(v[2]), __int_as_float(v[3]));
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < TN; j++) {
#pragma unroll
                for (int q = 0; q < 4; q++)
                    *reinterpret_cast<float4*>(patch + r_w * 128 + (((2 * q + hf) ^ ((r_w >> 1) & 7)) << 4)) =
                        make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
#pragma unroll
                for (int t = 0; t < 4; t++) {
                    const int rr = 8 * t + r_r;
                    const float4 v = *reinterpret_cast<const float4*>(patch + rr * 128 + ((c_r ^ ((rr >> 1) & 7)) << 4));
                    const i32x4 o = {__float_as_int(v.x + add[j][t].x), __float_as_int(v.y + add[j][t].y), __float_as_int(v.z + add[j][t].z),
                                     __float_as_int(v.w + add[j][t].w)};
                    __builtin_amdgcn_raw_buffer_store_b128(o, rsC, off_c[j][t], 0, 0);
                }
            }
        }
        if (!has_next) return;
    }
#undef SB
}

// Sums the ksplit fp32 partial tiles of each split tile in a fixed order and applies the epilogue.
// 64 workgroups per tile; a thread owns 4 consecutive columns of one row.
template <bool OUT_F32>
__global__ __launch_bounds__(256) void k_splitk_reduce(const float* __restrict__ partial, int block0, DmaGroup grp) {
    const int r = blockIdx.x >> 6, sub = blockIdx.x & 63;
    const int prob = grp.problem_of(block0 + r), ksplit = grp.ksplit.d;
    const DmaProblem& g = grp.p[prob];
    const int M = g.M, N = g.N, ldc = g.ldc, ldr = g.ldr, accumulate = g.accumulate;
    void* const Cv = g.C;
    const bf16_t* const R = g.R;
    int tm, tn;
    g.map.tile(block0 + r - grp.first[prob], tm, tn);
    const int q = sub * 256 + threadIdx.x;
    const int row = q >> 6, col = (q & 63) * 4;
    const float* p = partial + (size_t)r * ksplit * (DTILE * DTILE) + row * DTILE + col;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    for (int c = 0; c < ksplit; c++) {
        const float4 t = *reinterpret_cast<const float4*>(p + (size_t)c * (DTILE * DTILE));
        v[0] += t.x; v[1] += t.y; v[2] += t.z; v[3] += t.w;
    }
    const int m = tm * DTILE + row, n = tn * DTILE + col;
    if (m >= M || n >= N) return;
    if (OUT_F32) {
        float* c = reinterpret_cast<float*>(Cv) + (size_t)m * ldc + n;
        if (accumulate) {
            const float4 old = *reinterpret_cast<const float4*>(c);
            v[0] += old.x; v[1] += old.y; v[2] += old.z; v[3] += old.w;
        }
        *reinterpret_cast<float4*>(c) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
        if (R) {
            const uint2 rr = *reinterpret_cast<const uint2*>(R + (size_t)m * ldr + n);
            v[0] += lo_bf(rr.x); v[1] += hi_bf(rr.x); v[2] += lo_bf(rr.y); v[3] += hi_bf(rr.y);
        }
        uint2 o;
        o.x = pack_bf2(v[0], v[1]);
        o.y = pack_bf2(v[2], v[3]);
        *reinterpret_cast<uint2*>(reinterpret_cast<bf16_t*>(Cv) + (size_t)m * ldc + n) = o;
    }
}

// extent in bytes of each operand as laid out in memory (rows x ld), for the buffer bounds
static long extent_a(const GemmDesc& g) {
    const long rows = (g.kind == GEMM_TN) ? g.K : g.M, cols = (g.kind == GEMM_TN) ? g.M : g.K;
    return ((rows - 1) * g.lda + cols) * 2;
}
static long extent_b(const GemmDesc& g, int K) {
    const long rows = (g.kind == GEMM_NT) ? g.N : K, cols = (g.kind == GEMM_NT) ? K : g.N;
    return ((rows - 1) * g.ldb + cols) * 2;
}

// Compute units of the current device (one persistent workgroup each), asked once per device.
static int device_cus(hipError_t& err) {
    static std::atomic<int> cached[64];
    int dev = 0;
    err = hipGetDevice(&dev);
    if (err != hipSuccess) return 0;
    const int slot = dev & 63;
    int n = cached[slot].load(std::memory_order_relaxed);
    if (n > 0) return n;
    err = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
    if (err != hipSuccess) return 0;
    if (n < 8) n = 8;
    cached[slot].store(n, std::memory_order_relaxed);
    return n;
}

// k shares of each tile of the last, partial round of `tiles` (1: it is not cut)
static int tail_shares(const GemmDesc& g, int tiles, int cus) {
    const int rem = tiles % cus, nk = (g.K + DK - 1) / DK;
    if (rem == 0 || rem > cus / 2 || !g.ws) return 1;
    int s = std::min(cus / rem, 8);
    while (s > 1 && (nk / s < 4 || (size_t)rem * s * DTILE * DTILE * sizeof(float) > g.ws_bytes)) s--;
    return s;
}

// Full rounds of one tile per compute unit run as one persistent workgroup per unit.  A last, partial round of R
// tiles would leave most units idle, so it is cut along k into floor(units / R) shares per tile, which the same
// workgroups take up after their whole tiles (fp32 partials in `ws`, summed in a fixed order by a small second kernel).
template <int KIND, bool RES>
static auto dma_kernel() {
    if constexpr (KIND == GEMM_TN) return &k_gemm_dma_tn;
    else return &k_gemm_dma<KIND, RES>;
}
template <int KIND, bool RES = false>
static hipError_t launch_dma(const GemmDesc* g, int n, hipStream_t st) {
    constexpr int LDS = DSTAGES * 2 * DSTAGE_BYTES + 8 * 4096;   // two stages + the epilogue patches of the 8 waves
    static std::atomic<uint64_t> lds_ok{0};
    auto kern = dma_kernel<KIND, RES>();
    const hipError_t e = allow_lds((const void*)kern, LDS, lds_ok);
    if (e != hipSuccess) return e;
    hipError_t ce = hipSuccess;
    const int NUM_CU = device_cus(ce);
    if (ce != hipSuccess) return ce;
    DmaGroup grp{};
    grp.K = g[0].K;
    int tiles = 0;
    for (int i = 0; i < DMA_MAX; i++) grp.first[i] = INT_MAX;
    for (int i = 0; i < n; i++) {
        const GemmDesc& q = g[i];
        grp.p[i] = DmaProblem{(const bf16_t*)q.A, (const bf16_t*)q.B, q.C, (const bf16_t*)q.R, (uint32_t)extent_a(q), (uint32_t)extent_b(q, q.K),
                              q.lda, q.ldb, q.ldc, q.ldr, q.M, q.N, q.accumulate, tile_map(q.M, q.N, DTILE, DTILE)};
        grp.first[i] = tiles;
        tiles += grp.p[i].map.tiles();
    }
    const int ksplit = tail_shares(g[0], tiles, NUM_CU);
    const int tail = ksplit > 1 ? tiles % NUM_CU : 0, full = tiles - tail;
    grp.ksplit = divisor(ksplit);
    // one launch: a persistent workgroup per CU walks the whole tiles and then the k shares of the tail tiles
    const int n_items = full + tail * ksplit;
    kern<<<n_items < NUM_CU ? n_items : NUM_CU, 512, LDS, st>>>(grp, full, n_items, (float*)g[0].ws);
    if (tail > 0) k_splitk_reduce<KIND == GEMM_TN><<<tail * 64, 256, 0, st>>>((const float*)g[0].ws, full, grp);
    return hipGetLastError();
}

// Whether a problem's shares are left to the norm that reads its result, which then gathers them with one workgroup (or wave) a
// row: not more than 64 KB a row, which takes it about as long as the reduction kernel's launch.
static bool leaves_shares(const GemmDesc& g, int ksplit) { return (long)g.N * ksplit <= SPLIT_ROW && g.N % 8 == 0; }

// Plan of one problem or of a group: the kernel variant, k splits, the order of the problems (longest k loop first), the
// predicted time and, for several micro-batches, the problems (bits) whose sums over them are not formed one after the other.
struct Plan { int v, ksplit[RING_MAX], order[RING_MAX]; double t; unsigned apart; };

template <bool BWD, int MB, bool F, int NP, int BM, int BN, int WM, int WN, int NS, bool NORM>
static auto ring_kernel() {
    if constexpr (NORM) return &k_gemm_ring_norm<MB, F, NP, BM, BN, WM, WN, NS>;
    else return &k_gemm_ring<BWD, MB, F, NP, BM, BN, WM, WN, NS>;
}
template <bool BWD, int MB, bool F, int NP, int BM, int BN, int WM, int WN, int NS, bool NORM>
static hipError_t launch_ring_n(const GemmDesc* g, const int* order, const int* ksplit, unsigned apart, int n, hipStream_t st) {
    constexpr int LDS = NORM ? (NORM_K * BM + NS * BN * DK) * 2 : NS * (BM + BN) * DK * 2;
    static std::atomic<uint64_t> lds_ok{0};
    auto kern = ring_kernel<BWD, MB, F, NP, BM, BN, WM, WN, NS, NORM>();
    const hipError_t e = allow_lds((const void*)kern, LDS, lds_ok);
    if (e != hipSuccess) return e;
    RingGroup<MB, F, NP> grp;
    RingReduce<MB, F, NP> red;
    red.bm = divisor(BM); red.bn = divisor(BN);
    int starts[RING_MAX], red_starts[RING_MAX];
    for (int i = 0; i < RING_MAX; i++) starts[i] = red_starts[i] = INT_MAX;
    int first = 0, red_first = 0, n_red = 0, tn = 0;
    float* partial = (float*)g[0].ws;
    for (int i = 0; i < n; i++) {
        const GemmDesc& q = g[order[i]];
        const int s = ksplit[order[i]];
        RingProblem<MB, F>& p = grp.p[i];
        const int nk = (q.K + DK - 1) / DK;
        if constexpr (MB == 1) {
            p.A.p[0] = const_cast<void*>(q.A); p.B.p[0] = const_cast<void*>(q.B); p.C.p[0] = q.C; p.R.p[0] = const_cast<void*>(q.R);
        } else {
            for (int m = 0; m < MB; m++) {
                p.A.p[m] = q.each->A.p[m]; p.B.p[m] = q.each->B.p[m]; p.C.p[m] = q.each->C.p[m]; p.R.p[m] = q.each->R.p[m];
            }
        }
        p.kseg[0] = q.k1 ? q.k1 / DK : INT_MAX; p.kseg[1] = q.k2 ? q.k2 / DK : INT_MAX;
        p.Bseg[0] = (const bf16_t*)q.B1; p.Bseg[1] = (const bf16_t*)q.B2;
        p.a_bytes = (uint32_t)extent_a(q); p.b_bytes = (uint32_t)extent_b(q, q.k1 ? q.k1 : q.K);
        tn |= (q.kind == GEMM_TN) << i;
        p.lda = q.lda; p.ldb = q.ldb; p.ldc = q.ldc; p.ldr = q.ldr; p.M = q.M; p.N = q.N; p.K = q.K;
        p.accumulate = q.accumulate;
        p.map = tile_map(q.M, q.N, BM, BN);
        p.nk = nk;
        const int tiles = p.map.tiles();
        p.tiles = divisor(tiles); p.items = divisor(tiles * s); p.ksplit = divisor(s);
        if constexpr (F) {
            const GemmFuse& f = q.fuse;
            for (int m = 0; m < MB; m++) {
                p.X.p[m] = MB == 1 ? f.X : q.each->X.p[m];
                p.Y.p[m] = MB == 1 ? f.Y : q.each->Y.p[m];
            }
            p.fuse = f.kind; p.period = f.period; p.rot = f.rot; p.tokens = divisor(f.seq > 0 ? f.seq : 1); p.table_seq = f.table_seq; p.table = f.table;
            p.shift = f.kind == FUSE_ROPE ? (f.period == 128 ? 7 : 6) : 31;
        }
        starts[i] = p.first = first;
        p.micro = q.micro;
        p.seq = q.kind == GEMM_TN && s == 1 && !(apart >> order[i] & 1) ? q.micro : 1;
        first += tiles * s * (q.micro / p.seq);
        if (q.split) *q.split = GemmSplit{nullptr, 1, BM, BN, (q.N + BN - 1) / BN};
        p.partial = partial;
        if (s > 1 || (q.kind == GEMM_TN && p.seq < q.micro)) {
            if (nk < s) return hipErrorInvalidValue;
            partial += (size_t)tiles * s * q.micro * BM * BN;
            if (s > 1 && q.split && leaves_shares(q, s)) {
                q.split->partial = p.partial;
                q.split->ksplit = s;
                continue;
            }
            const int vectors = q.N / (q.fuse.kind == FUSE_ROPE || q.fuse.kind == FUSE_SWIGLU ? 8 : 4);
            const int blocks = (int)(((long)q.M * vectors + 255) / 256);
            red_starts[n_red] = red_first;
            auto& j = red.j[n_red++];
            j.first = red_first;
            static_cast<RingFuse<MB, F>&>(j) = p;
            j.C = p.C; j.R = p.R; j.partial = p.partial;
            j.ksplit = s; j.ldc = q.ldc; j.ldr = q.ldr; j.M = q.M; j.N = q.N; j.accumulate = q.accumulate; j.out_f32 = q.out_f32;
            j.micro = q.micro; j.tiles_n = p.map.tiles_n; j.blocks = divisor(blocks); j.vectors = divisor(vectors);
            red_first += blocks * (q.out_f32 ? 1 : q.micro);
        }
    }
    if (MB > 1 && (size_t)(partial - (float*)g[0].ws) * sizeof(float) > g[0].ws_room) return hipErrorInvalidValue;
    if constexpr (NORM) {
        const GemmNorm& q = *g[0].norm;
        RingNorm<MB> norm;
        for (int m = 0; m < MB; m++) { norm.xn.p[m] = q.xn.p[m]; norm.r.p[m] = q.r.p[m]; }
        norm.gain = (const bf16_t*)q.gain; norm.eps = q.eps; norm.writer = 0;
        kern<<<first, WM * WN * 64, (g[0].K * BM + NS * BN * DK) * 2, st>>>(starts[1], starts[2], starts[3], norm, grp);
        return hipGetLastError();
    } else {
        kern<<<first, WM * WN * 64, LDS, st>>>(starts[1], starts[2], starts[3], tn, grp);
    }
    if (n_red) k_ring_reduce<MB, F, NP><<<red_first, 256, 0, st>>>(red_starts[1], red_starts[2], red_starts[3], red);
    return hipGetLastError();
}

template <bool BWD, bool F, int BM, int BN, int WM, int WN, int NS, bool NORM>
static hipError_t launch_ring_f(const GemmDesc* g, const int* order, const int* ksplit, unsigned apart, int n, hipStream_t st) {
    if (g[0].micro > 1) return launch_ring_n<BWD, MICRO_MAX, F, RING_MAX, BM, BN, WM, WN, NS, NORM>(g, order, ksplit, apart, n, st);
    return n == 1 ? launch_ring_n<BWD, 1, F, 1, BM, BN, WM, WN, NS, NORM>(g, order, ksplit, apart, n, st)
                  : launch_ring_n<BWD, 1, F, RING_MAX, BM, BN, WM, WN, NS, NORM>(g, order, ksplit, apart, n, st);
}
template <bool BWD, int BM, int BN, int WM, int WN, int NS, bool NORM = false>
static hipError_t launch_ring(const GemmDesc* g, const Plan& p, int n, hipStream_t st) {
    constexpr bool CAN = BM * BN <= (BWD ? fuse_tile(FUSE_SWIGLU_BWD) : fuse_tile(FUSE_ROPE));
    if constexpr (CAN)
        if (g[0].fuse.kind) return launch_ring_f<BWD, true, BM, BN, WM, WN, NS, NORM>(g, p.order, p.ksplit, p.apart, n, st);
    return launch_ring_f<BWD, false, BM, BN, WM, WN, NS, NORM>(g, p.order, p.ksplit, p.apart, n, st);
}

// Which kernel, tile and k split: the smallest predicted time over the variants below.  A launch of W workgroups runs
// as rounds of 256 (one workgroup per CU) or 512 (two per CU); a round takes e + (k stages) * t, with t = t_full when
// the round fills every slot and t_one when the last round leaves each CU one workgroup at most; never less than the
// operands and the result take at 5 TB/s.  A k split adds a reduction kernel: 3 us and its traffic at 6.5 TB/s.
// The constants (microseconds) are a least-squares fit to 100000 measured launches of 5600 random problems (M 17..8192,
// N 64..28672, K 64..16384, all three kinds, weights read cold) on one MI355X: 7 to 11 % rms error (14 % for 256x256),
// the choice costs 1.6 % over the best variant of each problem.  Against one 128x128 register-staged kernel for
// everything below 64 tiles of 256x256 the problems of that class take half the time (333x4096x11008 NT: 152 -> 50 us,
// 36x8384x25152 NN: 336 -> 93 us, 128x512x2200 TN: 29 -> 8.5 us).
// Tiles of 192 rows are built for NT problems: 333x12288x4096 60 -> 51 us, 333x22016x4096 95 -> 78, 3300x3072x4096 89 -> 83.
// 192 rows or columns of a k-strided operand cannot be (its k row must be a power of two of 16-byte chunks): that rules
// out TN, and 192 columns of an NN problem.  192x128 and 192x256 would fit an NN problem; they were never measured there.
// A round is 256 workgroups here, the CUs of the card in its default partition, where the constants were measured; on fewer
// the choice is still correct, and only the 256x256 kernel adapts (its workgroups and its split follow the device's CUs).
struct Variant { int bm, bn, per_cu; bool nt_only; double t0, e, t_one, t_full; };
enum { V_64x64, V_64x128, V_128x128, V_128x128_2, V_128x256, V_192x128, V_192x192, V_192x256, V_DMA, V_COUNT };
static constexpr Variant VARIANTS[V_COUNT] = {
    {64, 64, 2, false, 1.76, 1.83, 0.256, 0.464},   {64, 128, 2, false, 1.69, 2.15, 0.372, 0.690},
    {128, 128, 1, false, 1.88, 2.65, 0.467, 0.589}, {128, 128, 2, false, 1.13, 3.10, 0.639, 0.997},
    {128, 256, 1, false, 2.10, 3.76, 0.741, 0.947}, {192, 128, 1, true, 2.34, 2.97, 0.619, 0.778},
    {192, 192, 1, true, 1.81, 4.58, 0.960, 1.067},  {192, 256, 1, true, 2.07, 4.57, 1.085, 1.305},
    {256, 256, 1, false, 0.97, 5.44, 1.587, 1.639},
};
static constexpr int SPLITS[] = {1, 2, 3, 4, 6, 8};

// Time of a k stage in a last round of `busy` workgroups, one per CU.  Where each CU holds one workgroup at most anyway,
// loops of more than 64 stages run the longer towards t_full the more CUs are busy (the power limit and the traffic
// behind L2 catch up with them): 4096x1536x12288 NN, 192 tiles of 128x256, 180 us where t_one alone predicts 148 and
// 256x256 tiles in two shares of k take 159.  On 130 random problems with 40 to 520 tiles of 256x256 the choice costs
// 1.25 % over the best variant of each, 1.6 % with t_one alone; the same ramp for shorter loops gains nothing.
static double stage_us(const Variant& q, long busy, double ks) {
    if (q.per_cu > 1 || ks <= 64.0) return q.t_one;
    return q.t_one + (q.t_full - q.t_one) * (busy / 256.0) * std::min(1.0, ks / 64.0 - 1.0);
}
static double out_bytes(const GemmDesc& g) { return (double)g.M * g.N * (g.out_f32 ? 8 : 2); }
static double floor_us(const GemmDesc& g) { return (2.0 * g.K * ((double)g.M + g.N) + out_bytes(g)) / 5.0e6; }
static long tiles_of(const GemmDesc& g, const Variant& q) { return (long)((g.M + q.bm - 1) / q.bm) * ((g.N + q.bn - 1) / q.bn); }
static int tile_size(int v) { return VARIANTS[v].bm * VARIANTS[v].bn; }
static bool may_split(const GemmDesc& g, const Variant& q, int s) {
    const long tiles = tiles_of(g, q);
    return s == 1 || (g.ws && (g.K + DK - 1) / DK / s >= 2 && tiles * (s - 1) <= 700 &&
                      (size_t)tiles * s * q.bm * q.bn * sizeof(float) <= g.ws_bytes);
}
static double reduce_us(const GemmDesc& g, const Variant& q, int s) {
    return s > 1 ? ((double)tiles_of(g, q) * q.bm * q.bn * 8.0 * s + out_bytes(g)) / 6.5e6 : 0.0;
}

// `tiles` tiles of 256x256 in one launch, which splits its last round itself.
static double dma_us(long tiles, int nk, double floor, bool ws) {
    const Variant& q = VARIANTS[V_DMA];
    const long full = tiles / 256, rem = tiles % 256;
    int s = rem > 0 && rem <= 128 && ws ? (int)(256 / rem > 8 ? 8 : 256 / rem) : 1;
    while (s > 1 && nk / s < 4) s--;
    double t = full * (q.e + nk * q.t_full) + (rem ? q.e + (double)nk / s * q.t_one : 0.0);
    if (t < floor) t = floor;
    if (s > 1) t += 2.0 + rem * s * 0.05;
    return 0.95 * (t + q.t0);   // another kernel has to promise more than the model's bias at these sizes
}

// One problem.  whole_only: it has to run as one piece (B in several segments), which the 256x256 kernel cannot.
static Plan plan_one(const GemmDesc& g, bool whole_only) {
    const int nk = (g.K + DK - 1) / DK;
    const double floor = floor_us(g);
    Plan best{V_DMA, {1}, {0}, 1e30};
    for (int v = 0; v < V_COUNT; v++) {
        const Variant& q = VARIANTS[v];
        const long tiles = tiles_of(g, q);
        if ((v == V_DMA && (whole_only || tiles < 64)) || (q.nt_only && g.kind != GEMM_NT)) continue;
        const long cap = 256L * q.per_cu;
        if (v == V_DMA) {
            const double t = dma_us(tiles, nk, floor, g.ws != nullptr);
            if (t < best.t) best = Plan{V_DMA, {1}, {0}, t};
            continue;
        }
        for (const int s : SPLITS) {
            if (!may_split(g, q, s)) break;
            const long w = tiles * s, full = w / cap, rem = w % cap;
            const double ks = (double)nk / s;
            double t = full * (q.e + ks * q.t_full) + (rem ? q.e + ks * (rem <= 256 ? stage_us(q, rem, ks) : q.t_full) : 0.0);
            if (t < floor) t = floor;
            if (s > 1) t += 3.0 + reduce_us(g, q, s);
            t += q.t0;
            if (t < best.t) best = Plan{v, {s}, {0}, t};
        }
    }
    return best;
}

// w workgroups of `least` to `most` k stages, `sum` in all, in one launch.  They are handed out longest first; the launch ends with the
// longest of them if all fit the chip at once, otherwise when the work is spent, give or take half a short one.
static double group_us(const Variant& q, long w, double most, double least, double sum) {
    const double slots = 256.0 * q.per_cu;
    if (w <= 256) return q.e + most * stage_us(q, w, most);
    if (w <= slots) return q.e + most * q.t_full;
    return std::max(q.e + most * q.t_full, (w * q.e + sum * q.t_full) / slots + 0.5 * (q.e + least * q.t_full));
}

// Several problems in one launch of one variant.  The splits tried are those that bring every problem's k loop below a common length.
static Plan plan_group(const GemmDesc* g, int n) {
    double floor = 0.0;
    for (int i = 0; i < n; i++) floor += floor_us(g[i]);
    Plan best{V_DMA, {1, 1, 1, 1}, {0, 1, 2, 3}, 1e30};
    for (int v = 0; v < V_DMA; v++) {
        const Variant& q = VARIANTS[v];
        if (q.nt_only && g[0].kind != GEMM_NT) continue;
        for (int lead = 0; lead < n; lead++)
            for (const int ls : SPLITS) {
                if (!may_split(g[lead], q, ls)) break;
                const double len = (double)((g[lead].K + DK - 1) / DK) / ls;
                Plan p{v, {1, 1, 1, 1}, {0, 1, 2, 3}, 0.0};
                long w = 0;
                size_t ws = 0;
                double reduce = 0.0, most = 0.0, least = 1e30, sum = 0.0;
                for (int i = 0; i < n; i++) {
                    const int nk = (g[i].K + DK - 1) / DK;
                    int s = 1;
                    for (const int c : SPLITS) {
                        if (!may_split(g[i], q, c)) break;
                        s = c;
                        if ((double)nk / c <= len) break;
                    }
                    p.ksplit[i] = s;
                    const long tiles = tiles_of(g[i], q);
                    w += tiles * s;
                    if (s > 1) ws += (size_t)tiles * s * q.bm * q.bn * sizeof(float);
                    reduce += reduce_us(g[i], q, s);
                    const double ks = (double)nk / s;
                    most = std::max(most, ks); least = std::min(least, ks); sum += tiles * s * ks;
                }
                if (ws > g[0].ws_bytes) continue;
                p.t = std::max(group_us(q, w, most, least, sum), floor) + q.t0 + (ws ? 3.0 + reduce : 0.0);
                if (p.t < best.t) best = p;
            }
    }
    auto len = [&](int i) { return (double)g[i].K / best.ksplit[i]; };
    for (int i = 1; i < n; i++)   // longest first
        for (int j = i; j > 0 && len(best.order[j]) > len(best.order[j - 1]); j--) std::swap(best.order[j], best.order[j - 1]);
    return best;
}

// A plan depends on sizes alone, and a program asks for the same few again and again: each thread remembers the last one
// of each of 256 hash slots (a group costs 5 to 10 us to plan).
struct PlanKey {
    int n, whole, sizes[RING_MAX][4];
    size_t ws;
    bool operator==(const PlanKey& o) const { return n == o.n && whole == o.whole && ws == o.ws && !memcmp(sizes, o.sizes, sizeof sizes); }
};
static Plan plan(const GemmDesc* g, int n, bool whole_only) {
    struct Slot { PlanKey key; Plan plan; };
    static thread_local Slot slots[256];
    PlanKey k{};
    k.n = n; k.whole = whole_only; k.ws = g[0].ws ? g[0].ws_bytes : 0;
    uint32_t h = (uint32_t)n * 2u + whole_only;
    for (int i = 0; i < n; i++) {
        const int v[4] = {g[i].kind, g[i].M, g[i].N, g[i].K};
        for (int j = 0; j < 4; j++) { k.sizes[i][j] = v[j]; h = (h ^ (uint32_t)v[j]) * 0x9E3779B1u; h ^= h >> 15; }
    }
    Slot& s = slots[h & 255];
    if (!(s.key == k)) s = Slot{k, n == 1 ? plan_one(g[0], whole_only) : plan_group(g, n)};   // key.n is 0 in an empty slot
    return s.plan;
}

static hipError_t launch_tiles256(const GemmDesc* g, int n, hipStream_t st) {
    bool res = false;
    for (int i = 0; i < n; i++) res |= g[i].R != nullptr;
    switch (g[0].kind) {
        case GEMM_NT: return res ? launch_dma<GEMM_NT, true>(g, n, st) : launch_dma<GEMM_NT>(g, n, st);
        case GEMM_NN: return res ? launch_dma<GEMM_NN, true>(g, n, st) : launch_dma<GEMM_NN>(g, n, st);
        default: return launch_dma<GEMM_TN>(g, n, st);
    }
}
template <bool BWD>
static hipError_t launch_variant(const GemmDesc* g, int n, const Plan& p, hipStream_t st) {
    if constexpr (!BWD)
        if (g[0].norm) return launch_ring<false, 64, 64, 2, 2, 4, true>(g, p, n, st);   // gemm_bf16 has seen to the rest
    switch (p.v) {
        case V_64x64: return launch_ring<BWD, 64, 64, 2, 2, 4>(g, p, n, st);
        case V_64x128: return launch_ring<BWD, 64, 128, 2, 2, 3>(g, p, n, st);
        case V_128x128: return launch_ring<BWD, 128, 128, 2, 4, 4>(g, p, n, st);
        case V_128x128_2: return launch_ring<BWD, 128, 128, 2, 2, 2>(g, p, n, st);
        case V_128x256: return launch_ring<BWD, 128, 256, 2, 4, 3>(g, p, n, st);
    }
    if constexpr (!BWD) {
        switch (p.v) {
            case V_192x128: return launch_ring<false, 192, 128, 2, 4, 4>(g, p, n, st);
            case V_192x192: return launch_ring<false, 192, 192, 2, 2, 3>(g, p, n, st);
            case V_192x256: return launch_ring<false, 192, 256, 2, 4, 2>(g, p, n, st);
        }
    }
    return launch_tiles256(g, n, st);
}
// A plan for several micro-batches: the tile and the k splits stay those of one, so that the bits do.  A workgroup forms a tile of a
// weight gradient for one micro-batch after the other, or each micro-batch's product has a workgroup of its own and the reduction
// adds them, in the same order: shorter k loops for the traffic of the partial sums.  The latter where it is predicted to take
// under 0.85 of the time: on 130 launches (hidden 256 to 2048, 64 to 3000 tokens, 2 to 8 micro-batches) it takes 0.63 to 0.98 of it
// there (three of 768x512 and 1536x512 over 2200 tokens with their input gradient 58.6 -> 49.6 us, eight of 768x768 over 1500
// 81 -> 55), and 1.13 at most where it is predicted to take less at all.
static Plan micro_plan(const GemmDesc* g, int n, const Plan& p) {
    const Variant& q = VARIANTS[p.v];
    const int micro = g[0].micro;
    Plan best = p;
    best.t = 1e30;
    for (int apart = 0; apart < 2; apart++) {
        Plan o = p;
        double len[RING_MAX], most = 0.0, least = 1e30, sum = 0.0, reduce = 0.0, floor = 0.0;
        long w = 0;
        size_t ws = 0;
        bool reduces = false;
        for (int i = 0; i < n; i++) {
            const int s = p.ksplit[i];
            const long tiles = tiles_of(g[i], q);
            const bool one = g[i].kind == GEMM_TN && s == 1, sums = one && !apart;   // whether a workgroup works for all micro-batches
            len[i] = (double)((g[i].K + DK - 1) / DK) / s * (sums ? micro : 1);
            if (one && apart) o.apart |= 1u << i;
            const long wgs = tiles * s * (sums ? 1 : micro);
            w += wgs;
            most = std::max(most, len[i]); least = std::min(least, len[i]); sum += wgs * len[i];
            floor += g[i].kind == GEMM_TN ? (2.0 * g[i].K * micro * ((double)g[i].M + g[i].N) + out_bytes(g[i])) / 5.0e6 : 0.0;
            if (s == 1 && !(one && apart)) continue;
            const size_t bytes = (size_t)wgs * q.bm * q.bn * sizeof(float);
            ws += bytes;
            if (s > 1 && g[i].split && leaves_shares(g[i], s)) continue;
            reduces = true;
            reduce += 2.0 * bytes / 6.5e6;
        }
        if (apart && (!o.apart || ws > g[0].ws_room)) break;
        o.t = std::max(group_us(q, w, most, least, sum), floor) + (reduces ? 3.0 + reduce : 0.0);
        for (int i = 1; i < n; i++)   // longest first
            for (int j = i; j > 0 && len[o.order[j]] > len[o.order[j - 1]]; j--) std::swap(o.order[j], o.order[j - 1]);
        if (o.t < 0.85 * best.t) best = o;
    }
    return best;
}

static hipError_t launch_planned(const GemmDesc* g, int n, const Plan& p, hipStream_t st) {
    if (g[0].kind == GEMM_NT) return launch_variant<false>(g, n, p, st);
    return launch_variant<true>(g, n, g[0].micro > 1 ? micro_plan(g, n, p) : p, st);
}

// The segments of a segmented problem one after the other, each adding to what the ones before it have left in C.
static int segments(const GemmDesc& g, GemmDesc out[3]) {
    const int at[4] = {0, g.k1 ? g.k1 : g.K, g.k2 ? g.k2 : g.K, g.K};
    const void* const b[3] = {g.B, g.B1, g.B2};
    int n = 0;
    for (int i = 0; i < 3 && at[i] < g.K; i++) {
        GemmDesc& o = out[n++];
        o = g;
        o.k1 = o.k2 = 0; o.B1 = o.B2 = nullptr; o.split = nullptr;
        o.A = (const bf16_t*)g.A + at[i];
        o.B = b[i];
        o.K = at[i + 1] - at[i];
        if (i) { o.R = g.C; o.ldr = g.ldc; }
    }
    return n;
}

static hipError_t check(const GemmDesc& g) {
    const long a_bytes = extent_a(g), b_bytes = extent_b(g, g.K);
    if (a_bytes >= (1L << 32) - (1L << 25) || b_bytes >= (1L << 32) - (1L << 25)) return hipErrorInvalidValue;
    if (g.lda > 65535 || g.ldb > 65535) return hipErrorInvalidValue;
    // C (and the residual) are addressed with 32-bit byte offsets below 2 GB
    if (((long)(g.M - 1) * g.ldc + g.N) * (g.out_f32 ? 4 : 2) >= (1L << 31)) return hipErrorInvalidValue;
    if (g.R && ((long)(g.M - 1) * g.ldr + g.N) * 2 >= (1L << 31)) return hipErrorInvalidValue;
    // a k-contiguous operand is fetched 64 k values at a time with no per-row bound
    if (g.kind != GEMM_TN && g.K % 64 != 0) return hipErrorInvalidValue;
    if (g.N % 4 != 0) return hipErrorInvalidValue;   // the epilogues move 4 columns at a time
    // activations come out in bf16 (NT, NN), parameter gradients in fp32 (TN)
    if ((g.out_f32 != 0) != (g.kind == GEMM_TN) || (g.out_f32 && g.R)) return hipErrorInvalidValue;
    // segments of B: rows of an NN problem, in order, each a whole number of k tiles
    if (g.k1 && (g.kind != GEMM_NN || !g.B1 || g.k1 % DK || g.k1 >= g.K)) return hipErrorInvalidValue;
    // fusions: whole heads of 64 or 128 columns, a whole gate|up row, a whole dm row; nothing is added
    const GemmFuse& f = g.fuse;
    if (f.kind && (g.R || g.accumulate)) return hipErrorInvalidValue;
    if (f.kind == FUSE_ROPE && (g.kind != GEMM_NT || (f.period != 64 && f.period != 128) || g.N % f.period || f.rot % f.period || f.rot > g.N ||
                                !f.table || f.seq <= 0 || f.table_seq < f.seq)) return hipErrorInvalidValue;
    if (f.kind == FUSE_SWIGLU && (g.kind != GEMM_NT || f.period != g.N || g.N % 64 || g.ldc != g.N || !f.X)) return hipErrorInvalidValue;
    if (f.kind == FUSE_SWIGLU_BWD && (g.kind != GEMM_NN || !f.X || !f.Y || (long)g.M * g.N * 4 >= (1L << 31))) return hipErrorInvalidValue;
    if (g.k2 && (!g.k1 || !g.B2 || g.k2 % DK || g.k2 <= g.k1 || g.k2 >= g.K)) return hipErrorInvalidValue;
    return hipSuccess;
}

// How a list of problems is launched, and the predicted time.
struct Route {
    enum { APART, RING, TILES256 } how;
    Plan group, each[DMA_MAX];   // each[i].v == V_COUNT: segment by segment
    double t;
};
static void route(const GemmDesc* g, int n, Route& r) {
    r.how = Route::APART;
    r.t = 0.0;
    for (int i = 0; i < n; i++) {
        r.each[i] = plan(g + i, 1, false);
        if (g[i].k1) {   // in one piece on the ring kernel, or segment by segment
            GemmDesc seg[3];
            const int m = segments(g[i], seg);
            double t = 0.0;
            for (int j = 0; j < m; j++) t += plan(seg + j, 1, false).t;
            r.each[i] = plan(g + i, 1, true);
            if (t < r.each[i].t) { r.each[i].v = V_COUNT; r.each[i].t = t; }
        }
        r.t += r.each[i].t;
    }
    if (n == 1) return;
    if (n <= RING_MAX) {
        r.group = plan(g, n, false);
        if (r.group.t < r.t) { r.how = Route::RING; r.t = r.group.t; }
    }
    bool alike = true;
    double floor = 0.0;
    long tiles = 0;
    for (int i = 0; i < n; i++) {
        alike = alike && g[i].kind == g[0].kind && g[i].K == g[0].K && !g[i].k1;
        floor += floor_us(g[i]);
        tiles += tiles_of(g[i], VARIANTS[V_DMA]);
    }
    if (alike && tiles >= 64) {
        const double t = dma_us(tiles, (g[0].K + DK - 1) / DK, floor, g[0].ws != nullptr);
        if (t < r.t) { r.how = Route::TILES256; r.t = t; }
    }
}

// Whether the weight gradients of a layer (dw, one k) are better left to one launch at the end than launched with the
// input gradients (groups[i] holds n[i] problems of which the last is the input gradient): 256x256 tiles of all of them
// fill the rounds of the chip that the projections one by one leave ragged, but then the small ones cannot fill up the
// input gradients' rounds.
bool gemm_bf16_defer(const GemmDesc* dw, int n_dw, const GemmDesc* const groups[3], const int n[3]) {
    if (n_dw > DMA_MAX) return false;
    Route r;
    route(dw, n_dw, r);
    if (r.how != Route::TILES256) return false;
    double last = r.t, with = 0.0;
    for (int i = 0; i < 3; i++) {
        route(groups[i], n[i], r);
        with += r.t;
        route(groups[i] + n[i] - 1, 1, r);
        last += r.t;
    }
    return last < 0.99 * with;
}

bool gemm_bf16_shares_launch(const GemmDesc* g, int n) {
    if (n < 2 || n > DMA_MAX) return false;
    Route r;
    route(g, n, r);
    return r.how != Route::APART;
}

// Weight gradients that 256x256 tiles would take, of too few tokens for those to be cut along k: several micro-batches go to the
// ring kernel all the same, which forms the same bits (whole k loops in order) and reads and writes a gradient once for all
// of them, which is most of the traffic of such a launch.  2 layers of hidden 4096, ffn 11008, 64 tokens, 8 micro-batches:
// 10.6 -> 4.4 ms.  One tile for all of them: two 128x128 workgroups a CU, of which one loads while the other writes.  24 random
// stages (hidden 2112 to 11776, 4 to 431 tokens, 2 to 8 micro-batches) take 0.90 to 1.00 of what they do with one workgroup of
// 128x256 (hidden 9856, 38 tokens, 8 micro-batches 6893 -> 6220 us; from 128 tokens on no change); with one of 128x128 16 others
// took 0.4 to 6 % longer, with 64x128 ones 6 % less to 3 % more.
constexpr int WHOLE_DW = V_128x128_2;
static bool whole_dw(const GemmDesc& g) { return g.kind == GEMM_TN && (g.K + DK - 1) / DK < 8; }   // see tail_shares

bool gemm_bf16_on_ring(const GemmDesc* g, int n, RingUse* use) {
    if (n < 1 || n > DMA_MAX) return false;
    Route r;
    route(g, n, r);
    const bool ring = r.how == Route::RING;
    if (ring && r.group.v >= V_DMA) return false;
    *use = RingUse{0, 0, 0};
    for (int i = 0; i < n; i++) {
        const Plan& p = ring ? r.group : r.each[i];
        int v = p.v, s = p.ksplit[ring ? i : 0];
        if (r.how == Route::TILES256 || v == V_DMA) {
            if (!whole_dw(g[i])) return false;
            v = WHOLE_DW; s = 1;
        } else if (v > V_DMA) return false;
        const int tile = tile_size(v);
        const long w = tiles_of(g[i], VARIANTS[v]) * s;
        const size_t b = s > 1 ? (size_t)w * tile * sizeof(float) : 0;
        use->partial = ring ? use->partial + b : std::max(use->partial, b);
        use->workgroups = ring ? use->workgroups + w : std::max(use->workgroups, w);
        use->tile = std::max(use->tile, tile);
    }
    return true;
}

// Whether the launch of these projections norms its rows itself: where it is one of whole 64x64 tiles, one workgroup a CU at most for
// a micro-batch, and a row has up to NORM_K columns.  Forward passes of hidden 128 and 256, 17 to 1100 tokens, take 6 to 18 % less.
// Several micro-batches, up to eight workgroups a CU, don't move the line: each of 48 steps of 2, 4 and 8 (hidden 128 to 256, 32 to 2000
// tokens, up to 256 workgroups a micro-batch) takes 1 to 8 % less.  Rows of 320 to 512 columns (twice the registers and instructions): 0 to 3 % less where a micro-batch is
// alone, up to 11 % more for four of 200 and more tokens.
static bool can_norm(const GemmDesc* g, int n, const Route& r) {
    const bool ring = r.how == Route::RING;
    const Plan& p = ring ? r.group : r.each[0];
    if (n > RING_MAX || (n > 1 && !ring) || p.v != V_64x64 || g[0].K > NORM_K) return false;
    long w = 0;
    for (int i = 0; i < n; i++) {
        if (g[i].kind != GEMM_NT || g[i].A != g[0].A || g[i].K != g[0].K || g[i].M != g[0].M || g[i].lda != g[i].K || p.ksplit[i] > 1 || g[i].R || g[i].split) return false;
        w += tiles_of(g[i], VARIANTS[V_64x64]);
    }
    return w <= 256;
}
bool gemm_bf16_norms(const GemmDesc* g, int n) {
    Route r;
    route(g, n, r);
    return can_norm(g, n, r);
}

// The launches of problems of several micro-batches: launch(first problem, problems, plan) of each, until one fails.
template <typename L>
static hipError_t micro_launches(const GemmDesc* g, int n, const Route& r, L launch) {
    if (r.how == Route::RING) return launch(0, n, r.group);
    const Plan whole{WHOLE_DW, {1, 1, 1, 1}, {0, 1, 2, 3}, 0.0, 0};
    hipError_t e = hipSuccess;
    const int step = r.how == Route::TILES256 ? RING_MAX : 1;
    for (int i = 0; i < n && e == hipSuccess; i += step)
        e = launch(i, std::min(n - i, step), r.how == Route::TILES256 || r.each[i].v == V_DMA ? whole : r.each[i]);
    return e;
}

hipError_t gemm_bf16(const GemmDesc* g, int n, hipStream_t st) {
    if (n < 1 || n > DMA_MAX) return hipErrorInvalidValue;
    for (int i = 0; i < n; i++) {
        if (g[i].M <= 0 || g[i].N <= 0 || g[i].K <= 0) return hipErrorInvalidValue;
        const hipError_t e = check(g[i]);
        if (e != hipSuccess) return e;
        if ((g[i].kind == GEMM_NT) != (g[0].kind == GEMM_NT)) return hipErrorInvalidValue;
    }
    Route r;
    route(g, n, r);
    for (int i = 0; i < n; i++)   // several micro-batches, fusions: where gemm_bf16_on_ring says so
        if (g[i].micro < 1 || g[i].micro > MICRO_MAX || g[i].micro != g[0].micro || (g[i].micro > 1 && !g[i].each) ||
            ((g[i].micro > 1 || g[i].fuse.kind) && (r.how == Route::TILES256 || (r.how == Route::RING ? r.group.v : r.each[i].v) >= V_DMA) &&
             !(g[i].micro > 1 && whole_dw(g[i]))) ||
            (g[i].fuse.kind == FUSE_SWIGLU_BWD && n > 1) || (g[i].fuse.kind != g[0].fuse.kind) ||
            (g[i].fuse.kind && tile_size(r.how == Route::RING ? r.group.v : r.each[i].v) > fuse_tile(g[i].fuse.kind)) ||
            g[i].norm != g[0].norm)
            return hipErrorInvalidValue;
    if (g[0].norm && !can_norm(g, n, r)) return hipErrorInvalidValue;
    if (g[0].micro > 1) return micro_launches(g, n, r, [&](int i, int m, const Plan& p) { return launch_planned(g + i, m, p, st); });
    if (r.how == Route::RING) return launch_planned(g, n, r.group, st);
    if (r.how == Route::TILES256) return launch_tiles256(g, n, st);
    for (int i = 0; i < n; i++) {
        hipError_t e = hipSuccess;
        if (r.each[i].v == V_COUNT) {
            GemmDesc seg[3];
            const int m = segments(g[i], seg);
            for (int j = 0; j < m && e == hipSuccess; j++) e = launch_planned(seg + j, 1, plan(seg + j, 1, false), st);
        } else e = launch_planned(g + i, 1, r.each[i], st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace hh

// For tests, not part of the public interface: how problems of these sizes are launched, without launching them.  A problem
// is kind, M, N, K and the first k of B's second and third segment (0: none).  Writes a line for each of the n problems
// of a call: "<how> <tile> <k shares>", where <how> is `alone`, `ring` or `tiles256` (together, on that kernel) or
// `segments` (one after the other, no tile); of 256x256 tiles the shares are those of the last round on 256 CUs.
static hh::GemmDesc sizes_of(const int* q) {
    hh::GemmDesc g{};
    static char somewhere[16];
    g.kind = q[0]; g.M = q[1]; g.N = q[2]; g.K = q[3]; g.k1 = q[4]; g.k2 = q[5];
    g.B1 = g.B2 = somewhere;
    g.out_f32 = g.kind == hh::GEMM_TN;
    g.ws = somewhere; g.ws_bytes = hh::GEMM_WS_BYTES;
    g.micro = 1;
    return g;
}
extern "C" int hh_internal_gemm_plan(const int* problems, int n, char* out, size_t size) {
    using namespace hh;
    if (n < 1 || n > DMA_MAX) return -1;
    GemmDesc g[DMA_MAX];
    long tiles = 0;
    for (int i = 0; i < n; i++) {
        g[i] = sizes_of(problems + 6 * i);
        tiles += tiles_of(g[i], VARIANTS[V_DMA]);
    }
    Route r;
    route(g, n, r);
    size_t at = 0;
    for (int i = 0; i < n; i++) {
        const bool ring = r.how == Route::RING, together = r.how == Route::TILES256;
        const int v = ring ? r.group.v : together ? (int)V_DMA : r.each[i].v;
        const int shares = v == V_DMA ? tail_shares(g[i], (int)(together ? tiles : tiles_of(g[i], VARIANTS[V_DMA])), 256)
                         : v == V_COUNT ? 1 : ring ? r.group.ksplit[i] : r.each[i].ksplit[0];
        char tile[32] = "-";
        if (v < V_COUNT) snprintf(tile, sizeof tile, "%dx%d%s", VARIANTS[v].bm, VARIANTS[v].bn, v == V_128x128_2 ? "/2" : "");
        const int w = snprintf(out + at, size - at, "%s %s %d\n", ring ? "ring" : together ? "tiles256" : v == V_COUNT ? "segments" : "alone",
                               tile, shares);
        if (w < 0 || (size_t)w >= size - at) return -1;
        at += (size_t)w;
    }
    return 0;
}
// The weight gradients (bits) of a call for several micro-batches whose products are apart, with that much room for partial sums; -1
// where such a call is refused.
extern "C" int hh_internal_products_apart(const int* problems, int n, int micro, size_t room) {
    using namespace hh;
    if (n < 1 || n > DMA_MAX) return -1;
    GemmDesc g[DMA_MAX];
    for (int i = 0; i < n; i++) {
        g[i] = sizes_of(problems + 6 * i);
        g[i].micro = micro; g[i].ws_room = room;
    }
    RingUse use;
    if (!gemm_bf16_on_ring(g, n, &use)) return -1;
    Route r;
    route(g, n, r);
    int apart = 0;
    (void)micro_launches(g, n, r, [&](int i, int m, const Plan& p) {
        if (g[i].kind != GEMM_NT) apart |= (int)(micro_plan(g + i, m, p).apart << i);
        return hipSuccess;
    });
    return apart;
}
// Whether one launch of these problems, all NT on one A, norms its rows itself.
extern "C" int hh_internal_gemm_norms(const int* problems, int n) {
    using namespace hh;
    if (n < 1 || n > RING_MAX) return -1;
    GemmDesc g[RING_MAX];
    for (int i = 0; i < n; i++) {
        g[i] = sizes_of(problems + 6 * i);
        g[i].lda = g[i].K;
    }
    return gemm_bf16_norms(g, n);
}
// n / d as the kernels form it
extern "C" int hh_internal_quotient(int n, int d) { return hh::quotient(n, hh::divisor(d)); }
// Whether the weight gradients of a layer are left to one launch at the end: the problems of its three groups, n of each.
extern "C" int hh_internal_gemm_defer(const int* problems, const int* n) {
    using namespace hh;
    GemmDesc g[3][RING_MAX], dw[DMA_MAX];
    const GemmDesc* const groups[3] = {g[0], g[1], g[2]};
    int n_dw = 0;
    for (int i = 0; i < 3; i++) {
        if (n[i] < 1 || n[i] > RING_MAX) return -1;
        for (int j = 0; j < n[i]; j++, problems += 6) {
            g[i][j] = sizes_of(problems);
            if (j + 1 < n[i] && n_dw < DMA_MAX) dw[n_dw++] = g[i][j];
        }
    }
    return gemm_bf16_defer(dw, n_dw, groups, n);
}
