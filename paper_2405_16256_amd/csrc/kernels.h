// Host-side launchers of the gfx950 kernels (internal to the library).
// All pointers are device pointers; every launcher only enqueues on `st`.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace hh {

enum { DT_F32 = 0, DT_BF16 = 1 };
inline size_t dt_size(int dt) { return dt == DT_BF16 ? 2 : 4; }

// One operand of up to MICRO_MAX micro-batches that a launch takes side by side: its address in each of them.
constexpr int MICRO_MAX = 8;
struct Each { void* p[MICRO_MAX]; };

// C[M,N] (=|+=) op(A) op(B) (+ R), leading dimensions in elements.
//   GEMM_NT: A[M,K] row-major, B[N,K] row-major   (y = x W^T)
//   GEMM_NN: A[M,K] row-major, B[K,N] row-major   (dX = dY W)
//   GEMM_TN: A[K,M] row-major, B[K,N] row-major   (dW = dY^T X)
enum { GEMM_NT = 0, GEMM_NN = 1, GEMM_TN = 2 };
// The operands of a problem that the launch repeats for several micro-batches (weight gradients: C is the same in all of
// them and their products are added in the order of the micro-batches, each as a launch of its own would add it).
struct GemmMicro { Each A, B, C, R, X, Y; };
// What a GEMM (in bf16 the ring kernel) can do with a product before it is written, in place of a launch of its own:
//   FUSE_ROPE       NT, C = q|k|v rows or a part of them: the rotary embedding of the first `rot` columns, heads of `period`
//   FUSE_SWIGLU     NT, C = gate|up rows [M, period]: X [M, period/2] = silu(gate) * up
//   FUSE_SWIGLU_BWD NN, the product is dm [M, N]: with X = gate|up, C = m and Y = dgate|dup
// Each on the product rounded to the storage type, as the launch would read it.
enum { FUSE_NONE = 0, FUSE_ROPE, FUSE_SWIGLU, FUSE_SWIGLU_BWD };
// The largest tile (rows x columns) on which the ring kernel does it.
constexpr int fuse_tile(int kind) { return kind == FUSE_ROPE ? 192 * 128 : kind == FUSE_SWIGLU ? 128 * 128 : 64 * 128; }
struct GemmFuse {
    int kind;
    int period, rot;
    int seq, table_seq; const float* table;   // FUSE_ROPE: as for rope()
    void* X; void* Y;
};
// Partial sums of an NT or NN problem that its launch has left to the kernel that reads the result: fp32 tiles
// [tile][micro-batch][share][bm*bn], to be added in the order of the shares (then the residual) and rounded.
struct GemmSplit { const float* partial; int ksplit, bm, bn, tiles_n; };
// The launch leaves at most SPLIT_ROW of them for a row, in two shares or more: rows of at most SPLIT_COLUMNS columns.
constexpr int SPLIT_ROW = 16384, SPLIT_COLUMNS = SPLIT_ROW / 2;
// The RMSNorm of the rows of A on the way into an NT launch: xn and r (of each micro-batch) are written beside the product.
struct GemmNorm { Each xn, r; const void* gain; float eps; };
constexpr int NORM_K = 256;
struct GemmDesc {
    int kind;
    int M, N, K;
    const void* A; int lda;
    const void* B; int ldb;
    void* C; int ldc;
    const void* R; int ldr;  // optional residual in the storage dtype, added before rounding (NULL: none)
    int out_f32;             // 1: C is fp32 regardless of the storage dtype (parameter gradients)
    int accumulate;          // 1: C += result
    // B of an NN problem in up to three allocations: rows k1.. at B1, rows k2.. at B2 (0: no such segment)
    const void* B1; int k1;
    const void* B2; int k2;
    void* ws;                // optional scratch for k-split partial sums (bf16 path), may be NULL
    size_t ws_bytes;         // of one micro-batch: what a plan may use
    size_t ws_room;          // micro > 1: what there is for all of them
    GemmFuse fuse;
    GemmSplit* split;        // not null: the launch may leave its partial sums (ksplit > 1 then, else C is complete)
    const GemmNorm* norm;    // not null (bf16, where gemm_bf16_norms): A holds x, and xn takes its place; one for a launch
    int micro;               // micro-batches; above 1 (bf16: where gemm_bf16_on_ring) their operands are in `each`
    const GemmMicro* each;
};
constexpr size_t GEMM_WS_BYTES = (size_t)64 << 20;   // enough for 256 partial tiles of 256x256 fp32

// The library's own scratch array (one per GPU, held until the process ends) and its size.
constexpr size_t STATIC_SCRATCH_BYTES = (size_t)128 << 20;
hipError_t static_scratch_init(int device);   // `device` must be current; looks the array's address up once
void* static_scratch(int device);             // that address (null before a successful init)
// Up to 4 problems (8 weight gradients in bf16) of which none reads what another writes, either all NT or none; they share launches where that is
// predicted to be faster.
hipError_t gemm(int dtype, const GemmDesc* g, int n, hipStream_t st);
// Whether all launches of these problems (bf16) are the ring kernel's, and if so: the bytes of partial sums that the largest of
// those launches keeps, its workgroups, and the largest tile.
struct RingUse { size_t partial; long workgroups; int tile; };
bool gemm_bf16_on_ring(const GemmDesc* g, int n, RingUse* use);
// Whether one launch of these problems (NT, one A) can norm the rows of A, and had better.
bool gemm_bf16_norms(const GemmDesc* g, int n);
// Whether they do; if not, gemm() on each of them alone launches the same.
bool gemm_shares_launch(int dtype, const GemmDesc* g, int n);

// xn = x * r * g, r = 1/sqrt(mean(x^2)+eps) per row.
// Here and below: micro-batches 0 .. n-1 side by side, an operand's address in each of them; the result of a micro-batch
// does not depend on n.
// split (bf16): x has yet to be summed (with the residual `res`) and written.
hipError_t rmsnorm_fwd(int dtype, const Each& x, const void* g, const Each& xn, const Each& r,
                       int n, int T, int H, float eps, hipStream_t st, const GemmSplit* split = nullptr, const Each* res = nullptr);
// dx = dres + r*(w - u*mean(w*u)), u = x*r, w = dxn*g; per-workgroup column sums of
// dxn*u go to partial[rmsnorm_bwd_blocks(T, H, partial_bytes)][H].
int rmsnorm_bwd_blocks(int T, int H, size_t partial_bytes);
hipError_t rmsnorm_bwd(int dtype, const Each& dxn, const Each& x, const Each& r, const void* g,
                       const Each& dres, const Each& dx, const Each& partial, size_t partial_bytes, int n, int T, int H, hipStream_t st,
                       const GemmSplit* split = nullptr,   // bf16: in place of dxn
                       float* gain = nullptr, int accumulate = 0);   // gain: gradient of g, written (+=) here; no partial sums then
// Whether rmsnorm_bwd had better write the gain's gradient itself (where nothing it reads is written by it).
bool rmsnorm_bwd_sums_gain(int T, int H, const GemmSplit* split);
// out[H] (=|+=) column sums of partial[rows][H], of one micro-batch after the other; one or two such sums in one launch
struct ColSum { Each partial; int rows; float* out; };
hipError_t colsum_reduce(const ColSum* jobs, int n_jobs, int n, int H, int accumulate, hipStream_t st);

// In-place rotary embedding of the first nrot heads (query heads, then key heads) of every row of a
// [T, ld] buffer.  table = cos[table_seq][d/2] followed by sin[table_seq][d/2], table_seq >= S.  (The backward rotation is
// part of attn_bwd.)
hipError_t rope(int dtype, const Each& qkv, int ld, int n, int T, int S, int nrot, int d, const float* table, int table_seq,
                hipStream_t st);

// gu[T,2F] = (gate | up);  m = silu(gate)*up
hipError_t swiglu_fwd(int dtype, const Each& gu, const Each& m, int n, int T, int F, hipStream_t st);
// dgu[T,2F] = (dgate | dup), and m recomputed
hipError_t swiglu_bwd(int dtype, const Each& dm, const Each& gu, const Each& dgu, const Each& m, int n, int T, int F, hipStream_t st);

// Causal attention over a [T, ld] buffer holding q | k | v column blocks of width nh*d, nkv*d, nkv*d;
// query head h uses key/value head h / (nh / nkv).  o [T, nh*d]; lse [B, nh, S] natural-log sum-exp of
// the scaled scores.
// micro.n micro-batches side by side, micro.saved bytes apart in qkv, o and lse, micro.ws bytes in dout, dvec, dqkv and
// scratch; how a micro-batch is split over workgroups does not depend on micro.n.
struct MicroStride { int n; size_t saved, ws; };
hipError_t attn_fwd(int dtype, const void* qkv, int ld, void* o, float* lse,
                    int B, int S, int nh, int nkv, int d, const MicroStride& micro, hipStream_t st);
// dqkv [T, ld] receives dq | dk | dv in the same layout.  dvec: scratch [B, nh, S] floats.  scratch: device
// memory of scratch_bytes, at least attn_bwd_scratch_bytes() (partial dK, dV sums when the query heads that share a
// key/value head are spread over several workgroups; may be null when it has no bytes; the fp32 path needs none and
// spreads the heads as far as what it is given reaches).  rope_table (as for rope(), rope_seq >= S;
// null: none): q and k were rotated before the forward call, and dq, dk are written as gradients of the
// unrotated q, k (the backward rotation applied before the one rounding to the storage type).
size_t attn_bwd_scratch_bytes(int dtype, int B, int S, int nh, int nkv, int d);
hipError_t attn_bwd(int dtype, const void* qkv, int ld, const void* o, const void* dout, const float* lse,
                    float* dvec, void* dqkv, void* scratch, size_t scratch_bytes, int B, int S, int nh, int nkv, int d,
                    const float* rope_table, int rope_seq, const MicroStride& micro, hipStream_t st);

}  // namespace hh
