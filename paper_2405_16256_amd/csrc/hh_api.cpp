// C ABI of the decoder-stage library: argument validation, buffer carving and
// the order in which the gfx950 kernels are enqueued.  No numeric work happens
// on the host except the rotary cos/sin table (built once per context).
#include "../../include/hh.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <memory>
#include <new>
#include <vector>

#include "kernels.h"

namespace hh {
hipError_t gemm_bf16(const GemmDesc* g, int n, hipStream_t st);
bool gemm_bf16_shares_launch(const GemmDesc* g, int n);
bool gemm_bf16_defer(const GemmDesc* dw, int n_dw, const GemmDesc* const groups[3], const int n[3]);
hipError_t gemm_f32(const GemmDesc* g, int n, hipStream_t st);
hipError_t attn_bf16_fwd(const void* qkv, int ld, void* o, float* lse, int B, int S, int nh, int nkv, int d, const MicroStride& micro,
                         hipStream_t st);
hipError_t attn_bf16_bwd(const void* qkv, int ld, const void* o, const void* dout, const float* lse, float* dvec,
                         void* dqkv, float* scratch, int B, int S, int nh, int nkv, int d,
                         const float* rope, int rope_seq, const MicroStride& micro, hipStream_t st);
size_t attn_bf16_bwd_scratch_bytes(int B, int S, int nh, int nkv, int d);
hipError_t attn_f32_fwd(const void* qkv, int ld, void* o, float* lse, int B, int S, int nh, int nkv, int d, const MicroStride& micro,
                        hipStream_t st);
hipError_t attn_f32_bwd(const void* qkv, int ld, const void* o, const void* dout, const float* lse, float* dvec,
                        void* dqkv, float* scratch, size_t scratch_bytes, int B, int S, int nh, int nkv, int d,
                        const float* rope, int rope_seq, const MicroStride& micro, hipStream_t st);

hipError_t gemm(int dtype, const GemmDesc* g, int n, hipStream_t st) {
    if (dtype == DT_BF16) return gemm_bf16(g, n, st);
    // the later segments of B one after the other behind the group, each adding to what the ones before it have left in C
    GemmDesc q[4];
    if (n < 1 || n > 4) return hipErrorInvalidValue;
    for (int i = 0; i < n; i++) {
        q[i] = g[i];
        if (q[i].k1) q[i].K = q[i].k1;
        q[i].k1 = q[i].k2 = 0;
    }
    hipError_t e = gemm_f32(q, n, st);
    for (int i = 0; i < n; i++) {
        const int at[3] = {g[i].k1, g[i].k2 ? g[i].k2 : g[i].K, g[i].K};
        const void* const b[2] = {g[i].B1, g[i].B2};
        for (int s = 0; s < 2 && g[i].k1 && at[s] < g[i].K && e == hipSuccess; s++) {
            GemmMicro each{};
            q[i].A = (const float*)g[i].A + at[s];
            q[i].B = b[s];
            q[i].K = at[s + 1] - at[s];
            q[i].R = g[i].C; q[i].ldr = g[i].ldc;
            for (int m = 0; m < g[i].micro && g[i].micro > 1; m++) {
                each.A.p[m] = (float*)g[i].each->A.p[m] + at[s];
                each.B.p[m] = const_cast<void*>(b[s]);
                each.C.p[m] = each.R.p[m] = g[i].each->C.p[m];
                q[i].each = &each;
            }
            e = gemm_f32(q + i, 1, st);
        }
    }
    return e;
}
bool gemm_shares_launch(int dtype, const GemmDesc* g, int n) { return dtype == DT_BF16 ? gemm_bf16_shares_launch(g, n) : n > 1; }
hipError_t attn_fwd(int dtype, const void* qkv, int ld, void* o, float* lse, int B, int S, int nh, int nkv, int d, const MicroStride& micro,
                    hipStream_t st) {
    return dtype == DT_BF16 ? attn_bf16_fwd(qkv, ld, o, lse, B, S, nh, nkv, d, micro, st) : attn_f32_fwd(qkv, ld, o, lse, B, S, nh, nkv, d, micro, st);
}
size_t attn_bwd_scratch_bytes(int dtype, int B, int S, int nh, int nkv, int d) {
    return dtype == DT_BF16 ? attn_bf16_bwd_scratch_bytes(B, S, nh, nkv, d) : 0;
}
hipError_t attn_bwd(int dtype, const void* qkv, int ld, const void* o, const void* dout, const float* lse, float* dvec,
                    void* dqkv, void* scratch, size_t scratch_bytes, int B, int S, int nh, int nkv, int d,
                    const float* rope_table, int rope_seq, const MicroStride& micro, hipStream_t st) {
    if (dtype == DT_BF16) return attn_bf16_bwd(qkv, ld, o, dout, lse, dvec, dqkv, (float*)scratch, B, S, nh, nkv, d, rope_table, rope_seq, micro, st);
    return attn_f32_bwd(qkv, ld, o, dout, lse, dvec, dqkv, (float*)scratch, scratch_bytes, B, S, nh, nkv, d, rope_table, rope_seq, micro, st);
}
}  // namespace hh

using namespace hh;
static_assert(HH_STATIC_SCRATCH_BYTES == STATIC_SCRATCH_BYTES, "the header states the size of the library's scratch array");

// ------------------------------------------------------------------ errors
static thread_local char g_err[512] = "";

static int fail(int code, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return code;
}
static int hip_fail(hipError_t e, const char* what) {
    return fail(HH_ERR_DEVICE, "%s: %s", what, hipGetErrorString(e));
}
#define HIP_TRY(call)                                        \
    do {                                                     \
        hipError_t e_ = (call);                              \
        if (e_ != hipSuccess) return hip_fail(e_, #call);    \
    } while (0)

extern "C" const char* hh_last_error(void) { return g_err; }
namespace hh {
// for the other translation units of the library
int set_error(int code, const char* msg) { return fail(code, "%s", msg); }
}  // namespace hh

// ------------------------------------------------------------------ context
struct TraceRec {
    hipEvent_t a, b;
    int kind;
    double work;
    size_t events;  // the record whose events bracket the launch (its own, unless GEMMs share one)
    double share;   // of the time between them that is this family's
    int count;      // micro-batches that the launch takes side by side: it stands for a launch of each
};
struct hh_ctx {
    int device;
    float* rope_table;  // device: cos[S][d/2] then sin[S][d/2]
    int rope_seq, rope_dim;
    float rope_base;
    std::vector<TraceRec> trace;  // events created by hh_trace_begin
    size_t trace_used;
    bool trace_on;
    uint32_t trace_mask;          // families recorded while trace_on
    void* gemm_ws;                // k-split scratch inside the caller's workspace, set by each hot call
    size_t gemm_room;             // its bytes where several micro-batches go side by side, set by each such call
    std::vector<float*> retired_tables;   // rotary tables replaced by a larger one: freed with the context
};

extern "C" int hh_ctx_create(hh_ctx** out, int device) {
    if (!out) return fail(HH_ERR_INVALID_ARG, "hh_ctx_create: out is NULL");
    *out = nullptr;
    int n = 0;
    hipError_t e = hipGetDeviceCount(&n);
    if (e != hipSuccess) return hip_fail(e, "hipGetDeviceCount");
    if (device < 0 || device >= n) return fail(HH_ERR_DEVICE, "hh_ctx_create: no HIP device %d (%d visible)", device, n);
    // the library's own scratch array lives at a different address on every GPU: look this GPU's up now
    int prev = 0;
    e = hipGetDevice(&prev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    e = hipSetDevice(device);
    if (e != hipSuccess) return hip_fail(e, "hipSetDevice");
    e = static_scratch_init(device);
    (void)hipSetDevice(prev);
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    hh_ctx* c = new (std::nothrow) hh_ctx{device, nullptr, 0, 0, 0.f, {}, 0, false, 0u, nullptr, {}};
    if (!c) return fail(HH_ERR_INVALID_ARG, "hh_ctx_create: out of host memory");
    *out = c;
    return HH_OK;
}

extern "C" int hh_ctx_destroy(hh_ctx* ctx) {
    if (!ctx) return HH_OK;
    if (ctx->rope_table) (void)hipFree(ctx->rope_table);
    for (float* t : ctx->retired_tables) (void)hipFree(t);
    for (auto& r : ctx->trace) { (void)hipEventDestroy(r.a); (void)hipEventDestroy(r.b); }
    delete ctx;
    return HH_OK;
}

// ---------------------------------------------------------------- validation
static int check_cfg(const hh_layer_cfg* c) {
    if (!c) return fail(HH_ERR_INVALID_ARG, "cfg is NULL");
    if (c->dtype != HH_F32 && c->dtype != HH_BF16) return fail(HH_ERR_INVALID_ARG, "cfg.dtype %d is not HH_F32/HH_BF16", c->dtype);
    if (c->hidden <= 0 || c->n_heads <= 0 || c->head_dim <= 0 || c->ffn <= 0 || c->seq <= 0 || c->micro_batch <= 0)
        return fail(HH_ERR_INVALID_ARG, "cfg has a non-positive dimension");
    if (!(c->rms_eps >= 0.f) || !(c->rope_base > 0.f)) return fail(HH_ERR_INVALID_ARG, "cfg.rms_eps must be >= 0 and rope_base > 0");
    if (c->n_kv_heads <= 0 || c->n_heads % c->n_kv_heads)
        return fail(HH_ERR_UNSUPPORTED_SHAPE, "n_kv_heads (%d) must be positive and divide n_heads (%d)", c->n_kv_heads, c->n_heads);
    if (c->head_dim != 64 && c->head_dim != 128) return fail(HH_ERR_UNSUPPORTED_SHAPE, "head_dim %d: only 64 and 128", c->head_dim);
    const int mult = c->dtype == HH_BF16 ? 64 : 8;
    const long A = (long)c->n_heads * c->head_dim;   // the kv width n_kv_heads*head_dim is a multiple of 64 as well
    if (c->hidden % mult || A % mult || c->ffn % mult)
        return fail(HH_ERR_UNSUPPORTED_SHAPE, "hidden, n_heads*head_dim and ffn must be multiples of %d for this dtype", mult);
    if (c->hidden > 32768) return fail(HH_ERR_UNSUPPORTED_SHAPE, "hidden %d exceeds 32768", c->hidden);
    // The kernels address every buffer with 32-bit byte offsets: outputs below 2^31 bytes, GEMM operands below
    // 2^32 - 2^25.  Packed q|k|v and gate|up gradients that would be larger are written part by part (see the
    // backward), so only the single projections bound the fp32 gradients.
    const long es = c->dtype == HH_BF16 ? 2 : 4;
    const long T = (long)c->seq * c->micro_batch;
    const long Q3 = A + 2L * c->n_kv_heads * c->head_dim;
    const long wide = std::max<long>(std::max<long>(c->hidden, Q3), 2L * c->ffn);
    if (wide > 65535) return fail(HH_ERR_UNSUPPORTED_SHAPE, "a row of %ld elements exceeds 65535", wide);
    if (T * wide * es >= (1L << 31))
        return fail(HH_ERR_UNSUPPORTED_SHAPE, "an activation of %ld x %ld elements reaches 2^31 bytes", T, wide);
    if ((long)c->hidden * std::max<long>(A, c->ffn) * 4 >= (1L << 31))
        return fail(HH_ERR_UNSUPPORTED_SHAPE, "the fp32 gradient of one projection reaches 2^31 bytes");
    if ((long)c->hidden * wide * es >= (1L << 32) - (1L << 25))
        return fail(HH_ERR_UNSUPPORTED_SHAPE, "a packed weight of %d x %ld elements reaches 2^32 bytes", c->hidden, wide);
    return HH_OK;
}

static int check_ptr(const void* p, const char* name) {
    if (!p) return fail(HH_ERR_INVALID_ARG, "%s is NULL", name);
    if ((uintptr_t)p & 15) return fail(HH_ERR_MISALIGNED, "%s is not 16-byte aligned", name);
    return HH_OK;
}
#define TRY(x)                \
    do {                      \
        int rc_ = (x);        \
        if (rc_ != HH_OK) return rc_; \
    } while (0)

static int check_weights(const hh_layer_weights* w) {
    if (!w) return fail(HH_ERR_INVALID_ARG, "weights is NULL");
    TRY(check_ptr(w->g_attn, "weights.g_attn")); TRY(check_ptr(w->wq, "weights.wq")); TRY(check_ptr(w->wk, "weights.wk"));
    TRY(check_ptr(w->wv, "weights.wv")); TRY(check_ptr(w->wo, "weights.wo")); TRY(check_ptr(w->g_mlp, "weights.g_mlp"));
    TRY(check_ptr(w->w_gate, "weights.w_gate")); TRY(check_ptr(w->w_up, "weights.w_up")); TRY(check_ptr(w->w_down, "weights.w_down"));
    return HH_OK;
}
static int check_grads(const hh_layer_grads* g) {
    if (!g) return fail(HH_ERR_INVALID_ARG, "grads is NULL");
    TRY(check_ptr(g->g_attn, "grads.g_attn")); TRY(check_ptr(g->wq, "grads.wq")); TRY(check_ptr(g->wk, "grads.wk"));
    TRY(check_ptr(g->wv, "grads.wv")); TRY(check_ptr(g->wo, "grads.wo")); TRY(check_ptr(g->g_mlp, "grads.g_mlp"));
    TRY(check_ptr(g->w_gate, "grads.w_gate")); TRY(check_ptr(g->w_up, "grads.w_up")); TRY(check_ptr(g->w_down, "grads.w_down"));
    return HH_OK;
}

// ------------------------------------------------------------ buffer layouts
static inline size_t up256(size_t n) { return (n + 255) & ~(size_t)255; }

struct Dims {
    int T, H, A, Akv, Q3, F, S, B, nh, nkv, d, dt;   // Akv = nkv*d; Q3 = A + 2*Akv: width of a q|k|v row
    size_t es;
};
static Dims dims_of(const hh_layer_cfg* c) {
    Dims d;
    d.S = c->seq; d.B = c->micro_batch; d.T = c->seq * c->micro_batch; d.H = c->hidden; d.nh = c->n_heads; d.d = c->head_dim;
    d.A = c->n_heads * c->head_dim; d.nkv = c->n_kv_heads; d.Akv = d.nkv * d.d; d.Q3 = d.A + 2 * d.Akv; d.F = c->ffn; d.dt = c->dtype == HH_BF16 ? DT_BF16 : DT_F32; d.es = dt_size(d.dt);
    return d;
}

struct SavedLayout {
    size_t xn, qkv, a, h, hn, gu, lse, r1, r2, total;
};
static SavedLayout saved_layout(const Dims& d) {
    SavedLayout s;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += up256(bytes); return o; };
    const size_t T = d.T;
    s.xn = take(T * d.H * d.es);
    s.qkv = take(T * d.Q3 * d.es);
    s.a = take(T * d.A * d.es);
    s.h = take(T * d.H * d.es);
    s.hn = take(T * d.H * d.es);
    s.gu = take(T * 2 * d.F * d.es);
    s.lse = take((size_t)d.B * d.nh * d.S * 4);
    s.r1 = take(T * 4);
    s.r2 = take(T * 4);
    s.total = off;
    return s;
}

struct WorkLayout {
    size_t m, dgu, dhn, dh, da, dqkv, dvec, dkv_part, partial, gemm_ws, total;
};
static WorkLayout work_layout(const Dims& d) {
    WorkLayout w;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += up256(bytes); return o; };
    const size_t T = d.T;
    w.m = take(T * d.F * d.es);            // forward: m; backward: dm, then m recomputed in place
    w.dgu = take(T * 2 * d.F * d.es);
    w.dhn = take(T * d.H * d.es);          // d(hn), later d(xn)
    w.dh = take(T * d.H * d.es);
    w.da = take(T * d.A * d.es);
    w.dqkv = take(T * d.Q3 * d.es);
    w.dvec = take((size_t)d.B * d.nh * d.S * 4);
    w.dkv_part = take(attn_bwd_scratch_bytes(d.dt, d.B, d.S, d.nh, d.nkv, d.d));   // partial dK, dV of grouped heads
    int rows = 8;                          // gain-gradient partials: one row per `rows` tokens, at most 256
    while ((d.T + rows - 1) / rows > 256) rows *= 2;
    w.partial = take((size_t)((d.T + rows - 1) / rows) * d.H * 4);
    w.gemm_ws = take(d.dt == DT_BF16 ? GEMM_WS_BYTES : 0);
    w.total = off;
    return w;
}

// The same for one of several micro-batches that go side by side: both sets of gain-gradient partials have a place of their own
// (`partial`, two times gain_bytes), and the GEMMs' scratch is not part of it.  Packed closer unless a layer defers its weight
// gradients: what the attention branch's backward needs takes the place of m and dgate|dup, whose last readers are the weight
// gradients of the MLP, and deferred ones read them at the very end.
static size_t gain_bytes(const Dims& d) { return (size_t)std::min(d.T, 256) * d.H * 4; }
static WorkLayout side_layout(const Dims& d, bool defers) {
    const WorkLayout one = work_layout(d);
    if (d.dt != DT_BF16) return one;   // whose attention keeps its partial sums in m | dgate|dup | d(hn)
    WorkLayout w = one;
    if (!defers) {
        w.da = w.m;
        w.dqkv = w.da + (one.dqkv - one.da);
        w.dvec = w.dqkv + (one.dvec - one.dqkv);
        w.dkv_part = w.dvec + (one.dkv_part - one.dvec);
        w.dhn = std::max(one.dhn, w.dkv_part + (one.partial - one.dkv_part));
        w.dh = w.dhn + (one.dh - one.dhn);
        w.partial = w.dh + (one.da - one.dh);
    }
    w.gemm_ws = w.total = w.partial + 2 * up256(gain_bytes(d));
    return w;
}

extern "C" int hh_layer_sizes(const hh_layer_cfg* cfg, size_t* saved_bytes, size_t* workspace_bytes) {
    TRY(check_cfg(cfg));
    const Dims d = dims_of(cfg);
    if (saved_bytes) *saved_bytes = saved_layout(d).total;
    if (workspace_bytes) *workspace_bytes = work_layout(d).total;
    return HH_OK;
}

extern "C" int hh_saved_layout_of(const hh_layer_cfg* cfg, hh_saved_layout* out) {
    TRY(check_cfg(cfg));
    if (!out) return fail(HH_ERR_INVALID_ARG, "out is NULL");
    const SavedLayout s = saved_layout(dims_of(cfg));
    out->xn = s.xn; out->qkv = s.qkv; out->a = s.a; out->h = s.h; out->hn = s.hn; out->gate_up = s.gu;
    out->lse = s.lse; out->r1 = s.r1; out->r2 = s.r2; out->total = s.total;
    return HH_OK;
}

static size_t act_bytes(const Dims& d) { return up256((size_t)d.T * d.H * d.es); }

extern "C" int hh_stage_sizes(const hh_layer_cfg* cfg, int n_layers, int n_micro, size_t* saved_pool_bytes,
                              size_t* workspace_bytes) {
    TRY(check_cfg(cfg));
    if (n_layers <= 0 || n_micro <= 0) return fail(HH_ERR_INVALID_ARG, "n_layers and n_micro must be positive");
    const Dims d = dims_of(cfg);
    const size_t per_micro = (size_t)n_layers * saved_layout(d).total + (size_t)(n_layers - 1) * act_bytes(d);
    if (saved_pool_bytes) *saved_pool_bytes = per_micro * (size_t)n_micro;
    if (workspace_bytes) *workspace_bytes = work_layout(d).total + act_bytes(d);  // + the gradient passed between layers
    return HH_OK;
}

extern "C" int hh_layer_flops(const hh_layer_cfg* cfg, double* fwd_flop, double* bwd_flop) {
    TRY(check_cfg(cfg));
    const Dims d = dims_of(cfg);
    const double T = d.T;
    const double gemm = T * (2.0 * (d.Q3 + d.A) * d.H + 6.0 * (double)d.H * d.F);
    const double attn = 4.0 * d.d * d.B * d.nh * ((double)d.S * (d.S + 1) / 2);
    if (fwd_flop) *fwd_flop = gemm + attn;
    if (bwd_flop) *bwd_flop = 2.0 * (gemm + attn);
    return HH_OK;
}

// ------------------------------------------------------------- rotary table
static int ensure_rope(hh_ctx* ctx, const hh_layer_cfg* c) {
    if (ctx->rope_table && ctx->rope_seq >= c->seq && ctx->rope_dim == c->head_dim && ctx->rope_base == c->rope_base) return HH_OK;
    HIP_TRY(hipSetDevice(ctx->device));
    if (ctx->rope_table) {
        // launches already enqueued, and graphs recorded earlier, still read the old table: it stays alive
        // until the context is destroyed
        ctx->retired_tables.push_back(ctx->rope_table);
        ctx->rope_table = nullptr;
    }
    const int S = c->seq, half = c->head_dim / 2;
    std::vector<float> host((size_t)2 * S * half);
    for (int i = 0; i < half; i++) {
        const double theta = std::pow((double)c->rope_base, -2.0 * i / c->head_dim);
        for (int s = 0; s < S; s++) {
            const double phi = s * theta;
            host[(size_t)s * half + i] = (float)std::cos(phi);
            host[(size_t)S * half + (size_t)s * half + i] = (float)std::sin(phi);
        }
    }
    HIP_TRY(hipMalloc((void**)&ctx->rope_table, host.size() * sizeof(float)));
    HIP_TRY(hipMemcpy(ctx->rope_table, host.data(), host.size() * sizeof(float), hipMemcpyHostToDevice));
    ctx->rope_seq = S; ctx->rope_dim = c->head_dim; ctx->rope_base = c->rope_base;
    return HH_OK;
}

extern "C" int hh_ctx_reserve(hh_ctx* ctx, const hh_layer_cfg* cfg) {
    TRY(check_cfg(cfg));
    if (!ctx) return fail(HH_ERR_INVALID_ARG, "ctx is NULL");
    return ensure_rope(ctx, cfg);
}

// ------------------------------------------------------------------ tracing
// When tracing is on, every kernel-family launch is bracketed by two events on the
// launch stream; hh_trace_end turns them into per-family time and work sums.
struct Traced {
    hh_ctx* ctx; hipStream_t st; TraceRec* rec;
    Traced(hh_ctx* c, hipStream_t s, int kind, int count, double work) : ctx(c), st(s), rec(nullptr) {
        if (c->trace_on && ((c->trace_mask >> kind) & 1u) && c->trace_used < c->trace.size()) {
            rec = &c->trace[c->trace_used++];
            rec->kind = kind; rec->work = work * count; rec->events = ctx->trace_used - 1; rec->share = 1.0; rec->count = count;
            (void)hipEventRecord(rec->a, st);
        }
    }
    ~Traced() { if (rec) (void)hipEventRecord(rec->b, st); }
};
#define TR(kind, work, call)                     \
    do {                                         \
        Traced t_(ctx, st, (kind), p.n, (double)(work)); \
        HIP_TRY(call);                           \
    } while (0)
static double attn_flop(const Dims& d) { return 4.0 * d.d * d.B * d.nh * ((double)d.S * (d.S + 1) / 2); }
static double gemm_flop(const GemmDesc& g) { return 2.0 * g.M * g.N * g.K * g.micro; }
static void gemm_scratch(const hh_ctx* ctx, GemmDesc& g) { g.ws = ctx->gemm_ws; g.ws_bytes = ctx->gemm_ws ? GEMM_WS_BYTES : 0; g.ws_room = ctx->gemm_room; }
// A group of GEMMs in one call.  Where they share a launch it is bracketed once and its time shared out to the members by
// their flops; members with launches of their own are traced (and launched, in the same way) one by one.
static hipError_t tgemm(hh_ctx* ctx, int dt, GemmDesc* g, int n, hipStream_t st) {
    double total = 0.0;
    for (int i = 0; i < n; i++) {
        gemm_scratch(ctx, g[i]);
        total += gemm_flop(g[i]);
    }
    if (n > 1 && ctx->trace_on && !gemm_shares_launch(dt, g, n)) {
        hipError_t e = hipSuccess;
        for (int i = 0; i < n && e == hipSuccess; i++) e = tgemm(ctx, dt, g + i, 1, st);
        return e;
    }
    const size_t first = ctx->trace_used;
    for (int i = 0; i < n; i++) {
        if (!(ctx->trace_on && ((ctx->trace_mask >> g[i].kind) & 1u) && ctx->trace_used < ctx->trace.size())) continue;
        TraceRec& r = ctx->trace[ctx->trace_used++];
        r.kind = g[i].kind; r.work = gemm_flop(g[i]); r.events = first; r.share = r.work / total; r.count = g[i].micro;
    }
    const bool traced = ctx->trace_used > first;
    if (traced) (void)hipEventRecord(ctx->trace[first].a, st);
    const hipError_t e = gemm(dt, g, n, st);
    if (traced) (void)hipEventRecord(ctx->trace[first].b, st);
    return e;
}
static hipError_t tgemm(hh_ctx* ctx, int dt, GemmDesc g, hipStream_t st) { return tgemm(ctx, dt, &g, 1, st); }

extern "C" int hh_trace_begin(hh_ctx* ctx, int max_launches, uint32_t kind_mask) {
    if (!ctx) return fail(HH_ERR_INVALID_ARG, "ctx is NULL");
    if (max_launches <= 0) return fail(HH_ERR_INVALID_ARG, "max_launches must be positive");
    HIP_TRY(hipSetDevice(ctx->device));
    while ((int)ctx->trace.size() < max_launches) {
        TraceRec r{nullptr, nullptr, 0, 0.0, 0, 1.0, 1};
        HIP_TRY(hipEventCreate(&r.a));
        hipError_t e = hipEventCreate(&r.b);
        if (e != hipSuccess) { (void)hipEventDestroy(r.a); return hip_fail(e, "hipEventCreate"); }
        ctx->trace.push_back(r);
    }
    ctx->trace_used = 0;
    ctx->trace_mask = kind_mask;
    ctx->trace_on = true;
    return HH_OK;
}

extern "C" int hh_trace_end(hh_ctx* ctx, hh_trace_sum* out, int n_kinds) {
    if (!ctx || !out) return fail(HH_ERR_INVALID_ARG, "ctx or out is NULL");
    if (n_kinds <= 0) return fail(HH_ERR_INVALID_ARG, "n_kinds must be positive");
    ctx->trace_on = false;
    for (int k = 0; k < n_kinds; k++) { out[k].kind = k; out[k].launches = 0; out[k].ms = 0.0; out[k].work = 0.0; }
    for (size_t i = 0; i < ctx->trace_used; i++) {
        const TraceRec& r = ctx->trace[i];
        const TraceRec& ev = ctx->trace[r.events];
        HIP_TRY(hipEventSynchronize(ev.b));
        float ms = 0.f;
        HIP_TRY(hipEventElapsedTime(&ms, ev.a, ev.b));
        if (r.kind < n_kinds) { out[r.kind].launches += r.count; out[r.kind].ms += ms * r.share; out[r.kind].work += r.work; }
    }
    ctx->trace_used = 0;
    return HH_OK;
}

// ------------------------------------------------------------ layer forward
static inline char* at(void* base, size_t off) { return (char*)base + off; }
static inline const char* at(const void* base, size_t off) { return (const char*)base + off; }

static GemmDesc desc(int kind, int M, int N, int K, const void* A, int lda, const void* B, int ldb, void* C, int ldc,
                     const void* R = nullptr, int ldr = 0, int out_f32 = 0, int acc = 0) {
    GemmDesc g;
    g.kind = kind; g.M = M; g.N = N; g.K = K; g.A = A; g.lda = lda; g.B = B; g.ldb = ldb; g.C = C; g.ldc = ldc;
    g.R = R; g.ldr = ldr; g.out_f32 = out_f32; g.accumulate = acc; g.ws = nullptr; g.ws_bytes = 0;
    g.B1 = g.B2 = nullptr; g.k1 = g.k2 = 0;
    g.fuse = GemmFuse{}; g.split = nullptr; g.norm = nullptr;
    g.micro = 1; g.each = nullptr;
    return g;
}

// The micro-batches that a pass takes through its launches side by side.  Their pool slots lie `pool_stride` bytes apart and
// their workspaces `ws_stride`; the boundary tensors are wherever the caller has them.  The code below names the addresses of
// the first micro-batch; at() gives those of the others.
struct Pass {
    int n;
    const WorkLayout* side;   // how the workspaces are laid out (null: work_layout)
    const char* pool; size_t pool_stride;
    const char* ws; size_t ws_stride;
    const void* const* x; void* const* y;
    const void* const* dy; void* const* dx;
    void* at(const void* p, int m) const {
        const char* c = (const char*)p;
        if (m == 0 || !c) return const_cast<char*>(c);
        if (c >= pool && c < pool + pool_stride) return const_cast<char*>(c) + m * pool_stride;
        if (c >= ws && c < ws + ws_stride) return const_cast<char*>(c) + m * ws_stride;
        if (c == x[0]) return const_cast<void*>(x[m]);
        if (c == y[0]) return y[m];
        if (c == dy[0]) return const_cast<void*>(dy[m]);   // dx[m] too where it is the same buffer
        if (c == dx[0]) return dx[m];
        return const_cast<char*>(c);   // parameters and their gradients
    }
    Each each(const void* p) const {
        Each e{};
        for (int m = 0; m < n; m++) e.p[m] = at(p, m);
        return e;
    }
    MicroStride stride() const { return MicroStride{n, pool_stride, ws_stride}; }
};
static const Pass ONE{1, nullptr, nullptr, 0, nullptr, 0, nullptr, nullptr, nullptr, nullptr};

// GEMMs of a pass: in every micro-batch of it.
static hipError_t pgemm(hh_ctx* ctx, const Pass& p, int dt, GemmDesc* g, int n, hipStream_t st) {
    GemmMicro ops[8];
    if (n > 8) return hipErrorInvalidValue;
    if (p.n > 1)
        for (int i = 0; i < n; i++) {
            ops[i] = GemmMicro{p.each(g[i].A), p.each(g[i].B), p.each(g[i].C), p.each(g[i].R), p.each(g[i].fuse.X), p.each(g[i].fuse.Y)};
            g[i].micro = p.n; g[i].each = ops + i;
        }
    return tgemm(ctx, dt, g, n, st);
}
static hipError_t pgemm(hh_ctx* ctx, const Pass& p, int dt, GemmDesc g, hipStream_t st) { return pgemm(ctx, p, dt, &g, 1, st); }

static bool qkv_in_one(const Dims& d, const hh_layer_weights* w) {
    return (const char*)w->wk == (const char*)w->wq + (size_t)d.A * d.H * d.es && (const char*)w->wv == (const char*)w->wk + (size_t)d.Akv * d.H * d.es;
}
static bool gate_up_in_one(const Dims& d, const hh_layer_weights* w) { return (const char*)w->w_up == (const char*)w->w_gate + (size_t)d.F * d.H * d.es; }

// Whether the launches of these GEMMs do what follows them on their way out: on the ring kernel's smaller tiles, and where a
// workgroup has a CU of its own.  That saves a launch of 3 to 5 us and costs the workgroups 1 to 2 us each, one after the
// other on a CU that has several (forward of hidden 512, 3798 tokens: 96.6 us, 98.5 with the rotation fused; backward of hidden
// 1984, 3820 tokens, 128x256 tiles: 510 us, 521 with the SwiGLU gradient fused).  Nor on k_gemm_dma, whose 256 workgroups
// all have their epilogues at once.
static bool can_fuse(const hh_ctx* ctx, const Dims& d, int kind, GemmDesc* g, int n) {
    if (d.dt != DT_BF16) return kind != FUSE_SWIGLU || d.F % 16 == 0;   // its column order is in pieces of 16
    RingUse use;
    for (int i = 0; i < n; i++) gemm_scratch(ctx, g[i]);
    return gemm_bf16_on_ring(g, n, &use) && use.tile <= fuse_tile(kind) && use.workgroups <= 256;
}

// The projections of a forward pass: q|k|v (one problem or three), out, gate|up (one or two), down.
struct FwdGemms {
    GemmDesc qkv[3], out, gu[2], down;
    int n_qkv, n_gu;
};
static void fwd_gemms(const Dims& d, const hh_layer_weights* w, const void* x, void* y, void* saved, void* m, FwdGemms& f) {
    const SavedLayout sl = saved_layout(d);
    const int T = d.T, H = d.H, A = d.A, F = d.F, Akv = d.Akv, Q3 = d.Q3;
    const size_t es = d.es;
    void* xn = at(saved, sl.xn); void* qkv = at(saved, sl.qkv); void* a = at(saved, sl.a); void* h = at(saved, sl.h);
    void* hn = at(saved, sl.hn); void* gu = at(saved, sl.gu);
    // q | k | v rows of width A, Akv, Akv (Akv < A with grouped-query attention)
    const int part_w[3] = {A, Akv, Akv}, part_c[3] = {0, A, A + Akv};
    const void* ws3[3] = {w->wq, w->wk, w->wv};
    f.n_qkv = qkv_in_one(d, w) ? 1 : 3;
    if (f.n_qkv == 1) f.qkv[0] = desc(GEMM_NT, T, Q3, H, xn, H, w->wq, H, qkv, Q3);
    else for (int i = 0; i < 3; i++) f.qkv[i] = desc(GEMM_NT, T, part_w[i], H, xn, H, ws3[i], H, at(qkv, (size_t)part_c[i] * es), Q3);
    f.out = desc(GEMM_NT, T, H, A, a, A, w->wo, A, h, H, x, H);
    f.n_gu = gate_up_in_one(d, w) ? 1 : 2;
    if (f.n_gu == 1) {
        f.gu[0] = desc(GEMM_NT, T, 2 * F, H, hn, H, w->w_gate, H, gu, 2 * F);
    } else {
        f.gu[0] = desc(GEMM_NT, T, F, H, hn, H, w->w_gate, H, gu, 2 * F);
        f.gu[1] = desc(GEMM_NT, T, F, H, hn, H, w->w_up, H, at(gu, (size_t)F * es), 2 * F);
    }
    f.down = desc(GEMM_NT, T, H, F, m, F, w->w_down, F, y, H, h, H);
}

// Addresses are those of the pass's first micro-batch.  gemm_ws: the GEMMs' scratch (null: in its place in the workspace).
static int layer_fwd_impl(hh_ctx* ctx, const Pass& p, const Dims& d, const hh_layer_cfg* cfg, const hh_layer_weights* w, const void* x,
                          void* y, void* saved, void* ws, void* gemm_ws, hipStream_t st) {
    const SavedLayout sl = saved_layout(d);
    const WorkLayout wl = p.side ? *p.side : work_layout(d);
    const int T = d.T, H = d.H, A = d.A, F = d.F, dt = d.dt, Akv = d.Akv, Q3 = d.Q3;
    const size_t es = d.es;
    const Each qkv = p.each(at(saved, sl.qkv)), h = p.each(at(saved, sl.h)), m = p.each(at(ws, wl.m));
    ctx->gemm_ws = d.dt != DT_BF16 ? nullptr : gemm_ws ? gemm_ws : at(ws, wl.gemm_ws);
    FwdGemms f;
    fwd_gemms(d, w, x, y, saved, m.p[0], f);
    const bool rotates = can_fuse(ctx, d, FUSE_ROPE, f.qkv, f.n_qkv), gates = f.n_gu == 1 && can_fuse(ctx, d, FUSE_SWIGLU, f.gu, 1);
    if (rotates)
        for (int i = 0; i < f.n_qkv; i++)   // all but v
            f.qkv[i].fuse = GemmFuse{FUSE_ROPE, d.d, f.n_qkv == 1 ? A + Akv : i < 2 ? f.qkv[i].N : 0, d.S, ctx->rope_seq, ctx->rope_table, nullptr, nullptr};
    if (gates) f.gu[0].fuse = GemmFuse{FUSE_SWIGLU, 2 * F, 0, 0, 0, nullptr, m.p[0], nullptr};

    // a norm is a launch of its own, or the first thing in its projections'
    auto norms = [&](GemmDesc* g, int n, const GemmNorm& q, const void* from) {
        for (int i = 0; i < n; i++) gemm_scratch(ctx, g[i]);
        if (dt != DT_BF16 || !gemm_bf16_norms(g, n)) return false;
        for (int i = 0; i < n; i++) { g[i].A = from; g[i].norm = &q; }
        return true;
    };
    const GemmNorm first{p.each(at(saved, sl.xn)), p.each(at(saved, sl.r1)), w->g_attn, cfg->rms_eps};
    if (!norms(f.qkv, f.n_qkv, first, x))
        TR(HH_TRACE_ELEMENTWISE, 2.0 * T * H * es, rmsnorm_fwd(dt, p.each(x), w->g_attn, first.xn, first.r, p.n, T, H, cfg->rms_eps, st));
    HIP_TRY(pgemm(ctx, p, dt, f.qkv, f.n_qkv, st));
    if (!rotates) TR(HH_TRACE_ELEMENTWISE, 2.0 * T * (A + Akv) * es, rope(dt, qkv, Q3, p.n, T, d.S, d.nh + d.nkv, d.d, ctx->rope_table, ctx->rope_seq, st));
    TR(HH_TRACE_ATTN_FWD, attn_flop(d), attn_fwd(dt, qkv.p[0], Q3, at(saved, sl.a), (float*)at(saved, sl.lse), d.B, d.S, d.nh, d.nkv, d.d,
                                                 p.stride(), st));
    GemmSplit left{};   // the second norm takes h's shares as they are where they are few
    if (dt == DT_BF16) f.out.split = &left;
    HIP_TRY(pgemm(ctx, p, dt, f.out, st));
    const bool sums = left.ksplit > 1;
    const Each res = p.each(x);
    const GemmNorm second{p.each(at(saved, sl.hn)), p.each(at(saved, sl.r2)), w->g_mlp, cfg->rms_eps};
    if (sums || !norms(f.gu, f.n_gu, second, h.p[0]))
        TR(HH_TRACE_ELEMENTWISE, 2.0 * T * H * es, rmsnorm_fwd(dt, h, w->g_mlp, second.xn, second.r, p.n, T, H, cfg->rms_eps, st, sums ? &left : nullptr,
                                                               &res));
    HIP_TRY(pgemm(ctx, p, dt, f.gu, f.n_gu, st));
    if (!gates) TR(HH_TRACE_ELEMENTWISE, 3.0 * T * F * es, swiglu_fwd(dt, p.each(at(saved, sl.gu)), m, p.n, T, F, st));
    HIP_TRY(pgemm(ctx, p, dt, f.down, st));
    return HH_OK;
}

extern "C" int hh_layer_fwd(hh_ctx* ctx, const hh_layer_cfg* cfg, const hh_layer_weights* w, const void* x, void* y,
                            void* saved, void* workspace, void* stream) {
    TRY(check_cfg(cfg));
    TRY(check_weights(w));
    TRY(check_ptr(x, "x")); TRY(check_ptr(y, "y")); TRY(check_ptr(workspace, "workspace"));
    if (saved && ((uintptr_t)saved & 15)) return fail(HH_ERR_MISALIGNED, "saved is not 16-byte aligned");
    if (x == y) return fail(HH_ERR_INVALID_ARG, "y must not alias x");
    if (!ctx) return fail(HH_ERR_INVALID_ARG, "ctx is NULL");
    TRY(ensure_rope(ctx, cfg));
    const Dims d = dims_of(cfg);
    void* sv = saved;
    void* wsp = workspace;
    if (!sv) {  // forward only: the saved block lives at the front of the workspace
        sv = workspace;
        wsp = at(workspace, saved_layout(d).total);
    }
    return layer_fwd_impl(ctx, ONE, d, cfg, w, x, y, sv, wsp, nullptr, (hipStream_t)stream);
}

extern "C" int hh_layer_fwd_noalloc(hh_ctx* ctx, const hh_layer_cfg* cfg, const hh_layer_weights* w, const void* x, void* y,
                                    void* stream) {
    TRY(check_cfg(cfg));
    TRY(check_weights(w));
    TRY(check_ptr(x, "x")); TRY(check_ptr(y, "y"));
    if (x == y) return fail(HH_ERR_INVALID_ARG, "y must not alias x");
    if (!ctx) return fail(HH_ERR_INVALID_ARG, "ctx is NULL");
    // the rotary table is the one thing the ordinary forward may allocate: here it has to be there already
    if (!(ctx->rope_table && ctx->rope_seq >= cfg->seq && ctx->rope_dim == cfg->head_dim && ctx->rope_base == cfg->rope_base))
        return fail(HH_ERR_INVALID_ARG, "hh_layer_fwd_noalloc: no rotary table for this (seq, head_dim, rope_base): call hh_ctx_reserve first");
    const Dims d = dims_of(cfg);
    const size_t saved_b = saved_layout(d).total, need = saved_b + work_layout(d).total;
    if (need > STATIC_SCRATCH_BYTES)
        return fail(HH_ERR_BUFFER_TOO_SMALL, "hh_layer_fwd_noalloc: this shape needs %zu bytes of scratch, the library's array holds %zu",
                    need, (size_t)STATIC_SCRATCH_BYTES);
    void* base = static_scratch(ctx->device);
    if (!base) return fail(HH_ERR_DEVICE, "hh_layer_fwd_noalloc: the scratch array of device %d was never looked up", ctx->device);
    // same carving as hh_layer_fwd with saved == NULL: the saved block first, the workspace behind it
    return layer_fwd_impl(ctx, ONE, d, cfg, w, x, y, base, at(base, saved_b), nullptr, (hipStream_t)stream);
}

// ----------------------------------------------------------- layer backward
// The GEMMs of a backward pass: dm, and three groups of independent ones -- the weight gradients that use an operand of an
// input gradient, and that input gradient last.
struct BwdGemms {
    GemmDesc dm, group[3][4], dw[7];
    int n[3], n_dw;
    bool defer;   // all the weight gradients (dw) in one launch after the last input gradient: predicted to be faster
};
static void bwd_gemms(const Dims& d, const WorkLayout& wl, const hh_layer_weights* w, const hh_layer_grads* g, const void* saved, const void* dy,
                      void* ws, int acc, BwdGemms& b) {
    const SavedLayout sl = saved_layout(d);
    const int T = d.T, H = d.H, A = d.A, F = d.F, Akv = d.Akv, Q3 = d.Q3;
    const size_t es = d.es;
    const void* xn = at(saved, sl.xn); const void* a = at(saved, sl.a); const void* hn = at(saved, sl.hn);
    void* m = at(ws, wl.m); void* dgu = at(ws, wl.dgu); void* dhn = at(ws, wl.dhn); void* dh = at(ws, wl.dh);
    void* da = at(ws, wl.da); void* dqkv = at(ws, wl.dqkv);
    void* dxn = dhn;
    const int part_w[3] = {A, Akv, Akv}, part_c[3] = {0, A, A + Akv};
    const bool dgu_packed = (char*)g->w_up == (char*)g->w_gate + (size_t)F * H * 4 && (size_t)2 * F * H * 4 < ((size_t)1 << 31);
    const bool dqkv_packed = (char*)g->wk == (char*)g->wq + (size_t)A * H * 4 && (char*)g->wv == (char*)g->wk + (size_t)Akv * H * 4 &&
                             (size_t)Q3 * H * 4 < ((size_t)1 << 31);
    GemmDesc (&group)[3][4] = b.group;
    int (&n)[3] = b.n;
    n[0] = n[1] = n[2] = 0;
    b.dm = desc(GEMM_NN, T, F, H, dy, H, w->w_down, F, m, F);
    group[0][n[0]++] = desc(GEMM_TN, H, F, T, dy, H, m, F, g->w_down, F, nullptr, 0, 1, acc);
    if (dgu_packed) {
        group[0][n[0]++] = desc(GEMM_TN, 2 * F, H, T, dgu, 2 * F, hn, H, g->w_gate, H, nullptr, 0, 1, acc);
    } else {
        group[0][n[0]++] = desc(GEMM_TN, F, H, T, dgu, 2 * F, hn, H, g->w_gate, H, nullptr, 0, 1, acc);
        group[0][n[0]++] = desc(GEMM_TN, F, H, T, at(dgu, (size_t)F * es), 2 * F, hn, H, g->w_up, H, nullptr, 0, 1, acc);
    }
    GemmDesc& to_hn = group[0][n[0]++] = desc(GEMM_NN, T, H, 2 * F, dgu, 2 * F, w->w_gate, H, dhn, H);
    if (!gate_up_in_one(d, w)) { to_hn.B1 = w->w_up; to_hn.k1 = F; }
    group[1][n[1]++] = desc(GEMM_TN, H, A, T, dh, H, a, A, g->wo, A, nullptr, 0, 1, acc);
    group[1][n[1]++] = desc(GEMM_NN, T, A, H, dh, H, w->wo, A, da, A);
    if (dqkv_packed) {
        group[2][n[2]++] = desc(GEMM_TN, Q3, H, T, dqkv, Q3, xn, H, g->wq, H, nullptr, 0, 1, acc);
    } else {
        float* gs[3] = {g->wq, g->wk, g->wv};
        for (int i = 0; i < 3; i++)
            group[2][n[2]++] = desc(GEMM_TN, part_w[i], H, T, at(dqkv, (size_t)part_c[i] * es), Q3, xn, H, gs[i], H, nullptr, 0, 1, acc);
    }
    GemmDesc& to_xn = group[2][n[2]++] = desc(GEMM_NN, T, H, Q3, dqkv, Q3, w->wq, H, dxn, H);
    if (!qkv_in_one(d, w)) { to_xn.B1 = w->wk; to_xn.k1 = A; to_xn.B2 = w->wv; to_xn.k2 = A + Akv; }
}
static void plan_deferral(const hh_ctx* ctx, const Dims& d, BwdGemms& b) {
    b.n_dw = 0;
    for (int i = 0; i < 3; i++)
        for (int j = 0; j < b.n[i]; j++) {
            gemm_scratch(ctx, b.group[i][j]);
            if (j + 1 < b.n[i]) b.dw[b.n_dw++] = b.group[i][j];
        }
    const GemmDesc* const groups[3] = {b.group[0], b.group[1], b.group[2]};
    b.defer = d.dt == DT_BF16 && gemm_bf16_defer(b.dw, b.n_dw, groups, b.n);
}

static int layer_bwd_impl(hh_ctx* ctx, const Pass& p, const Dims& d, const hh_layer_weights* w, const void* x, const void* saved,
                          const void* dy, void* dx, const hh_layer_grads* g, int acc, void* ws, void* gemm_ws, hipStream_t st) {
    const SavedLayout sl = saved_layout(d);
    const WorkLayout one = work_layout(d), wl = p.side ? *p.side : one;
    const int T = d.T, H = d.H, F = d.F, dt = d.dt;
    const size_t es = d.es;
    acc = acc ? 1 : 0;
    ctx->gemm_ws = d.dt != DT_BF16 ? nullptr : gemm_ws ? gemm_ws : at(ws, wl.gemm_ws);
    BwdGemms b;
    bwd_gemms(d, wl, w, g, saved, dy, ws, acc, b);
    plan_deferral(ctx, d, b);
    const bool defer = b.defer;

    // Partial column sums of the two gain gradients.  Those of the MLP norm go to the front of the m | dgate|dup stretch
    // if nobody needs that any more by then and it holds a row per workgroup, otherwise to `partial`; those of the
    // attention norm to the stretch (behind the others) or to `partial` likewise.  Unless both have to take `partial`,
    // one launch at the end reduces both.  (Side by side both have a place of their own, of as many rows.)
    const size_t want = gain_bytes(d), stretch = one.dhn - one.m, partial_b = one.gemm_ws - one.partial;
    const bool mlp_in = !defer && stretch >= want;
    const size_t taken = mlp_in ? up256(want) : 0;
    const bool attn_in = stretch - taken >= want;
    const Each part2 = p.each(at(ws, p.side || !mlp_in ? wl.partial : wl.m));
    const Each part1 = p.each(at(ws, p.side ? wl.partial + up256(want) : attn_in ? wl.m + taken : wl.partial));
    const size_t part2_b = mlp_in ? want : partial_b, part1_b = attn_in ? want : partial_b;
    const ColSum sums[2] = {{part2, rmsnorm_bwd_blocks(T, H, part2_b), g->g_mlp}, {part1, rmsnorm_bwd_blocks(T, H, part1_b), g->g_attn}};
    const bool sum_both = part1.p[0] != part2.p[0];
    // The norms take the shares of d(hn) and d(xn) as they are where those are few, nothing else uses the scratch before, and the
    // norm has a workgroup for every row or two (333 rows of 1280 in 42 workgroups: 6.8 + 4.5 us, 10.7 with eight shares).
    GemmSplit left[3] = {};
    if (dt == DT_BF16 && !defer)
        for (int i = 0; i < 3; i += 2)
            if (2 * sums[i / 2].rows >= T) b.group[i][b.n[i] - 1].split = left + i;
    auto run_group = [&](int i) { return defer ? pgemm(ctx, p, dt, &b.group[i][b.n[i] - 1], 1, st) : pgemm(ctx, p, dt, b.group[i], b.n[i], st); };

    // MLP branch: y = h + m Wd^T
    const Each m = p.each(at(ws, wl.m)), dgu = p.each(at(ws, wl.dgu)), dhn = p.each(at(ws, wl.dhn)), dh = p.each(at(ws, wl.dh));
    const bool gates = can_fuse(ctx, d, FUSE_SWIGLU_BWD, &b.dm, 1);                                                   // dgate|dup, m ...
    if (gates) b.dm.fuse = GemmFuse{FUSE_SWIGLU_BWD, 0, 0, 0, 0, nullptr, const_cast<char*>(at(saved, sl.gu)), at(ws, wl.dgu)};
    HIP_TRY(pgemm(ctx, p, dt, b.dm, st));                                                           // ... or dm (in the m buffer)
    if (!gates) TR(HH_TRACE_ELEMENTWISE, 6.0 * T * F * es, swiglu_bwd(dt, m, p.each(at(saved, sl.gu)), dgu, m, p.n, T, F, st));   // dgate|dup, m
    HIP_TRY(run_group(0));
    const GemmSplit* const split2 = left[0].ksplit > 1 ? left : nullptr;
    const bool gain2 = rmsnorm_bwd_sums_gain(T, H, split2);
    TR(HH_TRACE_ELEMENTWISE, 4.0 * T * H * es, rmsnorm_bwd(dt, dhn, p.each(at(saved, sl.h)), p.each(at(saved, sl.r2)), w->g_mlp, p.each(dy), dh,
                                                           part2, part2_b, p.n, T, H, st, split2, gain2 ? g->g_mlp : nullptr, acc));   // dh = dy + norm-bwd
    if (!sum_both && !gain2) TR(HH_TRACE_ELEMENTWISE, 4.0 * sums[0].rows * H, colsum_reduce(sums, 1, p.n, H, acc, st));

    // attention branch: h = x + a Wo^T
    HIP_TRY(run_group(1));
    // dq | dk | dv of the rotated q, k and of v, with the rotary embedding taken back out of dq and dk.  The fp32 path's
    // scratch is the m | dgate|dup | dhn stretch of the workspace behind the partial sums above, whose contents nobody
    // needs any more by now.
    const size_t part_at = dt == DT_BF16 ? wl.dkv_part : wl.m + taken, part_end = dt == DT_BF16 ? wl.partial : wl.dh;
    TR(HH_TRACE_ATTN_BWD, 2.0 * attn_flop(d), attn_bwd(dt, at(saved, sl.qkv), d.Q3, at(saved, sl.a), at(ws, wl.da), (const float*)at(saved, sl.lse),
                                                       (float*)at(ws, wl.dvec), at(ws, wl.dqkv), at(ws, part_at), part_end - part_at, d.B, d.S,
                                                       d.nh, d.nkv, d.d, ctx->rope_table, ctx->rope_seq, p.stride(), st));
    HIP_TRY(run_group(2));
    if (defer) HIP_TRY(pgemm(ctx, p, dt, b.dw, b.n_dw, st));
    // (A caller may write dx over x: the gain's gradient then comes from partial sums, as no other workgroup may read x.)
    const GemmSplit* const split1 = left[2].ksplit > 1 ? left + 2 : nullptr;
    const size_t act = (size_t)T * H * es;
    const bool apart = (const char*)x + act <= (const char*)dx || (const char*)dx + act <= (const char*)x;
    const bool gain1 = apart && gain2 && rmsnorm_bwd_sums_gain(T, H, split1);   // with sums to do anyway, in that launch
    TR(HH_TRACE_ELEMENTWISE, 4.0 * T * H * es, rmsnorm_bwd(dt, dhn, p.each(x), p.each(at(saved, sl.r1)), w->g_attn, dh, p.each(dx),
                                                           part1, part1_b, p.n, T, H, st, split1, gain1 ? g->g_attn : nullptr, acc));   // d(xn) in dhn; dx = dh + norm-bwd
    const int first = gain2 || !sum_both ? 1 : 0;   // of the sums left to do
    if (!gain1) TR(HH_TRACE_ELEMENTWISE, 4.0 * ((first ? 0 : sums[0].rows) + sums[1].rows) * H, colsum_reduce(sums + first, 2 - first, p.n, H, acc, st));
    return HH_OK;
}

extern "C" int hh_layer_bwd(hh_ctx* ctx, const hh_layer_cfg* cfg, const hh_layer_weights* w, const void* x,
                            const void* saved, const void* dy, void* dx, const hh_layer_grads* grads, int accumulate,
                            void* workspace, void* stream) {
    TRY(check_cfg(cfg));
    TRY(check_weights(w));
    TRY(check_grads(grads));
    TRY(check_ptr(x, "x")); TRY(check_ptr(saved, "saved")); TRY(check_ptr(dy, "dy")); TRY(check_ptr(dx, "dx"));
    TRY(check_ptr(workspace, "workspace"));
    if (!ctx) return fail(HH_ERR_INVALID_ARG, "ctx is NULL");
    TRY(ensure_rope(ctx, cfg));
    const Dims d = dims_of(cfg);
    return layer_bwd_impl(ctx, ONE, d, w, x, saved, dy, dx, grads, accumulate, workspace, nullptr, (hipStream_t)stream);
}

// --------------------------------------------------------------- stage step
struct StagePool {
    size_t saved_sz, act_sz, per_micro;
    char* base;
    int k;
    void* saved(int m, int l) const { return base + (size_t)m * per_micro + (size_t)l * (saved_sz + act_sz); }
    // output of layer l (< k-1) = input of layer l+1
    void* act(int m, int l) const { return base + (size_t)m * per_micro + (size_t)l * (saved_sz + act_sz) + saved_sz; }
};
static StagePool stage_pool(const Dims& d, int k, void* pool) {
    StagePool p;
    p.saved_sz = saved_layout(d).total; p.act_sz = act_bytes(d); p.k = k;
    p.per_micro = (size_t)k * p.saved_sz + (size_t)(k - 1) * p.act_sz;
    p.base = (char*)pool;
    return p;
}

static int check_stage_args(const hh_layer_cfg* cfg, int n_layers, const hh_layer_weights* w, const hh_layer_grads* g) {
    TRY(check_cfg(cfg));
    if (n_layers <= 0) return fail(HH_ERR_INVALID_ARG, "n_layers must be positive");
    if (!w || !g) return fail(HH_ERR_INVALID_ARG, "weights / grads array is NULL");
    for (int l = 0; l < n_layers; l++) {
        TRY(check_weights(&w[l]));
        TRY(check_grads(&g[l]));
    }
    return HH_OK;
}

// Forward of a pass's micro-batches through the stage, activations into the pool slots from `slot` on.
static int stage_fwd(hh_ctx* ctx, const Pass& ps, const Dims& d, const hh_layer_cfg* cfg, int k, const hh_layer_weights* w, const StagePool& p,
                     int slot, const void* x, void* y, void* workspace, void* gemm_ws, hipStream_t st) {
    for (int l = 0; l < k; l++) {
        const void* in = l == 0 ? x : p.act(slot, l - 1);
        void* out = l == k - 1 ? y : p.act(slot, l);
        TRY(layer_fwd_impl(ctx, ps, d, cfg, &w[l], in, out, p.saved(slot, l), workspace, gemm_ws, st));
    }
    return HH_OK;
}
// Backward of the micro-batches whose activations sit in the pool slots from `slot` on; gbuf: gradient flowing between layers,
// updated in place.
static int stage_bwd(hh_ctx* ctx, const Pass& ps, const Dims& d, int k, const hh_layer_weights* w, const hh_layer_grads* g,
                     const StagePool& p, int slot, const void* x, const void* dy, void* dx, int acc, void* workspace, void* gbuf, void* gemm_ws,
                     hipStream_t st) {
    for (int l = k - 1; l >= 0; l--) {
        const void* in = l == 0 ? x : p.act(slot, l - 1);
        const void* gin = l == k - 1 ? dy : gbuf;
        void* gout = l == 0 ? dx : gbuf;
        TRY(layer_bwd_impl(ctx, ps, d, &w[l], in, p.saved(slot, l), gin, gout, &g[l], acc, workspace, gemm_ws, st));
    }
    return HH_OK;
}

// How many micro-batches (of at most n_live) go through the launches side by side: as many as there is room for, in buffers that
// are sized for one after the other.  Side by side each has its own tensors (side_layout and the gradient between layers behind
// them), one after the other where a single one has its tensors and the GEMMs' partial sums, or in the pool's slots that a pass
// leaves free; the partial sums of all of them lie behind the tensors, or alone in the workspace.  In bf16 only where every
// GEMM goes to the ring kernel, with the tile and split of a micro-batch by itself, which larger micro-batches do not, or is a weight
// gradient of so few tokens that the ring kernel forms the same bits.
struct Side { int n; bool in_pool, defers; };
static size_t side_unit(const Dims& d, bool defers) { return side_layout(d, defers).total + act_bytes(d); }
static Side side_by_side(hh_ctx* ctx, const Dims& d, int k, const hh_layer_weights* w, const hh_layer_grads* g, int n_live, void* workspace) {
    const size_t total = work_layout(d).total + act_bytes(d), slot = stage_pool(d, k, nullptr).per_micro;
    size_t unit = side_unit(d, false);
    const Side one{1, false, false};
    auto in_pool = [&](int n) { return (size_t)n * unit <= (size_t)(n_live - n) * slot; };
    if (n_live < 2 || (2 * unit > total && !(n_live > 2 && in_pool(2)))) return one;
    bool defers = false;
    size_t partial = 0;   // of one micro-batch, the launch that has most
    ctx->gemm_ws = workspace;   // plans ask for sizes and for whether there is scratch, not where anything is
    for (int l = 0; l < k; l++) {
        FwdGemms f;
        fwd_gemms(d, &w[l], workspace, workspace, workspace, workspace, f);
        BwdGemms b;
        bwd_gemms(d, work_layout(d), &w[l], &g[l], workspace, workspace, workspace, 1, b);
        plan_deferral(ctx, d, b);
        if (d.dt != DT_BF16) continue;   // any
        auto take = [&](GemmDesc* q, int m) {
            RingUse use;
            for (int i = 0; i < m; i++) gemm_scratch(ctx, q[i]);
            if (!gemm_bf16_on_ring(q, m, &use)) return false;
            partial = std::max(partial, use.partial);
            return true;
        };
        if (!take(f.qkv, f.n_qkv) || !take(&f.out, 1) || !take(f.gu, f.n_gu) || !take(&f.down, 1) || !take(&b.dm, 1)) return one;
        for (int i = 0; i < 3; i++)
            if (!take(b.defer ? &b.group[i][b.n[i] - 1] : b.group[i], b.defer ? 1 : b.n[i])) return one;
        if (b.defer && !take(b.dw, b.n_dw)) return one;
        defers = defers || b.defer;
    }
    unit = side_unit(d, defers);
    int ws = std::min(n_live, MICRO_MAX), pool = std::min(n_live - 1, MICRO_MAX);
    while (ws > 1 && (size_t)ws * (unit + partial) > total) ws--;
    while (pool > 1 && !(in_pool(pool) && pool * partial <= total)) pool--;
    return pool > ws ? Side{pool, true, defers} : Side{ws, false, defers};
}

// Whether it does not matter in which order micro-batches and layers touch the buffers of a call: none that is written overlaps
// another one (but dx[m] may be dy[m], in all of them or none); inputs and weights may be shared, as wholes.
static bool separate_buffers(const Dims& d, int k, const hh_layer_weights* w, const hh_layer_grads* g, int n, const void* const* x, void* const* y,
                             const void* const* dy, void* const* dx, const StagePool& pool, int n_live, const void* workspace) {
    enum { X, DY, WEIGHT, WRITTEN };   // only buffers of one of the first three kinds may be one buffer
    struct Buf { uintptr_t at, end; int kind; };
    const size_t most = 4 * (size_t)n + 18 * (size_t)k + 2;
    const std::unique_ptr<Buf[]> v(new (std::nothrow) Buf[most]);
    if (!v) return false;
    size_t count = 0;
    auto add = [&](const void* p, size_t bytes, int kind) { v[count++] = {(uintptr_t)p, (uintptr_t)p + bytes, kind}; };
    const bool in_place = dx[0] == dy[0];
    const size_t act = (size_t)d.T * d.H * d.es;
    for (int m = 0; m < n; m++) {
        if ((dx[m] == dy[m]) != in_place) return false;
        add(x[m], act, X);
        add(y[m], act, WRITTEN);
        add(dy[m], act, in_place ? WRITTEN : DY);
        if (!in_place) add(dx[m], act, WRITTEN);
    }
    for (int l = 0; l < k; l++) {
        auto layer = [&](const auto& q, size_t gain, size_t es, int kind) {
            const size_t col = (size_t)d.H * es;
            add(q.g_attn, gain, kind); add(q.g_mlp, gain, kind);
            add(q.wq, d.A * col, kind); add(q.wk, d.Akv * col, kind); add(q.wv, d.Akv * col, kind); add(q.wo, d.A * col, kind);
            add(q.w_gate, d.F * col, kind); add(q.w_up, d.F * col, kind); add(q.w_down, d.F * col, kind);
        };
        layer(w[l], d.H * d.es, d.es, WEIGHT);
        layer(g[l], d.H * sizeof(float), sizeof(float), WRITTEN);
    }
    add(pool.base, pool.per_micro * (size_t)n_live, WRITTEN);
    add(workspace, work_layout(d).total + act_bytes(d), WRITTEN);
    std::sort(v.get(), v.get() + count, [](const Buf& a, const Buf& b) { return a.at < b.at; });
    uintptr_t end = v[0].end;
    for (size_t i = 1; i < count; i++) {
        const bool one = v[i].at == v[i - 1].at && v[i].kind == v[i - 1].kind && v[i].kind != WRITTEN;
        if (v[i].at < end && !one) return false;
        end = std::max(end, v[i].end);
    }
    return true;
}

// Both schedules: forward of the first n_live micro-batches, then backward of m followed by forward of
// m + n_live.  n_live == n_micro is "all forwards, then all backwards".  Backward always visits the
// micro-batches in ascending order, so the fp32 sums are formed in the same order for every n_live.
// Small micro-batches go through the launches side by side, a pass of up to n_live of them after the other: forward of all
// of a pass, then backward of all of it, which is the same results with no more activations alive.  Such launches are bound by
// latency and by the one chain of work of a workgroup, not by a unit of the chip.  Taken wherever it fits: of 200 random stages (both
// types, hidden 128 to 11776, 1 to 6864 tokens, 2 to 8 micro-batches) each takes 0.16 to 0.88 of its time one by one.
static int stage_run(hh_ctx* ctx, const hh_layer_cfg* cfg, int n_layers, const hh_layer_weights* w, int n_micro, int n_live,
                     const void* const* x, void* const* y, const void* const* dy, void* const* dx, const hh_layer_grads* g,
                     int zero_grads_first, void* saved_pool, void* workspace, void* stream) {
    TRY(check_stage_args(cfg, n_layers, w, g));
    if (n_micro <= 0) return fail(HH_ERR_INVALID_ARG, "n_micro must be positive");
    if (n_live <= 0 || n_live > n_micro) return fail(HH_ERR_INVALID_ARG, "n_live must be in 1..n_micro (got %d, n_micro %d)", n_live, n_micro);
    if (!x || !y || !dy || !dx) return fail(HH_ERR_INVALID_ARG, "x / y / dy / dx pointer array is NULL");
    for (int m = 0; m < n_micro; m++) {
        TRY(check_ptr(x[m], "x[m]")); TRY(check_ptr(y[m], "y[m]")); TRY(check_ptr(dy[m], "dy[m]")); TRY(check_ptr(dx[m], "dx[m]"));
        if (x[m] == y[m]) return fail(HH_ERR_INVALID_ARG, "y[m] must not alias x[m]");
    }
    TRY(check_ptr(saved_pool, "saved_pool")); TRY(check_ptr(workspace, "workspace"));
    if (!ctx) return fail(HH_ERR_INVALID_ARG, "ctx is NULL");
    TRY(ensure_rope(ctx, cfg));
    const Dims d = dims_of(cfg);
    const StagePool p = stage_pool(d, n_layers, saved_pool);
    hipStream_t st = (hipStream_t)stream;
    const WorkLayout wl = work_layout(d);
    const Side side = side_by_side(ctx, d, n_layers, w, g, n_live, workspace);
    if (side.n > 1 && separate_buffers(d, n_layers, w, g, n_micro, x, y, dy, dx, p, n_live, workspace)) {
        const WorkLayout sl = side_layout(d, side.defers);
        const size_t unit = side_unit(d, side.defers);
        const int passes = (n_micro + side.n - 1) / side.n;
        char* const ws = side.in_pool ? p.base + (size_t)side.n * p.per_micro : (char*)workspace;
        void* const gbuf = ws + unit - act_bytes(d);
        void* const gemm_ws = side.in_pool ? workspace : ws + (size_t)side.n * unit;
        ctx->gemm_room = wl.total + act_bytes(d) - (side.in_pool ? 0 : (size_t)side.n * unit);
        for (int i = 0, m = 0; i < passes; i++) {   // as alike as they can be
            const int n = (n_micro - m + passes - i - 1) / (passes - i);
            const Pass ps{n, d.dt == DT_BF16 ? &sl : nullptr, p.base, p.per_micro, ws, unit, x + m, y + m, dy + m, dx + m};
            TRY(stage_fwd(ctx, ps, d, cfg, n_layers, w, p, 0, x[m], y[m], ws, gemm_ws, st));
            TRY(stage_bwd(ctx, ps, d, n_layers, w, g, p, 0, x[m], dy[m], dx[m], m > 0 || !zero_grads_first, ws, gbuf, gemm_ws, st));
            m += n;
        }
        return HH_OK;
    }
    void* gbuf = at(workspace, wl.total);
    for (int m = 0; m < n_live; m++) TRY(stage_fwd(ctx, ONE, d, cfg, n_layers, w, p, m, x[m], y[m], workspace, nullptr, st));
    for (int m = 0; m < n_micro; m++) {
        const int acc = (m > 0 || !zero_grads_first) ? 1 : 0;
        const int slot = m % n_live;
        TRY(stage_bwd(ctx, ONE, d, n_layers, w, g, p, slot, x[m], dy[m], dx[m], acc, workspace, gbuf, nullptr, st));
        const int nxt = m + n_live;   // its activations take the slot just released
        if (nxt < n_micro) TRY(stage_fwd(ctx, ONE, d, cfg, n_layers, w, p, slot, x[nxt], y[nxt], workspace, nullptr, st));
    }
    return HH_OK;
}

// For tests, not part of the public interface: how many micro-batches such a call takes through its launches side by side.
extern "C" int hh_internal_side_by_side(const hh_layer_cfg* cfg, int n_layers, const hh_layer_weights* w, const hh_layer_grads* g, int n_micro,
                                        int n_live, const void* const* x, void* const* y, const void* const* dy, void* const* dx, void* saved_pool,
                                        void* workspace) {
    const Dims d = dims_of(cfg);
    hh_ctx ctx{0, nullptr, 0, 0, 0.f, {}, 0, false, 0u, nullptr, {}};
    const int n = side_by_side(&ctx, d, n_layers, w, g, n_live, workspace).n;
    return n > 1 && separate_buffers(d, n_layers, w, g, n_micro, x, y, dy, dx, stage_pool(d, n_layers, saved_pool), n_live, workspace) ? n : 1;
}

// Likewise: where the tensors of one of them lie (m, dgate|dup, d(hn), dh, da, dqkv, delta, partial dK and dV, gain partials, the
// gradient between layers, and the end), and the bytes of the partial dK and dV.
extern "C" void hh_internal_side_layout(const hh_layer_cfg* cfg, int n_layers, const hh_layer_weights* w, const hh_layer_grads* g, size_t at[11],
                                        size_t* dkv_part_bytes) {
    const Dims d = dims_of(cfg);
    hh_ctx ctx{0, nullptr, 0, 0, 0.f, {}, 0, false, 0u, nullptr, {}};
    const bool defers = side_by_side(&ctx, d, n_layers, w, g, 1 << 20, (void*)(uintptr_t)4096).defers;
    const WorkLayout s = side_layout(d, defers);
    const size_t all[11] = {s.m, s.dgu, s.dhn, s.dh, s.da, s.dqkv, s.dvec, s.dkv_part, s.partial, s.total, side_unit(d, defers)};
    std::copy(all, all + 11, at);
    *dkv_part_bytes = attn_bwd_scratch_bytes(d.dt, d.B, d.S, d.nh, d.nkv, d.d);
}

extern "C" int hh_stage_step(hh_ctx* ctx, const hh_layer_cfg* cfg, int n_layers, const hh_layer_weights* w, int n_micro,
                             const void* const* x, void* const* y, const void* const* dy, void* const* dx,
                             const hh_layer_grads* g, int zero_grads_first, void* saved_pool, void* workspace, void* stream) {
    return stage_run(ctx, cfg, n_layers, w, n_micro, n_micro, x, y, dy, dx, g, zero_grads_first, saved_pool, workspace, stream);
}

extern "C" int hh_stage_step_1f1b(hh_ctx* ctx, const hh_layer_cfg* cfg, int n_layers, const hh_layer_weights* w, int n_micro,
                                  int n_live, const void* const* x, void* const* y, const void* const* dy, void* const* dx,
                                  const hh_layer_grads* g, int zero_grads_first, void* saved_pool, void* workspace,
                                  void* stream) {
    return stage_run(ctx, cfg, n_layers, w, n_micro, n_live, x, y, dy, dx, g, zero_grads_first, saved_pool, workspace, stream);
}

// ------------------------------------------------------------------ profile
static float median(std::vector<float>& v) {
    std::sort(v.begin(), v.end());
    const size_t n = v.size();
    return n % 2 ? v[n / 2] : 0.5f * (v[n / 2 - 1] + v[n / 2]);
}

extern "C" int hh_layer_profile(hh_ctx* ctx, const hh_layer_cfg* cfg, int n_layers, const hh_layer_weights* w,
                                const hh_layer_grads* g, const void* x, const void* dy, int warmup, int iters,
                                void* saved_pool, void* workspace, hh_profile_rec* out, void* stream) {
    TRY(check_stage_args(cfg, n_layers, w, g));
    if (warmup < 0 || iters <= 0) return fail(HH_ERR_INVALID_ARG, "warmup must be >= 0 and iters > 0");
    TRY(check_ptr(x, "x")); TRY(check_ptr(dy, "dy")); TRY(check_ptr(saved_pool, "saved_pool")); TRY(check_ptr(workspace, "workspace"));
    if (!out) return fail(HH_ERR_INVALID_ARG, "out is NULL");
    if (!ctx) return fail(HH_ERR_INVALID_ARG, "ctx is NULL");
    TRY(ensure_rope(ctx, cfg));
    const Dims d = dims_of(cfg);
    const StagePool p = stage_pool(d, n_layers, saved_pool);
    hipStream_t st = (hipStream_t)stream;
    void* gbuf = at(workspace, work_layout(d).total);
    // the last layer's output has no slot in the pool (the caller's y in a stage step): park it in gbuf,
    // which is free during the forward sweep
    const int k = n_layers;
    std::vector<hipEvent_t> ev((size_t)4 * k);
    for (auto& e : ev) e = nullptr;
    int rc = HH_OK;
    auto cleanup = [&]() { for (auto e : ev) if (e) (void)hipEventDestroy(e); };
    for (auto& e : ev) {
        hipError_t he = hipEventCreate(&e);
        if (he != hipSuccess) { cleanup(); return hip_fail(he, "hipEventCreate"); }
    }
    std::vector<std::vector<float>> tf(k), tb(k);
    for (int it = 0; it < warmup + iters && rc == HH_OK; it++) {
        for (int l = 0; l < k && rc == HH_OK; l++) {
            const void* in = l == 0 ? x : p.act(0, l - 1);
            void* o = l == k - 1 ? gbuf : p.act(0, l);
            (void)hipEventRecord(ev[4 * l], st);
            rc = layer_fwd_impl(ctx, ONE, d, cfg, &w[l], in, o, p.saved(0, l), workspace, nullptr, st);
            (void)hipEventRecord(ev[4 * l + 1], st);
        }
        for (int l = k - 1; l >= 0 && rc == HH_OK; l--) {
            const void* in = l == 0 ? x : p.act(0, l - 1);
            const void* gin = l == k - 1 ? dy : gbuf;
            (void)hipEventRecord(ev[4 * l + 2], st);
            rc = layer_bwd_impl(ctx, ONE, d, &w[l], in, p.saved(0, l), gin, gbuf, &g[l], 1, workspace, nullptr, st);
            (void)hipEventRecord(ev[4 * l + 3], st);
        }
        if (rc != HH_OK) break;
        hipError_t he = hipStreamSynchronize(st);
        if (he != hipSuccess) { rc = hip_fail(he, "hipStreamSynchronize"); break; }
        if (it >= warmup)
            for (int l = 0; l < k; l++) {
                float a = 0.f, b = 0.f;
                (void)hipEventElapsedTime(&a, ev[4 * l], ev[4 * l + 1]);
                (void)hipEventElapsedTime(&b, ev[4 * l + 2], ev[4 * l + 3]);
                tf[l].push_back(a);
                tb[l].push_back(b);
            }
    }
    cleanup();
    if (rc != HH_OK) return rc;
    double ff = 0, bf = 0;
    (void)hh_layer_flops(cfg, &ff, &bf);
    const size_t A = d.A;
    const uint64_t nparam = 2ull * d.H + (2ull * A + 2ull * d.Akv) * d.H + 3ull * (uint64_t)d.F * d.H;
    for (int l = 0; l < k; l++) {
        hh_profile_rec& r = out[l];
        r.layer = l;
        r.fwd_ms = median(tf[l]);
        r.bwd_ms = median(tb[l]);
        r.fwd_flop = ff; r.bwd_flop = bf;
        r.fwd_tflops = (float)(ff / (r.fwd_ms * 1e-3) * 1e-12);
        r.bwd_tflops = (float)(bf / (r.bwd_ms * 1e-3) * 1e-12);
        r.weight_bytes = nparam * d.es;
        r.grad_bytes = nparam * 4;
        r.saved_act_bytes = p.saved_sz + (uint64_t)d.T * d.H * d.es;  // the saved block plus the layer's input
        r.p2p_bytes = (uint64_t)d.B * d.S * d.H * 2;
        r.workspace_bytes = work_layout(d).total + act_bytes(d);
    }
    return HH_OK;
}
