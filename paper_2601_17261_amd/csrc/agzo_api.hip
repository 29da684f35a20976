// C ABI of libagzo: argument checks, workspace carving and the stream-ordered sequence of kernel
// launches that makes up one AGZO step (Alg. 2) for a linear layer.  No arithmetic lives here.
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <initializer_list>
#include <mutex>
#include <new>
#include <vector>

#include "agzo_internal.h"
#include "fork.h"
#include "grow.h"
#include "overlap.h"

using namespace agzo;

struct ProfClass {
    std::vector<hipEvent_t> start, stop;
    size_t used = 0;
};

// Scratch of agzo_update_noalloc: the factor fragments of one bf16 update, for callers that cannot allocate.
// One copy per GPU, held until the process ends; its device address is resolved once per device (resolve_scratch).
constexpr size_t kStaticScratchBytes = (size_t)8 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

struct agzo_ctx {
    hipStream_t stream;
    int device;            // the device that was current at agzo_create
    char* static_scratch;  // device address of `scratch` on that device
    char err[512];
    char* ws;
    size_t ws_bytes;
    int* flag;   // device int: deferred numeric failure
    uint32_t prof;      // mask of timed kernel classes (bit = AGZO_PROF_* value)
    ProfClass pc[AGZO_PROF_KINDS];
    // base forwards of a set of layers run on a stream of the context's own beside the extraction (step_many_body)
    hipStream_t side;
    hipEvent_t fork, join;
    // clock telemetry: kClkSlots records of four 64-bit words (one per timed GEMM launch), then the probe's record
    unsigned long long* clk;
    size_t clk_used;
};
constexpr size_t kClkSlots = 8192;
constexpr size_t kClkBytes = (kClkSlots + 1) * 32 + 1024;

namespace {

int fail(agzo_ctx* c, int code, const char* fmt, ...) {
    if (c) {
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(c->err, sizeof(c->err), fmt, ap);
        va_end(ap);
    }
    return code;
}

#define HIPCHK(expr)                                                                              \
    do {                                                                                          \
        hipError_t e__ = (expr);                                                                  \
        if (e__ != hipSuccess) return fail(ctx, AGZO_EHIP, "%s: %s", #expr, hipGetErrorString(e__)); \
    } while (0)
#define TRY(expr)              \
    do {                       \
        int rc__ = (expr);     \
        if (rc__ != 0) return rc__; \
    } while (0)

inline bool timed(const agzo_ctx* c, int kind) { return ((c->prof >> kind) & 1u) != 0; }

// Optional timing of one kernel class with HIP events recorded on the ctx stream around each launch.
struct ProfScope {
    agzo_ctx* c;
    int kind;
    hipEvent_t stop = nullptr;
    ProfScope(agzo_ctx* ctx, int k) : c(ctx), kind(k) {
        if (!timed(c, kind)) return;
        ProfClass& pc = c->pc[kind];
        if (pc.used == pc.start.size()) {
            hipEvent_t a, b;
            if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess) return;
            pc.start.push_back(a);
            pc.stop.push_back(b);
        }
        (void)hipEventRecord(pc.start[pc.used], c->stream);
        stop = pc.stop[pc.used];
        pc.used++;
    }
    ~ProfScope() {
        if (stop) (void)hipEventRecord(stop, c->stream);
    }
};

// Device address of the static scratch array on the current device.  The array's name is only a host-side handle
// for the symbol: every use of its memory goes through the address looked up here, once per device.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
char* g_scratch_ptr[kMaxDevices] = {};

hipError_t resolve_scratch(int device, char** out) {
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[device]) {
        void* ptr = nullptr;
        hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[device] = static_cast<char*>(ptr);
    }
    *out = g_scratch_ptr[device];
    return hipSuccess;
}

inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }
inline int round16(int r) { return (r + 15) / 16 * 16; }
inline int64_t round32(int64_t n) { return (n + 31) / 32 * 32; }

// carve-out of the ctx workspace for one layer; everything a step can need at the same time
struct Plan {
    size_t off_S, off_Q, off_B, off_pack, off_T, off_TpackT, off_xtt, off_qr, off_part, off_Ybuf, off_ce_ms, off_ce_tl, off_upd, off_ext, off_xqpart, off_split, total;
    int rp, nsplit, sketch_tokens;
    int64_t m_pad;
    int n_part;
    size_t part_count;   // doubles in the loss-partials region
};

// base: where this layer's carve-out starts inside the workspace (several layers side by side in the batched calls)
// sketch_tokens: the range sketch comes out of the forward GEMM, one partial sum per token tile of that many (0: it does not)
Plan make_plan(const agzo_layer& L, bool need_ybuf, bool ce = false, bool shared = false, size_t base = 0, int sketch_tokens = 0) {
    Plan p;
    const bool bf = (L.dtype == AGZO_BF16);
    p.rp = round16(L.r);
    p.sketch_tokens = sketch_tokens;
    p.m_pad = sketch_tokens ? gemm_bf16_sketch_mpad(L.n_tokens) : round32(L.n_tokens);
    p.nsplit = !bf ? 1 : sketch_tokens ? gemm_bf16_sketch_splits(L.n_tokens, sketch_tokens) : xtt_num_splits(L.n_tokens, L.d_in);
    const int n_gemm = bf ? gemm_bf16_num_workgroups(L.n_tokens, L.d_out, !ce && !shared && L.tiling != AGZO_TILING_LARGE) : forward_f32_num_workgroups(L.n_tokens, L.d_out);
    p.n_part = n_gemm;
    size_t o = align_up(base);
    auto take = [&](size_t bytes) { size_t at = o; o += align_up(bytes); return at; };
    p.off_S = take((size_t)L.d_in * L.r * 4);
    p.off_Q = take((size_t)L.d_in * L.r * 4);
    p.off_B = take((size_t)L.d_in * L.r * 4);
    p.off_pack = take(bf ? (size_t)3 * p.rp * L.d_in * 2 : 0);
    p.off_T = take((size_t)L.n_tokens * L.r * 4);
    p.off_TpackT = take(bf ? (size_t)3 * p.rp * p.m_pad * 2 : 0);
    p.off_xtt = take(bf ? (size_t)p.nsplit * L.d_in * p.rp * 4 : 0);
    p.off_qr = take(qr_workspace_bytes(L.d_in, L.r));
    {
        size_t part = (size_t)n_gemm * 3;                                          // MSE: one double per tile and phase
        const size_t ce_part = std::max((size_t)2 * L.n_tokens, (size_t)6 * ((L.n_tokens + kCeCombineTokens - 1) / kCeCombineTokens));   // CE: (sum, count) pairs
        if (ce && ce_part > part) part = ce_part;
        p.part_count = part;
        p.off_part = take(part * 8);
    }
    p.off_ce_ms = take((ce && bf) ? (size_t)3 * gemm_bf16_ce_chunks(L.d_out) * L.n_tokens * 8 : 0);
    p.off_ce_tl = take((ce && bf) ? (size_t)3 * L.n_tokens * 4 : 0);
    p.off_upd = take(update_workspace_bytes(L.dtype, L.d_out, L.d_in, L.r));
    p.off_ext = take(bf ? gemm_bf16_ext_bytes(L.n_tokens, L.d_out, L.r) : 0);
    p.off_xqpart = take(bf ? xq_part_bytes(L.n_tokens, L.d_in, p.rp) : 0);
    p.off_Ybuf = take(need_ybuf ? (size_t)L.n_tokens * L.d_out * 4 : 0);
    p.off_split = 0;
    p.total = o;
    return p;
}

// with the scratch of a lone stored output (the forwards that a model makes layer by layer; Y may be NULL)
Plan make_forward_plan(const agzo_layer& L, const agzo_loss_spec* loss, bool fused_sketch, const void* W, const void* X, const void* Y) {
    const bool ce = loss && loss->kind == AGZO_LOSS_CE, stored = Y && L.dtype == AGZO_BF16 && L.y_dtype == AGZO_BF16 && (!loss || loss->kind == AGZO_LOSS_NONE);
    // where Y lies in X or W, few tiles are shares again: the launch that adds them stores behind every read
    auto rows = [](const void* at, int64_t ld, int64_t n, int64_t d) { return Rows{reinterpret_cast<uintptr_t>(at), 2 * ld, n, 2 * d}; };
    const Rows y = rows(Y, L.ldy, L.n_tokens, L.d_out);
    const bool over = stored && (rows_overlap(y, rows(X, L.ldx, L.n_tokens, L.d_in)) || rows_overlap(y, rows(W, L.ldw, L.d_out, L.d_in)));
    const bool few = stored && !over && gemm_bf16_few_tiles(L.n_tokens, L.d_out, L.d_in, L.tiling == AGZO_TILING_LARGE);
    Plan p = make_plan(L, W && L.dtype == AGZO_F32 && !Y && ce, ce, false, 0, !fused_sketch ? 0 : few ? 64 : 128);
    const size_t split = stored ? gemm_bf16_split_bytes(L.n_tokens, L.d_out, L.d_in, over) : 0;
    if (split) {
        p.off_split = p.total;
        p.total += align_up(split);
    }
    return p;
}

// wish: what a growth is to cover as well where there is room (grow.h)
int reserve(agzo_ctx* ctx, size_t bytes, size_t wish = 0) {
    if (bytes <= ctx->ws_bytes) return 0;
    HIPCHK(hipStreamSynchronize(ctx->stream));
    if (ctx->side) HIPCHK(hipStreamSynchronize(ctx->side));      // (joined to the above, unless joining failed)
    if (ctx->ws) HIPCHK(hipFree(ctx->ws));
    const size_t had = ctx->ws_bytes;
    ctx->ws = nullptr;
    ctx->ws_bytes = 0;
    void* p = nullptr;
    hipError_t e = hipSuccess;
    const size_t got = grow(had, bytes, wish, [&](size_t n) {
        if (e != hipSuccess) (void)hipGetLastError();      // (of the attempt before)
        e = hipMalloc(&p, n);
        return e == hipSuccess;
    });
    if (!got) return fail(ctx, AGZO_ENOMEM, "workspace of %zu bytes: %s", bytes, hipGetErrorString(e));
    ctx->ws = static_cast<char*>(p);
    ctx->ws_bytes = got;
    return 0;
}

int check_layer(agzo_ctx* ctx, const agzo_layer* L, bool need_w) {
    if (!ctx) return AGZO_EINVAL;
    if (!L) return fail(ctx, AGZO_EINVAL, "layer descriptor is NULL");
    if (L->n_tokens < 1 || L->d_in < 1 || (need_w && L->d_out < 1))
        return fail(ctx, AGZO_EINVAL, "empty layer: n_tokens=%lld d_in=%lld d_out=%lld", (long long)L->n_tokens,
                    (long long)L->d_in, (long long)L->d_out);
    if (L->n_tokens > (1LL << 24) || L->d_in > (1LL << 24) || L->d_out > (1LL << 24))
        return fail(ctx, AGZO_EINVAL, "dimension above 2^24");
    if (L->r < 1 || L->r > kMaxRank) return fail(ctx, AGZO_EINVAL, "r=%d outside 1..%d", L->r, kMaxRank);
    if (L->r > L->n_tokens || L->r > L->d_in) return fail(ctx, AGZO_EINVAL, "r=%d exceeds min(n_tokens, d_in)", L->r);
    if (L->dtype != AGZO_F32 && L->dtype != AGZO_BF16) return fail(ctx, AGZO_EINVAL, "dtype %d", L->dtype);
    if (L->tiling != AGZO_TILING_AUTO && L->tiling != AGZO_TILING_LARGE) return fail(ctx, AGZO_EINVAL, "tiling %d", L->tiling);
    if (L->ldx < L->d_in || (need_w && L->ldw < L->d_in)) return fail(ctx, AGZO_EINVAL, "leading dimension below d_in");
    if (L->dtype == AGZO_BF16) {
        if (L->d_in % 8 || L->ldx % 8 || (need_w && L->ldw % 8))
            return fail(ctx, AGZO_EINVAL, "bf16 layers need d_in, ldx, ldw multiples of 8");
    }
    return 0;
}

// bf16 operands travel as 16-byte vectors (direct global -> LDS loads included) and the kernels build 32-bit byte
// offsets of up to 512 rows from a tile's corner
int check_operands(agzo_ctx* ctx, const agzo_layer* L, const void* W, const void* X) {
    if (L->dtype != AGZO_BF16) return 0;
    if ((reinterpret_cast<uintptr_t>(X) & 15) || (reinterpret_cast<uintptr_t>(W) & 15))
        return fail(ctx, AGZO_EINVAL, "bf16 X and W must be 16-byte aligned");
    if (L->ldx >= (1LL << 22) || (W && L->ldw >= (1LL << 22)))
        return fail(ctx, AGZO_EINVAL, "bf16 layers need ldx and ldw below 2^22 elements");
    return 0;
}

int check_y(agzo_ctx* ctx, const agzo_layer* L, const void* Y) {
    if (!Y) return 0;
    if (L->ldy < L->d_out) return fail(ctx, AGZO_EINVAL, "ldy below d_out");
    if (L->y_dtype == AGZO_F32) return 0;
    if (L->y_dtype == AGZO_BF16 && L->dtype == AGZO_BF16) return 0;
    return fail(ctx, AGZO_EINVAL, "y_dtype %d not supported for layer dtype %d", L->y_dtype, L->dtype);
}

int check_loss(agzo_ctx* ctx, const agzo_layer* L, const agzo_loss_spec* loss, const double* loss_dev) {
    if (!loss || loss->kind == AGZO_LOSS_NONE) return 0;
    if (loss->kind != AGZO_LOSS_MSE && loss->kind != AGZO_LOSS_CE)
        return fail(ctx, AGZO_EINVAL, "loss kind %d not supported", loss->kind);
    if (!loss->target || !loss_dev) return fail(ctx, AGZO_EINVAL, "loss needs a target and an output scalar");
    if (loss->kind == AGZO_LOSS_CE) return 0;
    if (loss->ldt < L->d_out) return fail(ctx, AGZO_EINVAL, "ldt below d_out");
    if (loss->target_dtype != AGZO_F32 && loss->target_dtype != AGZO_BF16)
        return fail(ctx, AGZO_EINVAL, "target dtype %d", loss->target_dtype);
    return 0;
}

struct HipApi {
    typedef hipStream_t stream_t;
    typedef hipEvent_t event_t;
    typedef hipError_t error_t;
    static hipError_t record(hipEvent_t e, hipStream_t s) { return hipEventRecord(e, s); }
    static hipError_t wait(hipStream_t s, hipEvent_t e) { return hipStreamWaitEvent(s, e, 0); }
    static hipError_t synchronize(hipStream_t s) { return hipStreamSynchronize(s); }
};

// ---- internal building blocks; all take a ready workspace plan --------------------------------
inline float* wsf(agzo_ctx* c, size_t off) { return reinterpret_cast<float*>(c->ws + off); }
inline bf16_t* wsh(agzo_ctx* c, size_t off) { return reinterpret_cast<bf16_t*>(c->ws + off); }

// ---- sketches.  On the bf16 path a sketch first exists as per-token-range partials in the workspace
// (`splits`); they are summed either by the QR that consumes them or, when the caller wants S itself,
// by reduce_splits.  On the fp32 path S is produced directly.

// Omega^T planes -> splits (bf16) / S (fp32):  S = X^T Omega  (Alg. 1: Y <- H Omega)
int sketch_range(agzo_ctx* ctx, const agzo_layer& L, const Plan& p, const void* X, uint64_t seed, float* S) {
    hipStream_t st = ctx->stream;
    if (L.dtype == AGZO_BF16) {
        {
            ProfScope ps(ctx, AGZO_PROF_FILL);
            HIPCHK(launch_fill_normal_packT(wsh(ctx, p.off_TpackT), L.n_tokens, p.m_pad, L.r, p.rp, seed, AGZO_TAG_OMEGA, st));
        }
        ProfScope ps(ctx, AGZO_PROF_XTT);
        HIPCHK(launch_xtt_bf16(static_cast<const bf16_t*>(X), L.ldx, L.n_tokens, L.d_in, wsh(ctx, p.off_TpackT),
                               p.m_pad, p.rp, wsf(ctx, p.off_xtt), p.nsplit, st));
    } else {
        float* om = wsf(ctx, p.off_T);
        HIPCHK(launch_fill_normal(om, L.n_tokens, L.r, seed, AGZO_TAG_OMEGA, st));
        const F32SkinnyArgs a{static_cast<const float*>(X), L.ldx, L.n_tokens, L.d_in, om, L.r, S};
        HIPCHK(launch_xtt_f32_many(&a, 1, st));
    }
    return 0;
}

// whether the products X Q of a layer read Q as planes
bool reads_planes(const agzo_layer& L) { return L.dtype == AGZO_BF16 && !xq_narrow(L.n_tokens, L.d_in, L.r); }

// S = X^T (X Q)  (Alg. 1: Y <- H (H^T Q)).  Where it is read as planes, Q must already sit in the workspace as such.
int sketch_power(agzo_ctx* ctx, const agzo_layer& L, const Plan& p, const void* X, const float* Q, float* S) {
    hipStream_t st = ctx->stream;
    if (L.dtype == AGZO_BF16) {
        {
            ProfScope ps(ctx, AGZO_PROF_XQ);
            const XqArgs q{static_cast<const bf16_t*>(X), L.ldx, L.n_tokens, L.d_in, wsh(ctx, p.off_pack), L.r, p.rp, nullptr,
                           wsh(ctx, p.off_TpackT), p.m_pad, wsf(ctx, p.off_xqpart), nullptr, Q};
            HIPCHK(launch_xq_bf16_many(&q, 1, false, st));
        }
        ProfScope ps(ctx, AGZO_PROF_XTT);
        HIPCHK(launch_xtt_bf16(static_cast<const bf16_t*>(X), L.ldx, L.n_tokens, L.d_in, wsh(ctx, p.off_TpackT),
                               p.m_pad, p.rp, wsf(ctx, p.off_xtt), p.nsplit, st));
    } else {
        const float* Xf = static_cast<const float*>(X);
        float* T = wsf(ctx, p.off_T);
        const F32SkinnyArgs q{Xf, L.ldx, L.n_tokens, L.d_in, Q, L.r, T}, t{Xf, L.ldx, L.n_tokens, L.d_in, T, L.r, S};
        HIPCHK(launch_xq_f32_many(&q, 1, st));
        HIPCHK(launch_xtt_f32_many(&t, 1, st));
    }
    return 0;
}

int reduce_to_S(agzo_ctx* ctx, const agzo_layer& L, const Plan& p, float* S) {
    if (L.dtype == AGZO_BF16)
        HIPCHK(launch_reduce_splits(wsf(ctx, p.off_xtt), p.nsplit, L.d_in, p.rp, L.r, S, ctx->stream));
    return 0;
}

// Q = qr(S) for an explicit S
int op_qr(agzo_ctx* ctx, size_t off_qr, const float* S, int64_t d, int r, int rp, float* Q) {
    ProfScope ps(ctx, AGZO_PROF_QR);
    HIPCHK(launch_qr(S, nullptr, 0, rp, nullptr, d, r, Q, nullptr, ctx->ws + off_qr, ctx->flag, true, ctx->stream));
    return 0;
}

GemmBf16Args forward_bf16_args(agzo_ctx* ctx, const agzo_layer& L, const Plan& p, const void* W, const void* X, const float* P,
                               float eps_signed, uint64_t seed, void* Y, const GemmLossArgs& loss, bool shared) {
    GemmBf16Args a;
    a.X = static_cast<const bf16_t*>(X); a.ldx = L.ldx;
    a.W = static_cast<const bf16_t*>(W); a.ldw = L.ldw;
    a.M = L.n_tokens; a.N = L.d_out; a.K = L.d_in;
    a.Y = Y; a.y_dtype = L.y_dtype; a.ldy = L.ldy;
    a.P = P; a.r = L.r; a.eps_signed = eps_signed; a.seed = seed;
    a.loss = loss;
    a.shared = shared;
    a.large_tiles = (L.tiling == AGZO_TILING_LARGE);
    a.ext_ws = P ? ctx->ws + p.off_ext : nullptr;
    a.split_ws = p.off_split ? ctx->ws + p.off_split : nullptr;
    if (timed(ctx, AGZO_PROF_GEMM) && ctx->clk_used < kClkSlots) a.clk = ctx->clk + 4 * ctx->clk_used++;
    return a;
}

F32FwdArgs forward_f32_args(const agzo_layer& L, const void* W, const void* X, const float* P, float eps_signed, uint64_t seed,
                            const GemmLossArgs& loss, bool shared) {
    F32FwdArgs a;
    a.X = static_cast<const float*>(X); a.ldx = L.ldx;
    a.W = static_cast<const float*>(W); a.ldw = L.ldw;
    a.M = L.n_tokens; a.N = L.d_out; a.K = L.d_in;
    a.Y = nullptr; a.ldy = 0;
    a.P = P; a.r = L.r; a.eps_signed = eps_signed; a.s_lo = (uint32_t)seed; a.s_hi = (uint32_t)(seed >> 32);
    a.target = (loss.kind == AGZO_LOSS_MSE) ? loss.target : nullptr;
    a.target_dtype = loss.target_dtype; a.ldt = loss.ldt; a.partials = loss.partials;
    a.shared = shared ? 1 : 0;
    return a;
}

// a forward that is launched on another stream than the context's, on so many compute units of each XCD
struct SideForward { hipStream_t stream; int slots; };

// Y = X W^T (+ eps (P) G^T), loss
// shared = true: one pass over X and W evaluates the loss at W, W + eps Z, W - eps Z -> loss_dev[0..2]
int op_forward(agzo_ctx* ctx, const agzo_layer& L, const Plan& p, const void* W, const void* X, const float* P,
               float eps_signed, uint64_t seed, void* Y, const agzo_loss_spec* loss, double* loss_dev,
               bool shared = false, int part_slot = 0, bool defer_finish = false, bool fused_sketch = false, bool ext_ready = false, int ext_side = 0,
               const SideForward* side = nullptr) {
    hipStream_t st = side ? side->stream : ctx->stream;
    GemmLossArgs la;
    const bool has_loss = loss && loss->kind != AGZO_LOSS_NONE;
    la.kind = has_loss ? loss->kind : AGZO_LOSS_NONE;
    la.target_dtype = has_loss ? loss->target_dtype : AGZO_F32;
    la.target = has_loss ? loss->target : nullptr;
    la.ldt = has_loss ? loss->ldt : 0;
    const bool ce = has_loss && loss->kind == AGZO_LOSS_CE;
    // squared error: a step keeps the tile partials of its forwards side by side (slot = 0, 1, 2) and finishes them in
    // one launch.  Cross-entropy: every loss is finished by launches of its own right behind the forward; with fp32 storage all of
    // them use the region from its start, (sum, count) per token, with bf16, where a forward may run beside the others, slot by slot,
    // (sum, count) per kCeCombineTokens tokens and phase.
    {
        const size_t nblk = (size_t)((L.n_tokens + kCeCombineTokens - 1) / kCeCombineTokens);
        const size_t at = !ce ? (size_t)part_slot * p.n_part : L.dtype == AGZO_BF16 ? 2 * nblk * part_slot : 0;
        const size_t need = !has_loss ? 0 : ce ? (L.dtype == AGZO_BF16 ? 2 * nblk * (shared ? 3 : 1) : 2 * (size_t)L.n_tokens)
                                               : (size_t)p.n_part * (shared ? 3 : 1);
        if (at + need > p.part_count)
            return fail(ctx, AGZO_EHIP, "internal: loss scratch of %zu doubles at %zu exceeds its region of %zu", need, at,
                        p.part_count);
        la.partials = reinterpret_cast<double*>(ctx->ws + p.off_part) + at;
    }
    const int32_t* ids = ce ? static_cast<const int32_t*>(loss->target) : nullptr;
    if (ce && L.dtype == AGZO_BF16) {
        la.ce_ms = ctx->ws + p.off_ce_ms + (size_t)part_slot * gemm_bf16_ce_chunks(L.d_out) * L.n_tokens * 8;
        la.ce_tl = wsf(ctx, p.off_ce_tl) + (size_t)part_slot * L.n_tokens;
    }
    if (L.dtype == AGZO_BF16) {
        GemmBf16Args a = forward_bf16_args(ctx, L, p, W, X, P, eps_signed, seed, Y, la, shared);
        a.ext_ready = ext_ready;
        a.ext_side = ext_side;
        if (side) a.slots = side->slots;
        if (fused_sketch) { a.sk_T = wsh(ctx, p.off_TpackT); a.sk_mpad = p.m_pad; a.sk_partial = wsf(ctx, p.off_xtt); a.sk_tokens = p.sketch_tokens; }
        {
            ProfScope ps(ctx, AGZO_PROF_GEMM);
            HIPCHK(launch_gemm_bf16(a, st));
        }
        if (ce)
            HIPCHK(launch_ce_combine(la.ce_ms, la.ce_tl, ids, L.n_tokens, L.d_out, gemm_bf16_ce_chunks(L.d_out), shared ? 3 : 1,
                                     la.partials, loss_dev, st));
    } else {
        F32FwdArgs a = forward_f32_args(L, W, X, P, eps_signed, seed, la, shared);
        if (!ce) {
            a.Y = static_cast<float*>(Y); a.ldy = L.ldy;
            HIPCHK(launch_forward_f32_many(&a, 1, st));
        } else {
            // the logits go through memory: Y, or the workspace
            a.Y = Y ? static_cast<float*>(Y) : wsf(ctx, p.off_Ybuf);
            a.ldy = Y ? L.ldy : L.d_out;
            if (shared) { a.P = nullptr; a.shared = 0; }
            HIPCHK(launch_forward_f32_many(&a, 1, st));
            HIPCHK(launch_ce_rows_f32(a.Y, a.ldy, L.n_tokens, L.d_out, ids, la.partials, loss_dev, st));
            for (int ph = 1; shared && ph < 3; ++ph) {      // Y0 + eps D, then - 2 eps D
                HIPCHK(launch_rank_term_f32(a.Y, a.ldy, L.n_tokens, L.d_out, P, L.r, ph == 1 ? eps_signed : -2.f * eps_signed, seed, st));
                HIPCHK(launch_ce_rows_f32(a.Y, a.ldy, L.n_tokens, L.d_out, ids, la.partials, loss_dev + ph, st));
            }
        }
    }
    if (has_loss && !ce && !defer_finish)
        HIPCHK(launch_finish_loss(la.partials, p.n_part, 1.0 / ((double)L.n_tokens * (double)L.d_out), loss_dev,
                                  shared ? 3 : 1, st));
    return 0;
}

int check_update(agzo_ctx* ctx, const void* W, const float* B, int dtype, int64_t d_out, int64_t d_in, int64_t ldw, int r) {
    if (!W || !B) return fail(ctx, AGZO_EINVAL, "W or B is NULL");
    if (d_in < 1 || d_out < 1 || r < 1 || r > kMaxRank || r > d_in || ldw < d_in)
        return fail(ctx, AGZO_EINVAL, "bad layer shape");
    if (dtype != AGZO_F32 && dtype != AGZO_BF16) return fail(ctx, AGZO_EINVAL, "dtype %d", dtype);
    if (dtype == AGZO_BF16 && (d_in % 8 || ldw % 8 || (reinterpret_cast<uintptr_t>(W) & 15)))
        return fail(ctx, AGZO_EINVAL, "bf16 W needs d_in and ldw multiples of 8 and 16-byte aligned rows");
    if (dtype == AGZO_BF16 && ldw >= (1LL << 28)) return fail(ctx, AGZO_EINVAL, "bf16 W: ldw must be below 2^28");
    return 0;
}

int op_update(agzo_ctx* ctx, const agzo_layer& L, size_t off_upd, void* W, const float* B, uint64_t seed, float lr,
              const double* g_dev, float shift = 0.f) {
    ProfScope ps(ctx, AGZO_PROF_UPDATE);
    HIPCHK(launch_update(W, L.dtype, L.ldw, L.d_out, L.d_in, B, L.r, seed, lr, g_dev, ctx->ws + off_upd, ctx->stream, shift));
    return 0;
}

// ---- several layers at once (Alg. 2: the base forward computes every layer's basis before the perturbed passes; the
// extractions are independent, so every stage of Alg. 1 is one launch for all layers) ----
struct LayerJob {
    agzo_layer L;
    Plan p;
    const void* X;
    uint64_t seed;
    const float* S0;
    float* B;          // where the basis goes
};

// the same for fp32 storage: S (or T and S) of every job in the workspace
int stage_sketch_many_f32(agzo_ctx* ctx, const std::vector<LayerJob>& jobs, const int* idx, int n, bool range, const float* const* raw) {
    FillNormalArgs f[kBatchMax];
    F32SkinnyArgs q[kBatchMax], t[kBatchMax];
    for (int i = 0; i < n; ++i) {
        const LayerJob& j = jobs[idx[i]];
        const float* X = static_cast<const float*>(j.X);
        f[i] = FillNormalArgs{wsf(ctx, j.p.off_T), j.L.n_tokens, j.L.r, j.seed};
        q[i] = F32SkinnyArgs{X, j.L.ldx, j.L.n_tokens, j.L.d_in, raw && raw[i] ? raw[i] : wsf(ctx, j.p.off_Q), j.L.r, wsf(ctx, j.p.off_T),
                             raw && raw[i] ? ctx->flag : nullptr};
        t[i] = F32SkinnyArgs{X, j.L.ldx, j.L.n_tokens, j.L.d_in, wsf(ctx, j.p.off_T), j.L.r, wsf(ctx, j.p.off_S)};
    }
    if (range) HIPCHK(launch_fill_normal_many(f, n, AGZO_TAG_OMEGA, ctx->stream));
    else HIPCHK(launch_xq_f32_many(q, n, ctx->stream));
    HIPCHK(launch_xtt_f32_many(t, n, ctx->stream));
    return 0;
}

// one stage for the jobs idx[0..n) (one dtype): Omega^T planes + range sketch, or T = X Q planes + power sketch
// raw (power sketch; nullable): per job of idx the column that the last factorisation left to be normalised, NULL where Q is ready.  summed: where the
// partial sums of that column are all there is
// half_cu (here and below): forwards on another stream may hold half of every compute unit
int stage_sketch_many(agzo_ctx* ctx, const std::vector<LayerJob>& jobs, const int* idx, int n, bool range, bool half_cu, const float* const* raw = nullptr, const bool* summed = nullptr) {
    if (n > 0 && jobs[idx[0]].L.dtype != AGZO_BF16) return stage_sketch_many_f32(ctx, jobs, idx, n, range, raw);
    hipStream_t st = ctx->stream;
    if (range) {
        FillPackTArgs f[kBatchMax];
        for (int i = 0; i < n; ++i) {
            const LayerJob& j = jobs[idx[i]];
            f[i] = FillPackTArgs{wsh(ctx, j.p.off_TpackT), j.L.n_tokens, j.p.m_pad, j.L.r, j.p.rp, j.seed, AGZO_TAG_OMEGA};
        }
        ProfScope ps(ctx, AGZO_PROF_FILL);
        HIPCHK(launch_fill_normal_packT_many(f, n, st));
    } else {
        XqArgs q[kBatchMax];
        for (int i = 0; i < n; ++i) {
            const LayerJob& j = jobs[idx[i]];
            q[i] = XqArgs{static_cast<const bf16_t*>(j.X), j.L.ldx, j.L.n_tokens, j.L.d_in, wsh(ctx, j.p.off_pack), j.L.r, j.p.rp,
                          nullptr, wsh(ctx, j.p.off_TpackT), j.p.m_pad, wsf(ctx, j.p.off_xqpart), nullptr, wsf(ctx, j.p.off_Q)};
            if (summed && summed[i]) {
                q[i].Q = nullptr;
                q[i].splits = wsf(ctx, j.p.off_xtt);
                q[i].nsplit = j.p.nsplit;
                q[i].flag = ctx->flag;
            } else if (raw && raw[i]) {
                q[i].Q = raw[i];
                q[i].norm2 = reinterpret_cast<const double*>(ctx->ws + j.p.off_qr);
                q[i].norm_blocks = qr_norm_blocks(j.L.d_in);
                q[i].flag = ctx->flag;
            }
        }
        ProfScope ps(ctx, AGZO_PROF_XQ);
        HIPCHK(launch_xq_bf16_many(q, n, half_cu, st));
    }
    XttArgs t[kBatchMax];
    for (int i = 0; i < n; ++i) {
        const LayerJob& j = jobs[idx[i]];
        t[i] = XttArgs{static_cast<const bf16_t*>(j.X), j.L.ldx, j.L.n_tokens, j.L.d_in, wsh(ctx, j.p.off_TpackT), j.p.m_pad, j.p.rp,
                       wsf(ctx, j.p.off_xtt), j.p.nsplit, j.L.r == 1};
    }
    ProfScope ps(ctx, AGZO_PROF_XTT);
    HIPCHK(launch_xtt_bf16_many(t, n, half_cu, st));
    return 0;
}

// Alg. 1 for every job.  Jobs that share a dtype and a padded rank go through the batched kernels, at most kBatchMax per
// launch.  On return the workspace planes of every job that reads them hold its basis.
int basis_many_impl(agzo_ctx* ctx, const std::vector<LayerJob>& jobs, int K, int flags, bool half_cu = false) {
    std::vector<char> done(jobs.size(), 0);
    for (size_t a = 0; a < jobs.size(); ++a) {
        if (done[a]) continue;
        const LayerJob& ja = jobs[a];
        const bool bf = ja.L.dtype == AGZO_BF16;
        int idx[kBatchMax], n = 0;
        // (single columns are normalised rather than factored: launches of their own)
        for (size_t b = a; b < jobs.size() && n < kBatchMax; ++b)
            if (!done[b] && jobs[b].L.dtype == ja.L.dtype && jobs[b].p.rp == ja.p.rp && (jobs[b].L.r == 1) == (ja.L.r == 1)) {
                idx[n++] = (int)b;
                done[b] = 1;
            }
        // first sketch: the feature-space start (Q0 from the seed, then a power sketch), a given S0, or the range sketch
        bool given[kBatchMax];
        int need_idx[kBatchMax], n_need = 0;
        for (int i = 0; i < n; ++i) {
            const LayerJob& j = jobs[idx[i]];
            given[i] = false;
            if (flags & AGZO_INIT_FEATURE) {
                HIPCHK(launch_fill_normal(wsf(ctx, j.p.off_Q), j.L.d_in, j.L.r, j.seed, AGZO_TAG_Q0, ctx->stream));
                if (reads_planes(j.L)) HIPCHK(launch_pack_planes(wsf(ctx, j.p.off_Q), j.L.d_in, j.L.r, j.p.rp, wsh(ctx, j.p.off_pack), ctx->stream));
                need_idx[n_need++] = idx[i];
            } else if (j.S0) {
                given[i] = true;
            } else {
                need_idx[n_need++] = idx[i];
            }
        }
        if (n_need) TRY(stage_sketch_many(ctx, jobs, need_idx, n_need, !(flags & AGZO_INIT_FEATURE), half_cu));
        for (int k = 0; k <= K; ++k) {
            QrArgs q[kBatchMax];
            const float* raw[kBatchMax];
            bool summed[kBatchMax];
            int nq = 0;
            for (int i = 0; i < n; ++i) {
                const LayerJob& j = jobs[idx[i]];
                // a single column between power steps: the projection that follows normalises its result, one launch less, and a short one it also adds up
                const bool defer = bf && k < K && xq_narrow(j.L.n_tokens, j.L.d_in, j.L.r), partials = bf && !(k == 0 && given[i]);
                summed[i] = n == 1 && defer && partials && xq_sums_column(j.L.n_tokens, j.L.d_in, j.p.nsplit);
                raw[i] = nullptr;
                if (summed[i]) continue;
                if (!bf && k < K && j.L.r == 1) {                // (and with fp32 storage, where the sums are in fp64, it finds the norm as well)
                    raw[i] = k == 0 && given[i] ? j.S0 : wsf(ctx, j.p.off_S);
                    continue;
                }
                float* out = (k == K) ? j.B : wsf(ctx, j.p.off_Q);
                bf16_t* planes = reads_planes(j.L) ? wsh(ctx, j.p.off_pack) : nullptr;
                QrArgs& one = q[nq++];
                if (!partials)
                    one = QrArgs{(k == 0 && given[i]) ? j.S0 : wsf(ctx, j.p.off_S), nullptr, 0, j.p.rp, nullptr, j.L.d_in, j.L.r, out,
                                 planes, ctx->ws + j.p.off_qr};
                else
                    one = QrArgs{nullptr, wsf(ctx, j.p.off_xtt), j.p.nsplit, j.p.rp, wsf(ctx, j.p.off_S), j.L.d_in, j.L.r, out,
                                 planes, ctx->ws + j.p.off_qr};
                one.defer = defer;
                if (defer) raw[i] = one.splits ? one.S_out : one.S;
            }
            if (nq) {
                ProfScope ps(ctx, AGZO_PROF_QR);
                HIPCHK(launch_qr_many(q, nq, ctx->flag, k == K, ctx->stream));
            }
            if (k < K) TRY(stage_sketch_many(ctx, jobs, idx, n, false, half_cu, raw, summed));
        }
    }
    return 0;
}

// Alg. 1 for one layer
int op_basis(agzo_ctx* ctx, const agzo_layer& L, const Plan& p, const void* X, int K, uint64_t seed, const float* S0, int flags, float* B) {
    try {
        return basis_many_impl(ctx, {LayerJob{L, p, X, seed, S0, B}}, K, flags);
    } catch (const std::bad_alloc&) {      // (below a C entry)
        return fail(ctx, AGZO_ENOMEM, "no host memory for the list of one layer");
    }
}

// P = X B for every job (one launch per kBatchMax jobs of a dtype and padded rank, and one behind it), behind basis_many_impl.  ext: the
// W sides of the jobs' extension operands, which the same launches write with the X sides (ext_ws = NULL: neither)
int project_many(agzo_ctx* ctx, const std::vector<LayerJob>& jobs, const std::vector<GemmExtArgs>& ext, bool half_cu) {
    std::vector<char> done(jobs.size(), 0);
    for (size_t a = 0; a < jobs.size(); ++a) {
        if (done[a]) continue;
        const LayerJob& ja = jobs[a];
        if (ja.L.dtype != AGZO_BF16) {
            F32SkinnyArgs s[kBatchMax];
            int n = 0;
            for (size_t b = a; b < jobs.size() && n < kBatchMax; ++b) {
                const LayerJob& j = jobs[b];
                if (done[b] || j.L.dtype == AGZO_BF16 || j.p.rp != ja.p.rp) continue;
                s[n++] = F32SkinnyArgs{static_cast<const float*>(j.X), j.L.ldx, j.L.n_tokens, j.L.d_in, j.B, j.L.r, wsf(ctx, j.p.off_T)};
                done[b] = 1;
            }
            HIPCHK(launch_xq_f32_many(s, n, ctx->stream));
            continue;
        }
        XqArgs q[kBatchMax];
        int n = 0;
        for (size_t b = a; b < jobs.size() && n < kBatchMax; ++b) {
            const LayerJob& j = jobs[b];
            if (done[b] || j.L.dtype != AGZO_BF16 || j.p.rp != ja.p.rp) continue;
            q[n++] = XqArgs{static_cast<const bf16_t*>(j.X), j.L.ldx, j.L.n_tokens, j.L.d_in, wsh(ctx, j.p.off_pack), j.L.r, j.p.rp,
                            wsf(ctx, j.p.off_T), nullptr, j.p.m_pad, wsf(ctx, j.p.off_xqpart), nullptr, j.B};
            if (ext[b].ext_ws) {
                q[n - 1].Xext = static_cast<bf16_t*>(ext[b].ext_ws);
                q[n - 1].ext = &ext[b];
            }
            done[b] = 1;
        }
        ProfScope ps(ctx, AGZO_PROF_XQ);
        HIPCHK(launch_xq_bf16_many(q, n, half_cu, ctx->stream));
    }
    return 0;
}

// checked items, workspace reserved: the factor fragments of all matrices start at workspace offset `off`.
// fp32 matrices (no workspace) update_many_max() to a launch; bf16 matrices with r = 1 in rank-1 sweeps of up to kBatchMax per launch (no
// workspace); the other bf16 matrices by padded rank, update_many_max() to a pair of launches
int update_many_at(agzo_ctx* ctx, const agzo_update_item* items, int n, size_t off) {
    for (int nk = -1; nk <= (kMaxRank + 15) / 16; ++nk) {
        std::vector<UpdateDesc> group;
        size_t group_bytes = 0;
        const int cap = (nk == 0) ? kBatchMax : update_many_max();
        auto flush = [&]() -> int {
            if (group.empty()) return 0;
            ProfScope ps(ctx, AGZO_PROF_UPDATE);
            if (nk < 0) {
                HIPCHK(launch_update_f32_many(group.data(), (int)group.size(), ctx->stream));
            } else if (nk == 0) {
                HIPCHK(launch_update_rank1_many(group.data(), (int)group.size(), ctx->stream));
            } else {
                HIPCHK(launch_update_many(group.data(), (int)group.size(), nk, ctx->ws + off, ctx->stream));
                off += group_bytes;
            }
            group.clear();
            group_bytes = 0;
            return 0;
        };
        for (int m = 0; m < n; ++m) {
            const agzo_update_item& u = items[m];
            if ((nk < 0) != (u.dtype == AGZO_F32)) continue;
            if (nk >= 0 && (nk == 0 ? u.r != 1 : (u.r == 1 || (u.r + 15) / 16 != nk))) continue;
            group.push_back(UpdateDesc{u.W, u.B, u.g_dev, u.ldw, u.d_out, u.d_in, u.seed, u.lr, u.r});
            if (nk > 0) group_bytes += update_workspace_bytes(u.dtype, u.d_out, u.d_in, u.r);
            if ((int)group.size() == cap) TRY(flush());
        }
        TRY(flush());
    }
    return AGZO_OK;
}

}  // namespace

extern "C" {

int agzo_create(agzo_ctx** out, void* hip_stream) {
    if (!out) return AGZO_EINVAL;
    agzo_ctx* ctx = new (std::nothrow) agzo_ctx;
    if (!ctx) return AGZO_ENOMEM;
    ctx->stream = static_cast<hipStream_t>(hip_stream);
    ctx->err[0] = 0;
    ctx->ws = nullptr;
    ctx->ws_bytes = 0;
    ctx->flag = nullptr;
    ctx->prof = 0;
    ctx->clk = nullptr;
    ctx->clk_used = 0;
    ctx->side = nullptr;
    ctx->fork = ctx->join = nullptr;
    ctx->device = -1;
    ctx->static_scratch = nullptr;
    hipError_t e = hipGetDevice(&ctx->device);
    if (e == hipSuccess) e = resolve_scratch(ctx->device, &ctx->static_scratch);
    if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&ctx->flag), 256);
    if (e == hipSuccess) e = hipMemset(ctx->flag, 0, 256);
    if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&ctx->clk), kClkBytes);
    if (e == hipSuccess) e = hipMemset(ctx->clk, 0, kClkBytes);
    // (Non-blocking: the context's stream may be the default stream, which others would otherwise wait for.  Made here although few
    // contexts use it, 23 us of 33, and not by the first call that does: what follows the making of a stream is faster on the context's own
    // too, the dense estimator over seven 0.6B-sized layers 426 us a pass and 434 without, its first pass 0.9 ms and 1.35)
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ctx->fork, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ctx->join, hipEventDisableTiming);
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&ctx->side, hipStreamNonBlocking);
    if (e != hipSuccess) {
        if (ctx->flag) (void)hipFree(ctx->flag);
        if (ctx->clk) (void)hipFree(ctx->clk);
        if (ctx->fork) (void)hipEventDestroy(ctx->fork);
        if (ctx->join) (void)hipEventDestroy(ctx->join);
        delete ctx;
        return AGZO_EHIP;
    }
    *out = ctx;
    return AGZO_OK;
}

void agzo_destroy(agzo_ctx* ctx) {
    if (!ctx) return;
    (void)hipStreamSynchronize(ctx->stream);
    if (ctx->side) {
        (void)hipStreamSynchronize(ctx->side);    // (joined to the above, unless joining failed)
        (void)hipStreamDestroy(ctx->side);
    }
    if (ctx->fork) (void)hipEventDestroy(ctx->fork);
    if (ctx->join) (void)hipEventDestroy(ctx->join);
    if (ctx->ws) (void)hipFree(ctx->ws);
    if (ctx->flag) (void)hipFree(ctx->flag);
    if (ctx->clk) (void)hipFree(ctx->clk);
    for (auto& pc : ctx->pc) {
        for (hipEvent_t e : pc.start) (void)hipEventDestroy(e);
        for (hipEvent_t e : pc.stop) (void)hipEventDestroy(e);
    }
    delete ctx;
}

const char* agzo_last_error(const agzo_ctx* ctx) { return ctx ? ctx->err : "null context"; }

int agzo_check(agzo_ctx* ctx) {
    if (!ctx) return AGZO_EINVAL;
    HIPCHK(hipStreamSynchronize(ctx->stream));
    int h = 0;
    HIPCHK(hipMemcpy(&h, ctx->flag, sizeof(int), hipMemcpyDeviceToHost));
    if (h) {
        HIPCHK(hipMemset(ctx->flag, 0, sizeof(int)));
        return fail(ctx, AGZO_ENUMERIC, "Cholesky pivot <= 0: the sketch is rank deficient");
    }
    return AGZO_OK;
}

int agzo_profile_enable(agzo_ctx* ctx, int32_t mask) {
    if (!ctx) return AGZO_EINVAL;
    HIPCHK(hipStreamSynchronize(ctx->stream));
    ctx->prof = (uint32_t)mask & ((1u << AGZO_PROF_KINDS) - 1u);
    for (auto& pc : ctx->pc) pc.used = 0;
    ctx->clk_used = 0;
    return AGZO_OK;
}

namespace {
// rate of the constant counter that wall_clock64() reads, in Hz
int wall_rate(agzo_ctx* ctx, double* hz) {
    int dev = 0, khz = 0;
    HIPCHK(hipGetDevice(&dev));
    HIPCHK(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
    if (khz <= 0) return fail(ctx, AGZO_EHIP, "device reports no wall clock rate");
    *hz = 1e3 * khz;
    return 0;
}
}  // namespace

int agzo_profile_clock(agzo_ctx* ctx, int64_t* launches, double* mean_ghz) {
    if (!ctx) return AGZO_EINVAL;
    if (!launches || !mean_ghz) return fail(ctx, AGZO_EINVAL, "bad clock query");
    HIPCHK(hipStreamSynchronize(ctx->stream));
    double hz = 0.0;
    TRY(wall_rate(ctx, &hz));
    std::vector<unsigned long long> h(4 * ctx->clk_used);
    if (ctx->clk_used) HIPCHK(hipMemcpy(h.data(), ctx->clk, h.size() * 8, hipMemcpyDeviceToHost));
    double cycles = 0.0, ticks = 0.0;
    for (size_t i = 0; i < ctx->clk_used; ++i) {
        cycles += (double)(h[4 * i + 2] - h[4 * i]);
        ticks += (double)(h[4 * i + 3] - h[4 * i + 1]);
    }
    *launches = (int64_t)ctx->clk_used;
    *mean_ghz = (ticks > 0.0) ? cycles / ticks * hz * 1e-9 : 0.0;
    return AGZO_OK;
}

int agzo_probe_mfma(agzo_ctx* ctx, const void* operands, int32_t duty, int32_t iters, double* tflops, double* clock_ghz) {
    if (!ctx) return AGZO_EINVAL;
    if (!operands || !tflops || !clock_ghz) return fail(ctx, AGZO_EINVAL, "NULL argument");
    if (duty < 1 || duty > 9 || iters < 1 || iters > (1 << 20)) return fail(ctx, AGZO_EINVAL, "need 1 <= duty <= 9 and 1 <= iters <= 2^20");
    double hz = 0.0;
    TRY(wall_rate(ctx, &hz));
    int dev = 0, cus = 0;
    HIPCHK(hipGetDevice(&dev));
    HIPCHK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    unsigned long long* rec = ctx->clk + 4 * kClkSlots;
    HIPCHK(launch_probe_mfma(operands, duty, iters, rec, ctx->stream));
    HIPCHK(hipStreamSynchronize(ctx->stream));
    unsigned long long h[4];
    HIPCHK(hipMemcpy(h, rec, sizeof(h), hipMemcpyDeviceToHost));
    const double seconds = (double)(h[3] - h[1]) / hz;
    if (seconds <= 0.0) return fail(ctx, AGZO_EHIP, "probe returned no time");
    // 16 MFMAs of 32x32x16 per issued group, 4 waves per workgroup, one workgroup per CU
    // (duty 9: the flop count of 8 groups from 256 instructions of 16x16x32)
    const double flops = 2.0 * 32 * 32 * 16 * 16.0 * (duty == 9 ? 8 : duty) * (double)iters * 4.0 * cus;
    *tflops = flops / seconds * 1e-12;
    *clock_ghz = (double)(h[2] - h[0]) / seconds * 1e-9;
    return AGZO_OK;
}

int agzo_profile_read(agzo_ctx* ctx, int32_t kind, int64_t* launches, double* total_ms) {
    if (!ctx) return AGZO_EINVAL;
    if (kind < 0 || kind >= AGZO_PROF_KINDS || !launches || !total_ms) return fail(ctx, AGZO_EINVAL, "bad profile query");
    HIPCHK(hipStreamSynchronize(ctx->stream));
    ProfClass& pc = ctx->pc[kind];
    double sum = 0.0;
    for (size_t i = 0; i < pc.used; ++i) {
        float ms = 0.f;
        HIPCHK(hipEventElapsedTime(&ms, pc.start[i], pc.stop[i]));
        sum += ms;
    }
    *launches = (int64_t)pc.used;
    *total_ms = sum;
    return AGZO_OK;
}

int agzo_philox_words(agzo_ctx* ctx, uint32_t* dst, int64_t rows, int32_t cols, uint64_t seed, uint32_t tag) {
    if (!ctx) return AGZO_EINVAL;
    if (rows < 0 || cols < 0 || rows > 0xFFFFFFFFLL) return fail(ctx, AGZO_EINVAL, "bad shape");
    if (!dst && rows * cols > 0) return fail(ctx, AGZO_EINVAL, "dst is NULL");
    HIPCHK(launch_philox_words(dst, rows, cols, seed, tag, ctx->stream));
    return AGZO_OK;
}

int agzo_fill_normal(agzo_ctx* ctx, float* dst, int64_t rows, int32_t cols, uint64_t seed, uint32_t tag) {
    if (!ctx) return AGZO_EINVAL;
    if (rows < 0 || cols < 0 || rows > 0xFFFFFFFFLL) return fail(ctx, AGZO_EINVAL, "bad shape");
    if (!dst && rows * cols > 0) return fail(ctx, AGZO_EINVAL, "dst is NULL");
    ProfScope ps(ctx, AGZO_PROF_FILL);
    HIPCHK(launch_fill_normal(dst, rows, cols, seed, tag, ctx->stream));
    return AGZO_OK;
}

int agzo_layer_forward_sketch(agzo_ctx* ctx, const agzo_layer* L, const void* W, const void* X, void* Y, int32_t mode,
                              const float* Q, uint64_t seed, float* S, const agzo_loss_spec* loss, double* loss_dev) {
    const bool gemm = (W != nullptr);
    TRY(check_layer(ctx, L, gemm));
    if (!X) return fail(ctx, AGZO_EINVAL, "X is NULL");
    TRY(check_operands(ctx, L, W, X));
    if (!gemm && (Y || (loss && loss->kind != AGZO_LOSS_NONE))) return fail(ctx, AGZO_EINVAL, "Y or loss without W");
    if (mode != AGZO_SKETCH_NONE && mode != AGZO_SKETCH_RANGE && mode != AGZO_SKETCH_POWER && mode != AGZO_SKETCH_RANGE_FUSED)
        return fail(ctx, AGZO_EINVAL, "sketch mode %d", mode);
    const bool fused = (mode == AGZO_SKETCH_RANGE_FUSED);
    if (fused) {
        const bool ce = loss && loss->kind == AGZO_LOSS_CE;
        if (!gemm || L->dtype != AGZO_BF16 || ce || !gemm_bf16_fuses_sketch(L->n_tokens, L->d_out, L->r, L->tiling == AGZO_TILING_LARGE))
            return fail(ctx, AGZO_EINVAL, "the fused range sketch needs a bf16 forward in the 128 x 128 tiling (few 256 x 256 tiles, "
                                          "no cross-entropy, tiling AUTO), r <= 16 and at most 8192 tokens");
    }
    if (mode != AGZO_SKETCH_NONE && !S) return fail(ctx, AGZO_EINVAL, "S is NULL");
    if (gemm) {
        TRY(check_y(ctx, L, Y));
        TRY(check_loss(ctx, L, loss, loss_dev));
    }
    const Plan p = make_forward_plan(*L, loss, fused, W, X, Y);
    TRY(reserve(ctx, p.total));
    if (fused) {
        {
            ProfScope ps(ctx, AGZO_PROF_FILL);
            HIPCHK(launch_fill_normal_packT(wsh(ctx, p.off_TpackT), L->n_tokens, p.m_pad, L->r, p.rp, seed, AGZO_TAG_OMEGA, ctx->stream));
        }
        TRY(op_forward(ctx, *L, p, W, X, nullptr, 0.f, seed, Y, loss, loss_dev, false, 0, false, true));
        TRY(reduce_to_S(ctx, *L, p, S));
        return AGZO_OK;
    }
    if (gemm) TRY(op_forward(ctx, *L, p, W, X, nullptr, 0.f, seed, Y, loss, loss_dev));
    if (mode == AGZO_SKETCH_RANGE) {
        TRY(sketch_range(ctx, *L, p, X, seed, S));
        TRY(reduce_to_S(ctx, *L, p, S));
    }
    if (mode == AGZO_SKETCH_POWER) {
        if (!Q) {   // no Q given: the Gaussian feature-space start of the flagged variant, from the seed
            float* Q0 = wsf(ctx, p.off_Q);
            HIPCHK(launch_fill_normal(Q0, L->d_in, L->r, seed, AGZO_TAG_Q0, ctx->stream));
            Q = Q0;
        }
        if (reads_planes(*L)) HIPCHK(launch_pack_planes(Q, L->d_in, L->r, p.rp, wsh(ctx, p.off_pack), ctx->stream));
        TRY(sketch_power(ctx, *L, p, X, Q, S));
        TRY(reduce_to_S(ctx, *L, p, S));
    }
    return AGZO_OK;
}

int agzo_qr(agzo_ctx* ctx, const float* S, int64_t d_in, int32_t r, float* Q) {
    if (!ctx) return AGZO_EINVAL;
    if (!S || !Q) return fail(ctx, AGZO_EINVAL, "S or Q is NULL");
    if (r < 1 || r > kMaxRank || d_in < r) return fail(ctx, AGZO_EINVAL, "need 1 <= r <= min(64, d_in)");
    TRY(reserve(ctx, qr_workspace_bytes(d_in, r)));
    return op_qr(ctx, 0, S, d_in, r, round16(r), Q);
}

int agzo_basis(agzo_ctx* ctx, const agzo_layer* L, const void* X, int32_t K, uint64_t seed, const float* S0,
               int32_t flags, float* B) {
    TRY(check_layer(ctx, L, false));
    if (!X || !B) return fail(ctx, AGZO_EINVAL, "X or B is NULL");
    TRY(check_operands(ctx, L, nullptr, X));
    if (K < 0 || K > 64) return fail(ctx, AGZO_EINVAL, "K=%d outside 0..64", K);
    const Plan p = make_plan(*L, false);
    TRY(reserve(ctx, p.total));
    return op_basis(ctx, *L, p, X, K, seed, S0, flags, B);
}

int agzo_perturbed_forward(agzo_ctx* ctx, const agzo_layer* L, const void* W, const void* X, const float* B,
                           uint64_t seed, float eps_signed, void* Y, const agzo_loss_spec* loss, double* loss_dev) {
    TRY(check_layer(ctx, L, true));
    if (!W || !X || !B) return fail(ctx, AGZO_EINVAL, "W, X or B is NULL");
    TRY(check_operands(ctx, L, W, X));
    TRY(check_y(ctx, L, Y));
    TRY(check_loss(ctx, L, loss, loss_dev));
    const Plan p = make_forward_plan(*L, loss, false, W, X, Y);
    TRY(reserve(ctx, p.total));
    float* P = wsf(ctx, p.off_T);
    if (L->dtype != AGZO_BF16) {
        const F32SkinnyArgs a{static_cast<const float*>(X), L->ldx, L->n_tokens, L->d_in, B, L->r, P};
        HIPCHK(launch_xq_f32_many(&a, 1, ctx->stream));
        return op_forward(ctx, *L, p, W, X, P, eps_signed, seed, Y, loss, loss_dev);
    }
    const bool narrow = !reads_planes(*L), direct = !narrow && xq_ext_ok(L->n_tokens, L->d_in, L->r);
    XqArgs q{static_cast<const bf16_t*>(X), L->ldx, L->n_tokens, L->d_in, wsh(ctx, p.off_pack), L->r, p.rp, P, nullptr, p.m_pad, wsf(ctx, p.off_xqpart), nullptr, B};
    if (timed(ctx, AGZO_PROF_GEMM)) {      // the operands are prepared inside the forward's time
        if (!narrow && !direct) HIPCHK(launch_pack_planes(B, L->d_in, L->r, p.rp, wsh(ctx, p.off_pack), ctx->stream));
        {
            ProfScope ps(ctx, AGZO_PROF_XQ);
            HIPCHK(direct ? launch_xq_ext(q, nullptr, ctx->stream) : launch_xq_bf16_many(&q, 1, false, ctx->stream));
        }
        return op_forward(ctx, *L, p, W, X, P, eps_signed, seed, Y, loss, loss_dev);
    }
    // the projection writes the X side of the extension operands; where it multiplies the fp32 basis itself (xq_narrow(), xq_ext_ok()) it needs
    // no planes of B and shares a launch with the W side, else the planes and the W side are a launch ahead
    q.T = nullptr;
    q.Xext = wsh(ctx, p.off_ext);
    GemmExtArgs ext{ctx->ws + p.off_ext, L->n_tokens, L->d_out, nullptr, L->r, eps_signed, 0.f, false, seed, B, wsh(ctx, p.off_pack), L->d_in};
    if (narrow || direct) {
        ext.planes = nullptr;
        if (narrow) q.ext = &ext;
        ProfScope ps(ctx, AGZO_PROF_XQ);
        HIPCHK(narrow ? launch_xq_bf16_many(&q, 1, false, ctx->stream) : launch_xq_ext(q, &ext, ctx->stream));
    } else {
        HIPCHK(launch_gemm_ext_prep_many(&ext, 1, ctx->stream));
        ProfScope ps(ctx, AGZO_PROF_XQ);
        HIPCHK(launch_xq_bf16_many(&q, 1, false, ctx->stream));
    }
    return op_forward(ctx, *L, p, W, X, P, eps_signed, seed, Y, loss, loss_dev, false, 0, false, false, true);
}

int agzo_update(agzo_ctx* ctx, const agzo_layer* L, void* W, const float* B, uint64_t seed, float lr,
                const double* g_dev) {
    if (!ctx) return AGZO_EINVAL;
    if (!L) return fail(ctx, AGZO_EINVAL, "layer descriptor is NULL");
    if (L->tiling != AGZO_TILING_AUTO && L->tiling != AGZO_TILING_LARGE) return fail(ctx, AGZO_EINVAL, "tiling %d", L->tiling);
    TRY(check_update(ctx, W, B, L->dtype, L->d_out, L->d_in, L->ldw, L->r));
    TRY(reserve(ctx, update_workspace_bytes(L->dtype, L->d_out, L->d_in, L->r)));
    TRY(op_update(ctx, *L, 0, W, B, seed, lr, g_dev));
    return AGZO_OK;
}

int agzo_update_noalloc(agzo_ctx* ctx, const agzo_layer* L, void* W, const float* B, uint64_t seed, float lr,
                        const double* g_dev) {
    if (!ctx) return AGZO_EINVAL;
    if (!L) return fail(ctx, AGZO_EINVAL, "layer descriptor is NULL");
    if (L->tiling != AGZO_TILING_AUTO && L->tiling != AGZO_TILING_LARGE) return fail(ctx, AGZO_EINVAL, "tiling %d", L->tiling);
    TRY(check_update(ctx, W, B, L->dtype, L->d_out, L->d_in, L->ldw, L->r));
    const size_t need = update_workspace_bytes(L->dtype, L->d_out, L->d_in, L->r);
    if (need > kStaticScratchBytes)
        return fail(ctx, AGZO_EINVAL, "factor fragments of this update take %zu bytes, the static scratch holds %zu",
                    need, kStaticScratchBytes);
    int dev = -1;
    HIPCHK(hipGetDevice(&dev));
    if (dev != ctx->device || !ctx->static_scratch)
        return fail(ctx, AGZO_EINVAL, "current device %d is not the context's device %d", dev, ctx->device);
    // the preparation launch rewrites every fragment the sweep reads, so nothing left by an earlier call is seen
    HIPCHK(launch_update(W, L->dtype, L->ldw, L->d_out, L->d_in, B, L->r, seed, lr, g_dev, ctx->static_scratch, ctx->stream));
    return AGZO_OK;
}

int agzo_update_many(agzo_ctx* ctx, const agzo_update_item* items, int32_t n) {
    if (!ctx) return AGZO_EINVAL;
    if (n < 0 || (n > 0 && !items)) return fail(ctx, AGZO_EINVAL, "bad item list");
    size_t need = 0;
    for (int m = 0; m < n; ++m) {
        const agzo_update_item& u = items[m];
        if (u.reserved != 0) return fail(ctx, AGZO_EINVAL, "item %d: reserved field must be 0", m);
        TRY(check_update(ctx, u.W, u.B, u.dtype, u.d_out, u.d_in, u.ldw, u.r));
        need += update_workspace_bytes(u.dtype, u.d_out, u.d_in, u.r);
    }
    TRY(reserve(ctx, need));
    return update_many_at(ctx, items, n, 0);
}

int agzo_dense_perturb(agzo_ctx* ctx, void* theta, int32_t dtype, int64_t rows, int64_t cols, int64_t ld, uint64_t seed,
                       float scale, const double* g_dev) {
    if (!ctx) return AGZO_EINVAL;
    if (rows < 0 || cols < 0 || ld < cols) return fail(ctx, AGZO_EINVAL, "bad shape %lld x %lld, ld %lld", (long long)rows, (long long)cols, (long long)ld);
    if (dtype != AGZO_F32 && dtype != AGZO_BF16) return fail(ctx, AGZO_EINVAL, "dtype %d", dtype);
    if (rows > 0xFFFFFFFFLL || (cols + 3) / 4 > 0xFFFFFFFFLL) return fail(ctx, AGZO_EINVAL, "rows and cols/4 must fit 32-bit counters");
    if (!theta && rows * cols > 0) return fail(ctx, AGZO_EINVAL, "theta is NULL");
    ProfScope ps(ctx, AGZO_PROF_FILL);
    HIPCHK(launch_dense_axpy(theta, dtype, rows, cols, ld, seed, scale, g_dev, ctx->stream));
    return AGZO_OK;
}

int agzo_two_point(agzo_ctx* ctx, double* out4_dev, float eps, int32_t flags) {
    if (!ctx) return AGZO_EINVAL;
    if (!out4_dev) return fail(ctx, AGZO_EINVAL, "out4_dev is NULL");
    if (!(eps > 0.f)) return fail(ctx, AGZO_EINVAL, "eps must be positive");
    HIPCHK(launch_two_point(out4_dev, eps, (flags & AGZO_ONE_SIDED) ? 1 : 0, ctx->stream));
    return AGZO_OK;
}

int agzo_basis_many(agzo_ctx* ctx, const agzo_basis_item* items, int32_t n, int32_t K, int32_t flags) {
    if (!ctx) return AGZO_EINVAL;
    if (n < 0 || (n > 0 && !items)) return fail(ctx, AGZO_EINVAL, "bad item list");
    if (K < 0 || K > 64) return fail(ctx, AGZO_EINVAL, "K=%d outside 0..64", K);
    std::vector<LayerJob> jobs((size_t)n);
    size_t total = 0;
    for (int m = 0; m < n; ++m) {
        const agzo_basis_item& it = items[m];
        TRY(check_layer(ctx, &it.layer, false));
        if (!it.X || !it.B) return fail(ctx, AGZO_EINVAL, "item %d: X or B is NULL", m);
        TRY(check_operands(ctx, &it.layer, nullptr, it.X));
        LayerJob& j = jobs[(size_t)m];
        j.L = it.layer; j.X = it.X; j.seed = it.seed; j.S0 = it.S0; j.B = it.B;
        j.p = make_plan(j.L, false, false, false, total);
        total = j.p.total;
    }
    TRY(reserve(ctx, total));
    return basis_many_impl(ctx, jobs, K, flags);
}

namespace {
// The base forwards need nothing of the extraction nor it of them, and the extraction is a chain of some twenty launches that are bound by
// latency or by memory: for a set of layers they run beside it, those in 128 x 128 tiles on half of every compute unit.  The two streams
// wait for each other twice, some 20 us, and what counts is the layers whose forwards run there (bf16, squared error), not those of the
// call (one 4096 x 4096 layer on 1024 tokens among three small fp32 ones: 349 us a step, 389 with two streams).  Measured (us a step, one
// stream and two): seven layers 0.6B-sized on 512 tokens (16 GFLOP) 233
// and 233, on 1024 299 and 290, on 2048 428 and 416, 4B-sized on 128 383 and 360, on 512 617 and 570, on 3001 2075 and 1935; four
// of them on 512 272 and 265, on 4096 790 and 750; two on 4096 444 and 452; one 4096 x 4096 layer on 1024 tokens 232 and 249.
// The rule has no line for the rank or the tiles of the forwards.  At r > 16 the second form of X^T T needs more LDS than forwards in
// 128 x 128 tiles leave, and starts where those end; forwards in 256 x 256 tiles hold whole compute units, and the extraction fills the
// rounds that they do not: 4B-sized on 512 tokens 682 and 642 at r = 32, 899 and 887 at 64, on 4096 2786 and 2676, 3183 and 3005 (with
// their large tiles on the context's stream 2779 and 3177), 8B-sized on 16384, r = 16, 15173 and 14976
// Forwards in 128 x 128 tiles should not outlast the extraction: they would stay on half of every compute unit, and the perturbed ones
// that follow find no room beside them (8B-sized, r = 1, on 768 tokens 1122 and 1231, on 2304 2647 and 2774).  The extraction takes time
// for its launches (more with a factorisation than with a norm), the rank and the sweeps over X: with K = 3 and up to
// 200 + 60 [r > 1] + r GFLOP and 800 per value of X, two streams were never more than 1.2 % slower over the three sets' sizes, 256
// to 16384 tokens and r = 1 to 64, and no more than 0.7 % faster beyond; with K from 0 to 6 the line taken as the number of sweeps
// never more than 3 % slower (without it up to 13)
// Where 256 x 256 tiles in lists take every layer they get compute units of their own, as many as let both be done first
// (launch_gemm_bf16_beside()): the 4B-sized layers on 1500 tokens 1097 and 1005, 8B-sized on 1000 1284 and 1209
constexpr int kBesideLayers = 4;
constexpr double kBesideFlops = 20e9;
bool beside_fits(const std::vector<GemmBf16Args>& forwards, int K) {
    double half_cu = 0.0, values = 0.0, flops = 0.0;
    int r = 1;
    for (const GemmBf16Args& a : forwards) {
        const double f = 2.0 * (double)a.M * (double)a.N * (double)a.K;
        flops += f;
        if (gemm_bf16_small_tiles(a.M, a.N, a.large_tiles)) half_cu += f;
        values += (double)a.M * (double)a.K;
        r = std::max(r, a.r);
    }
    return (int)forwards.size() >= kBesideLayers && flops >= kBesideFlops &&
           half_cu <= (1e9 * (200 + (r > 1 ? 60 : 0) + r) + 800.0 * values) * ((2 * K + 2) / 8.0);
}
// What the extraction takes by itself: the latencies of its launches, and two sweeps over X a step at 5.7 TB/s (one for up to kProductsOfOneX layers
// that share it)
GemmBeside extraction_us(const std::vector<GemmBf16Args>& forwards, int K) {
    double bytes = 0.0;
    int r = 1;
    for (size_t i = 0; i < forwards.size(); ++i) {
        const GemmBf16Args& a = forwards[i];
        int before = 0;          // with the same activations
        for (size_t j = 0; j < i; ++j) {
            const GemmBf16Args& b = forwards[j];
            before += b.X == a.X && b.ldx == a.ldx && b.M == a.M && b.K == a.K && b.r <= 16 && a.r <= 16;
        }
        const bool loads = before % kProductsOfOneX == 0;
        bytes += (double)a.M * (double)a.K * ((loads ? 1.0 : 0.0) + (loads || xq_narrow(a.M, a.K, a.r) ? 1.0 : 0.0));
        r = std::max(r, a.r);
    }
    return GemmBeside{(r > 1 ? 37.0 : 28.0) * (K + 1), bytes * (2 * K + 2) / 5.7e6};
}
// Alg. 2 for n single-layer problems (agzo_step_many; agzo_step is the same with n = 1, so that their results agree bit for
// bit).  Squared-error layers run every stage together: the evaluations of part 1 (f0, or all three in the shared schedule) and
// of part 2 (f+ and f-) go to the launch functions as one list, and one launch finishes every loss and scalar.  Cross-entropy
// layers evaluate one by one (every evaluation is finished by launches of its own).
int step_many_body(agzo_ctx* ctx, const agzo_step_item* items, int n, int K, float eps, float lr, int flags) {
    const bool shared = (flags & AGZO_SHARED_FORWARD) != 0, one_sided = (flags & AGZO_ONE_SIDED) != 0;
    std::vector<LayerJob> jobs((size_t)n);
    size_t total = 0;
    for (int m = 0; m < n; ++m) {
        const agzo_step_item& it = items[m];
        TRY(check_layer(ctx, &it.layer, true));
        if (!it.W || !it.X || !it.out_dev) return fail(ctx, AGZO_EINVAL, "item %d: W, X or out_dev is NULL", m);
        if (it.loss.kind == AGZO_LOSS_NONE) return fail(ctx, AGZO_EINVAL, "item %d: a step needs a loss", m);
        TRY(check_loss(ctx, &it.layer, &it.loss, it.out_dev));
        TRY(check_operands(ctx, &it.layer, it.W, it.X));
        TRY(check_update(ctx, it.W, reinterpret_cast<const float*>(it.X) /* B is the call's own: any non-NULL */, it.layer.dtype, it.layer.d_out, it.layer.d_in, it.layer.ldw, it.layer.r));
        LayerJob& j = jobs[(size_t)m];
        j.L = it.layer; j.X = it.X; j.seed = it.seed; j.S0 = nullptr;
        j.p = make_plan(j.L, j.L.dtype == AGZO_F32 && it.loss.kind == AGZO_LOSS_CE, it.loss.kind == AGZO_LOSS_CE, shared, total);
        total = j.p.total;
    }
    size_t upd_bytes = 0;
    for (int m = 0; m < n; ++m)
        if (!items[m].B_out) upd_bytes += update_workspace_bytes(items[m].layer.dtype, items[m].layer.d_out, items[m].layer.d_in, items[m].layer.r);
    TRY(reserve(ctx, total + upd_bytes));
    for (int m = 0; m < n; ++m) jobs[(size_t)m].B = items[m].B_out ? items[m].B_out : wsf(ctx, jobs[(size_t)m].p.off_B);
    hipStream_t st = ctx->stream;
    Fork<HipApi> beside(st, ctx->side, ctx->fork, ctx->join);
    bool half_cu = false;          // forwards on the other stream hold half of every compute unit
    // the Gaussian factors with the coefficients of both perturbed evaluations (shared: what each of them adds), where the forwards read
    // them from operands that the projection has written (timed: each forward prepares its own, inside its time)
    std::vector<GemmExtArgs> sides((size_t)n);
    for (int m = 0; m < n; ++m) {
        const agzo_step_item& it = items[m];
        const LayerJob& j = jobs[(size_t)m];
        if (j.L.dtype != AGZO_BF16 || timed(ctx, AGZO_PROF_GEMM)) continue;
        GemmLossArgs la;
        la.kind = it.loss.kind;
        const GemmBf16Args f = forward_bf16_args(ctx, j.L, j.p, it.W, it.X, wsf(ctx, j.p.off_T), eps, it.seed, nullptr, la, shared);
        if (gemm_bf16_reads_ext(f))
            sides[(size_t)m] = GemmExtArgs{f.ext_ws, f.M, f.N, nullptr, f.r, eps, shared ? -2.f * eps : -eps, shared || !one_sided, it.seed};
    }

    // the base forward of a lone layer beside its extraction, in 256 x 256 tiles on compute units of its own where both are done sooner so.  (A
    // factorisation takes longer with the rank: one layer 2048 wide, r = 64, about 200 us more than at 16)
    int base_slots = 0;
    if (n == 1 && !shared && items[0].layer.dtype == AGZO_BF16 && ctx->prof == 0 && ctx->side) {
        GemmLossArgs la;
        la.kind = items[0].loss.kind; la.target_dtype = items[0].loss.target_dtype; la.target = items[0].loss.target; la.ldt = items[0].loss.ldt;
        const std::vector<GemmBf16Args> f(1, forward_bf16_args(ctx, jobs[0].L, jobs[0].p, items[0].W, items[0].X, nullptr, 0.f, 0, nullptr, la, false));
        GemmBeside extraction = extraction_us(f, K);
        extraction.latency_us += (K + 1) * std::max(0, f[0].r - 16);
        base_slots = gemm_bf16_slots_beside(f[0], extraction);
    }

    // the squared-error evaluations of phases [ph0, ph1): 0 = f0 (or, shared, all three from one pass), 1 = f+, 2 = f-; the
    // loss partials of phase ph go to slot ph of the layer's region
    auto forward_mse = [&](int ph0, int ph1) -> int {
        std::vector<GemmBf16Args> bf;
        std::vector<F32FwdArgs> f32;
        const bool perturbed = shared || ph0 > 0;
        for (int m = 0; m < n; ++m) {
            const agzo_step_item& it = items[m];
            if (it.loss.kind != AGZO_LOSS_MSE) continue;
            const LayerJob& j = jobs[(size_t)m];
            if (3 * (size_t)j.p.n_part > j.p.part_count) return fail(ctx, AGZO_EHIP, "internal: loss scratch of layer %d", m);
            GemmLossArgs la;
            la.kind = AGZO_LOSS_MSE; la.target_dtype = it.loss.target_dtype; la.target = it.loss.target; la.ldt = it.loss.ldt;
            const float* P = perturbed ? wsf(ctx, j.p.off_T) : nullptr;
            const bool ready = perturbed && sides[(size_t)m].ext_ws;
            for (int ph = ph0; ph < ph1; ++ph) {
                la.partials = reinterpret_cast<double*>(ctx->ws + j.p.off_part) + (size_t)ph * j.p.n_part;
                const float e = ph == 2 ? -eps : eps;
                if (j.L.dtype == AGZO_F32) {
                    f32.push_back(forward_f32_args(j.L, it.W, it.X, P, e, it.seed, la, shared));
                } else {
                    bf.push_back(forward_bf16_args(ctx, j.L, j.p, it.W, it.X, P, e, it.seed, nullptr, la, shared));
                    bf.back().ext_ready = ready;
                    bf.back().ext_side = ph == 2 ? 1 : 0;
                }
            }
        }
        for (size_t b = 0; b < f32.size(); b += kBatchMax)
            HIPCHK(launch_forward_f32_many(f32.data() + b, (int)std::min(f32.size() - b, (size_t)kBatchMax), st));
        if (bf.empty()) return 0;
        if (ph1 == 1 && !shared && ctx->prof == 0 && ctx->side && beside_fits(bf, K)) {
            const int count = (int)bf.size();
            half_cu = !gemm_bf16_listed(bf.data(), count);
            HIPCHK(beside.run([&](hipStream_t side) {
                return half_cu ? launch_gemm_bf16_many(bf.data(), count, true, side) : launch_gemm_bf16_beside(bf.data(), count, extraction_us(bf, K), side);
            }));
            return 0;
        }
        if (ph1 == 1 && base_slots > 0) {
            bf[0].slots = base_slots;
            HIPCHK(beside.run([&](hipStream_t side) { return launch_gemm_bf16(bf[0], side); }));
            return 0;
        }
        if (!timed(ctx, AGZO_PROF_GEMM)) {
            HIPCHK(launch_gemm_bf16_many(bf.data(), (int)bf.size(), false, st));
            return 0;
        }
        for (const GemmBf16Args& a : bf) {      // timed: a launch of its own for every forward (the results are the same)
            ProfScope ps(ctx, AGZO_PROF_GEMM);
            HIPCHK(launch_gemm_bf16(a, st));
        }
        return 0;
    };
    auto forward_ce = [&](int m, const float* P, float e, double* dst, bool sh, int slot) -> int {
        const agzo_step_item& it = items[m];
        if (it.loss.kind != AGZO_LOSS_CE) return 0;
        const LayerJob& j = jobs[(size_t)m];
        auto forward = [&](const SideForward* side) {
            return op_forward(ctx, j.L, j.p, it.W, it.X, P, e, it.seed, nullptr, &it.loss, dst, sh, slot, false, false, P && sides[(size_t)m].ext_ws, slot == 2 ? 1 : 0, side);
        };
        if (P || base_slots == 0) return forward(nullptr);
        int rc = 0;
        HIPCHK(beside.run([&](hipStream_t side) {
            const SideForward s{side, base_slots};
            rc = forward(&s);
            return hipSuccess;
        }));
        return rc;
    };
    // Alg. 2, part 1: the base forward of every layer, and every layer's basis from the same activations
    if (!shared) {
        TRY(forward_mse(0, 1));
        for (int m = 0; m < n; ++m) TRY(forward_ce(m, nullptr, 0.f, items[m].out_dev, false, 0));
    }
    TRY(basis_many_impl(ctx, jobs, K, flags & AGZO_INIT_FEATURE, half_cu));
    // parts 2-3: the perturbed evaluations
    TRY(project_many(ctx, jobs, sides, half_cu));
    if (shared) TRY(forward_mse(0, 1));
    else TRY(forward_mse(1, one_sided ? 2 : 3));
    for (int m = 0; m < n; ++m) {
        const float* P = wsf(ctx, jobs[(size_t)m].p.off_T);
        if (shared) {
            TRY(forward_ce(m, P, eps, items[m].out_dev, true, 0));
        } else {
            TRY(forward_ce(m, P, +eps, items[m].out_dev + 1, false, 1));
            if (!one_sided) TRY(forward_ce(m, P, -eps, items[m].out_dev + 2, false, 2));
        }
    }
    HIPCHK(beside.close());
    // the scalars, then every update in one batched call
    std::vector<agzo_update_item> upd;
    std::vector<FinishTwoPointArgs> fin;
    for (int m = 0; m < n; ++m) {
        const agzo_step_item& it = items[m];
        const LayerJob& j = jobs[(size_t)m];
        if (it.loss.kind == AGZO_LOSS_MSE)
            fin.push_back(FinishTwoPointArgs{reinterpret_cast<const double*>(ctx->ws + j.p.off_part), j.p.n_part,
                                             1.0 / ((double)j.L.n_tokens * (double)j.L.d_out), it.out_dev});
        else
            HIPCHK(launch_two_point(it.out_dev, eps, one_sided ? 1 : 0, st));
        if (!it.B_out) {
            agzo_update_item u;
            u.W = it.W; u.B = j.B; u.g_dev = it.out_dev + 3;
            u.d_out = j.L.d_out; u.d_in = j.L.d_in; u.ldw = j.L.ldw; u.r = j.L.r; u.dtype = j.L.dtype;
            u.seed = it.seed; u.lr = lr; u.reserved = 0;
            upd.push_back(u);
        }
    }
    for (size_t b = 0; b < fin.size(); b += kBatchMax)
        HIPCHK(launch_finish_two_point_many(fin.data() + b, (int)std::min(fin.size() - b, (size_t)kBatchMax), (shared || !one_sided) ? 3 : 2, eps,
                                            one_sided ? 1 : 0, st));
    if (upd.empty()) return AGZO_OK;
    // the update's factor fragments go behind the layers' carve-outs, which still hold the bases
    return update_many_at(ctx, upd.data(), (int)upd.size(), total);
}
int step_many_impl(agzo_ctx* ctx, const agzo_step_item* items, int n, int K, float eps, float lr, int flags) {
    try {
        return step_many_body(ctx, items, n, K, eps, lr, flags);
    } catch (const std::bad_alloc&) {      // (a C entry)
        return fail(ctx, AGZO_ENOMEM, "no host memory for the lists of %d layers", n);
    }
}
}  // namespace

int agzo_step_many(agzo_ctx* ctx, const agzo_step_item* items, int32_t n, int32_t K, float eps, float lr, int32_t flags) {
    if (!ctx) return AGZO_EINVAL;
    if (n < 0 || (n > 0 && !items)) return fail(ctx, AGZO_EINVAL, "bad item list");
    if (K < 0 || K > 64) return fail(ctx, AGZO_EINVAL, "K=%d outside 0..64", K);
    if (!(eps > 0.f)) return fail(ctx, AGZO_EINVAL, "eps must be positive");
    if (flags & AGZO_NAIVE_INPLACE) return fail(ctx, AGZO_EINVAL, "the in-place comparator runs layer by layer (agzo_step)");
    return step_many_impl(ctx, items, n, K, eps, lr, flags);
}

namespace {
int check_glue(agzo_ctx* ctx, int64_t n, int64_t d, std::initializer_list<const void*> ptrs, std::initializer_list<int64_t> lds) {
    if (!ctx) return AGZO_EINVAL;
    if (n < 0 || d < 0 || d % 8) return fail(ctx, AGZO_EINVAL, "rows of %lld values: need a non-negative multiple of 8", (long long)d);
    for (const void* p : ptrs)
        if ((!p && n * d > 0) || (reinterpret_cast<uintptr_t>(p) & 15)) return fail(ctx, AGZO_EINVAL, "NULL or misaligned tensor");
    for (int64_t ld : lds)
        if (ld < d || ld % 8) return fail(ctx, AGZO_EINVAL, "leading dimension %lld below the row length or not a multiple of 8", (long long)ld);
    if (n > 0x7FFFFFFFLL) return fail(ctx, AGZO_EINVAL, "too many rows");
    return 0;
}
}  // namespace

int agzo_glue_rmsnorm(agzo_ctx* ctx, const void* x, int64_t ldx, void* y, int64_t ldy, const float* gain, int64_t n, int64_t d,
                      float eps) {
    TRY(check_glue(ctx, n, d, {x, y}, {ldx, ldy}));
    HIPCHK(launch_glue_rmsnorm(static_cast<const bf16_t*>(x), ldx, static_cast<bf16_t*>(y), ldy, gain, n, d, eps, ctx->stream));
    return AGZO_OK;
}

int agzo_glue_swiglu(agzo_ctx* ctx, const void* a, int64_t lda, const void* u, int64_t ldu, void* m, int64_t ldm, int64_t n,
                     int64_t d) {
    TRY(check_glue(ctx, n, d, {a, u, m}, {lda, ldu, ldm}));
    HIPCHK(launch_glue_swiglu(static_cast<const bf16_t*>(a), lda, static_cast<const bf16_t*>(u), ldu, static_cast<bf16_t*>(m), ldm,
                              n, d, ctx->stream));
    return AGZO_OK;
}

int agzo_glue_attention(agzo_ctx* ctx, const void* q, int64_t ldq, const void* k, int64_t ldk, const void* v, int64_t ldv,
                        void* out, int64_t ldo, int32_t n_seq, int32_t seq_len, int32_t n_heads, int32_t n_kv_heads,
                        float rope_theta) {
    if (!ctx) return AGZO_EINVAL;
    if (n_seq < 0 || seq_len < 0 || n_heads < 1 || n_kv_heads < 1 || n_heads % n_kv_heads || n_heads > 65535 || n_seq > 65535)
        return fail(ctx, AGZO_EINVAL, "bad attention shape: %d sequences of %d tokens, %d heads on %d kv heads", n_seq, seq_len, n_heads,
                    n_kv_heads);
    if (!(rope_theta > 1.f)) return fail(ctx, AGZO_EINVAL, "rope_theta must exceed 1");
    const int64_t n = (int64_t)n_seq * seq_len, dq = (int64_t)n_heads * 128, dkv = (int64_t)n_kv_heads * 128;
    TRY(check_glue(ctx, n, dq, {q, out}, {ldq, ldo}));
    TRY(check_glue(ctx, n, dkv, {k, v}, {ldk, ldv}));
    if (n == 0) return AGZO_OK;
    // (a growth covers as much as the layer's inputs: its MLP's forwards ask for about that next, and a growth waits for the stream)
    const GlueCopies copies = glue_attention_copies(static_cast<const bf16_t*>(q), ldq, static_cast<const bf16_t*>(v), ldv, static_cast<const bf16_t*>(out), ldo, n_seq, seq_len, n_heads, n_kv_heads);
    TRY(reserve(ctx, glue_attention_workspace_bytes(n_seq, seq_len, n_heads, n_kv_heads, copies), (size_t)n * (n_heads + 2 * n_kv_heads) * 256));
    HIPCHK(launch_glue_attention(static_cast<const bf16_t*>(q), ldq, static_cast<const bf16_t*>(k), ldk, static_cast<const bf16_t*>(v), ldv,
                                 static_cast<bf16_t*>(out), ldo, n_seq, seq_len, n_heads, n_kv_heads, rope_theta, ctx->ws, ctx->stream));
    return AGZO_OK;
}

int agzo_glue_add(agzo_ctx* ctx, void* h, int64_t ldh, const void* delta, int64_t ldd, int64_t n, int64_t d) {
    TRY(check_glue(ctx, n, d, {h, delta}, {ldh, ldd}));
    HIPCHK(launch_glue_add(static_cast<bf16_t*>(h), ldh, static_cast<const bf16_t*>(delta), ldd, n, d, ctx->stream));
    return AGZO_OK;
}

// Alg. 2 for one layer.  B_out == NULL: the basis stays in the workspace and the update runs at the end;
// otherwise the basis goes to B_out and W is left as it was (the caller updates once g is final).
static int step_impl(agzo_ctx* ctx, const agzo_layer* L, void* W, const void* X, const agzo_loss_spec* loss, int32_t K,
                     float eps, float lr, uint64_t seed, int32_t flags, double* out_dev, float* B_out) {
    TRY(check_layer(ctx, L, true));
    if (!W || !X || !out_dev) return fail(ctx, AGZO_EINVAL, "W, X or out_dev is NULL");
    if (!loss || loss->kind == AGZO_LOSS_NONE) return fail(ctx, AGZO_EINVAL, "a step needs a loss");
    TRY(check_loss(ctx, L, loss, out_dev));
    if (K < 0 || K > 64) return fail(ctx, AGZO_EINVAL, "K=%d outside 0..64", K);
    if (!(eps > 0.f)) return fail(ctx, AGZO_EINVAL, "eps must be positive");
    TRY(check_operands(ctx, L, W, X));
    if (!(flags & AGZO_NAIVE_INPLACE)) {
        agzo_step_item it;
        it.layer = *L; it.W = W; it.X = X; it.loss = *loss; it.seed = seed; it.out_dev = out_dev; it.B_out = B_out;
        return step_many_impl(ctx, &it, 1, K, eps, lr, flags);
    }
    // the comparator: perturb in place, plain forward, undo
    const Plan p = make_plan(*L, L->dtype == AGZO_F32 && loss->kind == AGZO_LOSS_CE, loss->kind == AGZO_LOSS_CE);
    TRY(reserve(ctx, p.total));
    hipStream_t st = ctx->stream;
    float* B = B_out ? B_out : wsf(ctx, p.off_B);
    const bool one_sided = (flags & AGZO_ONE_SIDED) != 0;
    // squared error: the forwards leave their tile partials side by side and one launch reduces them and forms g;
    // cross-entropy finishes each loss on its own and only g is left to do
    const bool mse = loss->kind == AGZO_LOSS_MSE;
    auto finish = [&](int nphase) -> int {
        if (mse) {
            const FinishTwoPointArgs f{reinterpret_cast<const double*>(ctx->ws + p.off_part), p.n_part,
                                       1.0 / ((double)L->n_tokens * (double)L->d_out), out_dev};
            HIPCHK(launch_finish_two_point_many(&f, 1, nphase, eps, one_sided ? 1 : 0, st));
        } else {
            HIPCHK(launch_two_point(out_dev, eps, one_sided ? 1 : 0, st));
        }
        return 0;
    };
    TRY(op_forward(ctx, *L, p, W, X, nullptr, 0.f, seed, nullptr, loss, out_dev + 0, false, 0, mse));
    TRY(op_basis(ctx, *L, p, X, K, seed, nullptr, flags & AGZO_INIT_FEATURE, B));
    TRY(op_update(ctx, *L, p.off_upd, W, B, seed, -eps, nullptr));
    TRY(op_forward(ctx, *L, p, W, X, nullptr, 0.f, seed, nullptr, loss, out_dev + 1, false, 1, mse));
    if (!one_sided) {
        TRY(op_update(ctx, *L, p.off_upd, W, B, seed, 2.f * eps, nullptr));
        TRY(op_forward(ctx, *L, p, W, X, nullptr, 0.f, seed, nullptr, loss, out_dev + 2, false, 2, mse));
        TRY(op_update(ctx, *L, p.off_upd, W, B, seed, -eps, nullptr));
    } else if (B_out) {
        TRY(op_update(ctx, *L, p.off_upd, W, B, seed, eps, nullptr));
    } else {
        // Alg. 2 as printed: W still holds W + eps Z here, and the last line takes the perturbation out and applies
        // the update in one sweep, W <- W - (eps + lr g) Z
        TRY(finish(2));
        TRY(op_update(ctx, *L, p.off_upd, W, B, seed, lr, out_dev + 3, eps));
        return AGZO_OK;
    }
    TRY(finish(one_sided ? 2 : 3));
    if (!B_out) TRY(op_update(ctx, *L, p.off_upd, W, B, seed, lr, out_dev + 3));
    return AGZO_OK;
}

int agzo_step(agzo_ctx* ctx, const agzo_layer* L, void* W, const void* X, const agzo_loss_spec* loss, int32_t K,
              float eps, float lr, uint64_t seed, int32_t flags, double* out_dev) {
    return step_impl(ctx, L, W, X, loss, K, eps, lr, seed, flags, out_dev, nullptr);
}

int agzo_step_no_update(agzo_ctx* ctx, const agzo_layer* L, void* W, const void* X, const agzo_loss_spec* loss,
                        int32_t K, float eps, uint64_t seed, int32_t flags, double* out_dev, float* B_out) {
    if (ctx && !B_out) return fail(ctx, AGZO_EINVAL, "B_out is NULL");
    return step_impl(ctx, L, W, X, loss, K, eps, 0.f, seed, flags, out_dev, B_out);
}

}  // extern "C"
