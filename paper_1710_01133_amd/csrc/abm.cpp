// libabm runtime: contexts, plans, argument checking and the C ABI entry
// points declared in include/abm.h.  Every arithmetic step of the method runs
// in the kernels (K0 weights, K1 plain path, far-field and chain kernels of
// the blocked path); this file only validates, allocates and enqueues.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "abm.h"
#include "abm_kernels.h"
#include "abm_runtime.h"

namespace abm {

static thread_local std::string g_last_error;

abm_status fail(abm_status code, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return code;
}

abm_status hip_fail(hipError_t e, const char* what)
{
    return fail(e == hipErrorOutOfMemory ? ABM_ENOMEM : ABM_EDEVICE, "%s: %s", what,
                hipGetErrorString(e));
}

int rhs_dim(int rhs)
{
    switch (rhs) {
    case ABM_RHS_LINEAR: return 1;
    case ABM_RHS_DUFFING: return 2;
    case ABM_RHS_LORENZ: return 3;
    case ABM_RHS_POLY: return 1;
    case ABM_RHS_LCR: return 2;
    case ABM_RHS_DIAG: return 2;
    default: return -1;
    }
}

double order_of(const abm_problem& p, int comp)
{
    return p.alphas[0] > 0.0 ? p.alphas[comp] : p.alpha;
}

bool orders_differ(const abm_problem& p)
{
    for (int i = 1; i < p.d; ++i)
        if (order_of(p, i) != order_of(p, 0)) return true;
    return false;
}

int deriv_mask(const abm_problem& p)
{
    int m = 0;
    for (int i = 0; i < p.d; ++i)
        if (order_of(p, i) > 1.0) m |= 1 << i;
    return m;
}

bool same_orders(const abm_problem& a, const abm_problem& b)
{
    if (a.d != b.d) return false;
    for (int i = 0; i < a.d; ++i)
        if (order_of(a, i) != order_of(b, i)) return false;
    return true;
}

int64_t n_out(int64_t N, int64_t stride)
{
    if (stride == 0) return 1;
    return N / stride + 1 + (N % stride ? 1 : 0);
}

abm_status validate(const abm_problem& p, int idx)
{
    const int d = rhs_dim(p.rhs);
    if (d < 0) return fail(ABM_EINVAL, "problem %d: unknown rhs %d", idx, p.rhs);
    if (p.d != d) return fail(ABM_EINVAL, "problem %d: d=%d but rhs %d has dimension %d", idx, p.d, p.rhs, d);
    for (int i = 0; i < d; ++i) {
        const double al = order_of(p, i);
        if (!(al > 0.0 && al <= 2.0))
            return fail(ABM_EINVAL, "problem %d: order %g of component %d outside (0, 2]", idx, al, i);
        if (al > 1.0 && !std::isfinite(p.x1[i]))
            return fail(ABM_EINVAL, "problem %d: x1 not finite", idx);
    }
    if (!(p.h > 0.0) || !std::isfinite(p.h))
        return fail(ABM_EINVAL, "problem %d: h=%g must be positive and finite", idx, p.h);
    if (p.N < 1 || p.N > kMaxSteps)
        return fail(ABM_EINVAL, "problem %d: N=%lld outside [1, %lld]", idx, (long long)p.N,
                    (long long)kMaxSteps);
    if (p.out_stride < 0) return fail(ABM_EINVAL, "problem %d: out_stride < 0", idx);
    if (p.far_prec < ABM_FAR_FP64 || p.far_prec > ABM_FAR_I8)
        return fail(ABM_EINVAL, "problem %d: unknown far_prec %d", idx, p.far_prec);
    for (int i = 0; i < d; ++i)
        if (!std::isfinite(p.x0[i])) return fail(ABM_EINVAL, "problem %d: x0 not finite", idx);
    for (int i = 0; i < 8; ++i)
        if (!std::isfinite(p.p[i])) return fail(ABM_EINVAL, "problem %d: p not finite", idx);
    return ABM_OK;
}

// Shape fields a plan fixes; x0, p and h may change between solves.
static bool same_shape(const abm_problem& a, const abm_problem& b)
{
    return a.rhs == b.rhs && a.d == b.d && same_orders(a, b) && a.N == b.N &&
           a.far_prec == b.far_prec && a.out_stride == b.out_stride;
}

int env_int(const char* name, int dflt)
{
    const char* v = getenv(name);
    if (!v || !*v) return dflt;
    return atoi(v);
}

// Device bytes the plan being made on this thread may still allocate: no
// bound, unless the ABM_PLAN_MEM_MIB test hook sets one (allocations beyond it
// fail as the device's own would).
static thread_local int64_t t_alloc_left = INT64_MAX;

int64_t alloc_left() { return t_alloc_left; }
void set_alloc_left(int64_t bytes) { t_alloc_left = bytes; }

abm_status dev_alloc(void** p, size_t bytes, const char* what)
{
    *p = nullptr;
    if (bytes == 0) return ABM_OK;
    if (t_alloc_left != INT64_MAX && (int64_t)bytes > t_alloc_left) return hip_fail(hipErrorOutOfMemory, what);
    hipError_t e = hipMalloc(p, bytes);
    if (e != hipSuccess) {
        *p = nullptr;
        return hip_fail(e, what);
    }
    if (t_alloc_left != INT64_MAX) t_alloc_left -= (int64_t)bytes;
    return ABM_OK;
}

void dev_free(void* p)
{
    if (p) (void)hipFree(p);
}

static void free_tables(abm_plan_s* pl)
{
    for (auto& t : pl->tables) {
        dev_free(t.gam);
        dev_free(t.b);
        dev_free(t.a);
        dev_free(t.c);
        free_reduced(t);
    }
    pl->tables.clear();
}

}  // namespace abm

using namespace abm;

extern "C" {

const char* abm_strerror(abm_status s)
{
    switch (s) {
    case ABM_OK: return "ok";
    case ABM_EINVAL: return "invalid argument";
    case ABM_ENOMEM: return "out of memory";
    case ABM_EDEVICE: return "device failure";
    case ABM_EAGAIN: return "not finished";
    case ABM_ENOENT: return "unknown ticket";
    case ABM_ECANCELED: return "cancelled";
    default: return "unknown status";
    }
}

const char* abm_last_error(void) { return g_last_error.c_str(); }

abm_status abm_ctx_create(int device, void* hip_stream, size_t arena_bytes, abm_ctx** out)
{
    if (!out) return fail(ABM_EINVAL, "out is NULL");
    *out = nullptr;
    int n = 0;
    hipError_t e = hipGetDeviceCount(&n);
    if (e != hipSuccess) return hip_fail(e, "hipGetDeviceCount");
    if (device < 0 || device >= n) return fail(ABM_EINVAL, "device %d of %d", device, n);
    e = hipSetDevice(device);
    if (e != hipSuccess) return hip_fail(e, "hipSetDevice");
    abm_ctx* c = new abm_ctx();
    c->device = device;
    c->stream = (hipStream_t)hip_stream;
    c->arena_bytes = arena_bytes ? arena_bytes : ((size_t)1 << 30);
    hipDeviceProp_t prop;
    e = hipGetDeviceProperties(&prop, device);
    if (e != hipSuccess) {
        delete c;
        return hip_fail(e, "hipGetDeviceProperties");
    }
    c->n_cu = prop.multiProcessorCount;
    // the serving state exists from the start (its thread and device memory
    // only from the first submit), so concurrent first submits and polls
    // never race to create it
    abm_status s = serve_create(c);
    if (s != ABM_OK) {
        delete c;
        return s;
    }
    *out = c;
    return ABM_OK;
}

void abm_ctx_destroy(abm_ctx* ctx)
{
    if (!ctx) return;
    serve_shutdown(ctx);
    delete ctx;
}

abm_status abm_plan(abm_ctx* ctx, const abm_problem* probs, int32_t B, abm_plan_t** out)
{
    return abm_plan_tuned(ctx, probs, B, nullptr, out);
}

abm_status abm_plan_tuned(abm_ctx* ctx, const abm_problem* probs, int32_t B,
                          const abm_tuning* tune, abm_plan_t** out)
{
    if (!ctx || !probs || !out) return fail(ABM_EINVAL, "NULL argument");
    *out = nullptr;
    if (B < 1) return fail(ABM_EINVAL, "B=%d must be >= 1", B);
    for (int i = 0; i < B; ++i) {
        abm_status s = validate(probs[i], i);
        if (s != ABM_OK) return s;
    }
    hipError_t e = hipSetDevice(ctx->device);
    if (e != hipSuccess) return hip_fail(e, "hipSetDevice");
    bool dd = false;
    for (int i = 0; i < B; ++i) dd |= probs[i].far_prec == ABM_FAR_DD;
    if (dd && B != 1)
        return fail(ABM_EINVAL, "double-double (ABM_FAR_DD) runs one trajectory per plan, on abm_solve");
    abm_plan_s* pl = new abm_plan_s();
    pl->ctx = ctx;
    pl->B = B;
    pl->dd = dd;
    pl->shape.assign(probs, probs + B);
    if (tune) pl->tune = *tune;
    abm_status st = ABM_OK;
    const int mem_mib = env_int("ABM_PLAN_MEM_MIB", 0);
    set_alloc_left(mem_mib > 0 ? (int64_t)mem_mib << 20 : INT64_MAX);

    // one weight table per distinct order, long enough for its longest user
    pl->table_of.assign((size_t)B * 4, 0);
    for (int i = 0; i < B; ++i) {
        for (int c = 0; c < probs[i].d; ++c) {
            const double al = order_of(probs[i], c);
            int found = -1;
            for (size_t j = 0; j < pl->tables.size(); ++j)
                if (pl->tables[j].alpha == al) found = (int)j;
            if (found < 0) {
                WeightTable t{};
                t.alpha = al;
                pl->tables.push_back(t);
                found = (int)pl->tables.size() - 1;
            }
            pl->tables[found].n = std::max<int64_t>(pl->tables[found].n, probs[i].N);
            pl->table_of[(size_t)i * 4 + c] = found;
        }
        for (int c = probs[i].d; c < 4; ++c) pl->table_of[(size_t)i * 4 + c] = pl->table_of[(size_t)i * 4];
    }
    for (auto& t : pl->tables) {
        // padded so that block kernels may read a full tile past N; a
        // double-double table holds (hi, lo) pairs
        const int64_t n = t.n + kWeightPad;
        const size_t w = dd ? 2 : 1;
        if ((st = dev_alloc((void**)&t.gam, 2 * w * sizeof(double), "weights")) ||
            (st = dev_alloc((void**)&t.b, w * n * sizeof(double), "weights")) ||
            (st = dev_alloc((void**)&t.a, w * n * sizeof(double), "weights")) ||
            (st = dev_alloc((void**)&t.c, w * n * sizeof(double), "weights")))
            break;
        e = dd ? launch_weights_dd(t.alpha, n, t.gam, t.b, t.a, t.c, ctx->stream)
               : launch_weights(t.alpha, n, t.gam, t.b, t.a, t.c, ctx->stream);
        if (e != hipSuccess) {
            st = hip_fail(e, "weight kernel");
            break;
        }
    }
    if (st == ABM_OK) st = dev_alloc((void**)&pl->status, sizeof(uint32_t), "status");
    if (st == ABM_OK) {
        e = launch_fill_u32(pl->status, 0, 1, ctx->stream);
        if (e != hipSuccess) st = hip_fail(e, "fill");
    }
    if (st == ABM_OK && dd) {
        // double-double: the plain path only, and it must fit
        st = plain_setup(pl);
    } else if (st == ABM_OK && B == 1) {
        // the plain path is optional: a history too long for it leaves plain_ok false
        const abm_status ps = plain_setup(pl);
        if (ps == ABM_ENOMEM || ps == ABM_EDEVICE) st = ps;
        if (ps != ABM_OK) pl->plain_error = abm_last_error();
    }
    if (st == ABM_OK && !dd) st = batch_setup(pl);
    set_alloc_left(INT64_MAX);
    if (st != ABM_OK) {
        abm_plan_destroy(pl);
        return st;
    }
    *out = pl;
    return ABM_OK;
}

void abm_plan_destroy(abm_plan_t* pl)
{
    if (!pl) return;
    (void)hipSetDevice(pl->ctx->device);
    (void)hipStreamSynchronize(pl->ctx->stream);
    free_tables(pl);
    dev_free(pl->part);
    dev_free(pl->flags);
    dev_free(pl->status);
    batch_teardown(pl);
    delete pl;
}

abm_status abm_plan_check(abm_plan_t* pl)
{
    if (!pl) return fail(ABM_EINVAL, "plan is NULL");
    hipError_t e = hipStreamSynchronize(pl->ctx->stream);
    if (e != hipSuccess) return hip_fail(e, "hipStreamSynchronize");
    uint32_t bits = 0;
    e = hipMemcpy(&bits, pl->status, sizeof bits, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(e, "status read");
    if (bits) {
        (void)launch_fill_u32(pl->status, 0, 1, pl->ctx->stream);
        (void)hipStreamSynchronize(pl->ctx->stream);
        return fail(ABM_EDEVICE, "device status 0x%x (%s%s)", bits,
                    (bits & 1u) ? "wait timed out " : "", (bits & 2u) ? "non-finite state" : "");
    }
    return ABM_OK;
}

abm_status abm_plan_weights(abm_plan_t* pl, int32_t idx, int64_t n, double* b, double* a,
                            double* c)
{
    if (!pl) return fail(ABM_EINVAL, "plan is NULL");
    if (idx < 0 || idx >= pl->B) return fail(ABM_EINVAL, "idx %d outside [0, %d)", idx, pl->B);
    const WeightTable& t = pl->tables[pl->table_of[(size_t)idx * 4]];
    if (n < 0 || n > t.n + kWeightPad)
        return fail(ABM_EINVAL, "n=%lld outside [0, %lld]", (long long)n, (long long)(t.n + kWeightPad));
    const size_t bytes = (pl->dd ? 2 : 1) * n * sizeof(double);
    hipError_t e = hipSetDevice(pl->ctx->device);
    if (e == hipSuccess) e = hipStreamSynchronize(pl->ctx->stream);
    if (e == hipSuccess && b) e = hipMemcpy(b, t.b, bytes, hipMemcpyDeviceToHost);
    if (e == hipSuccess && a) e = hipMemcpy(a, t.a, bytes, hipMemcpyDeviceToHost);
    if (e == hipSuccess && c) e = hipMemcpy(c, t.c, bytes, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(e, "weight copy");
    return ABM_OK;
}

abm_status abm_solve(abm_plan_t* pl, const abm_problem* prob, double* y_out)
{
    if (!pl || !prob || !y_out) return fail(ABM_EINVAL, "NULL argument");
    if (pl->B != 1) return fail(ABM_EINVAL, "abm_solve needs a plan made for one problem (B=%d)", pl->B);
    if (!pl->plain_ok) return fail(ABM_EINVAL, "plain path unavailable: %s", pl->plain_error.c_str());
    abm_status s = validate(*prob, 0);
    if (s != ABM_OK) return s;
    if (!same_shape(*prob, pl->shape[0]))
        return fail(ABM_EINVAL, "problem does not match the plan (rhs, d, orders, N, far_prec, out_stride)");
    hipError_t e = hipSetDevice(pl->ctx->device);
    if (e != hipSuccess) return hip_fail(e, "hipSetDevice");
    e = plain_run(pl, *prob, y_out, false);
    if (e != hipSuccess) return hip_fail(e, "plain kernel launch");
    return ABM_OK;
}

}  // extern "C"

namespace abm {

// Up to kAloneBlocks blocks workgroup 0 runs alone: the waves beside its
// sequencer then keep up (2048 steps, us per step alone / with 2 workgroups:
// linear 0.068 / 0.074, oscillator 0.119 / 0.117; 4096 steps: 0.091 / 0.067
// and 0.150 / 0.107).  Beyond, a worker per kWorkerChunks chunks: fewer fall
// behind the sequencer at the end of the run (200000-step oscillator, 46
// chunks each: 0.111 against 0.100 us per step), more only add traffic on the
// flags (linear, 65536 steps: 0.056 at 16 chunks each, 0.063 at 8).
// Double-double: the waves beside its sequencer fall behind earlier (us per
// step alone / with 3 workgroups, 1024 steps: linear 0.456 / 0.464, oscillator
// 1.056 / 1.058; 2048 steps: 0.595 / 0.445 and 1.249 / 1.037).
constexpr int kAloneBlocks = 32, kAloneBlocksDd = 16;
constexpr int kWorkerChunks = 16;

// what W workers and nred reducers keep
static void size_workers(const abm_problem& p, PlainShape* sh)
{
    const bool dd = p.far_prec == ABM_FAR_DD;
    const size_t chunk = (size_t)p.d * kPlainBlock * (dd ? 2 : 1), slot = 2 * chunk;
    const int64_t chunks = (p.N + kPlainBlock - 1) / kPlainBlock;
    const int64_t each = (chunks + sh->W - 1) / sh->W;
    sh->nloc = (int)std::min<int64_t>(each, dd ? plain_dd_worker_chunks(p.d) : plain_worker_chunks(p.d));
    sh->nspill = (int)(each - sh->nloc);
    sh->work_doubles = kPlainRing * chunk + kPlainSlots * (size_t)(sh->nred + sh->W) * slot +
                       (size_t)sh->W * sh->nspill * chunk;
    sh->flags = kPlainFlagPad + sh->W + sh->nred;
}

abm_status plain_shape(const abm_problem& p, int n_cu, PlainShape* out)
{
    const int d = p.d;
    const bool dd = p.far_prec == ABM_FAR_DD;
    const int words = dd ? 2 : 1;
    const int gcap = std::min(n_cu, 256);      // one workgroup per CU is always resident
    // The longest history accepted, as many 256-row pieces as the LDS of gcap
    // workgroups could hold less a fixed part: 2.55e6 steps of two components
    // on 256 CUs, 1.24e6 in double-double.  Workers keep fewer (119 chunks of
    // 64 rows, 39 in double-double: 1.8e6 and 6e5 steps) and spill the rest to
    // device memory.
    const size_t fixed = dd ? (size_t)1216 * d : (size_t)512 * d;
    const int64_t rows_max = (int64_t)gcap * 256 * ((kPlainLds - fixed) / ((size_t)2048 * d * words));
    if ((p.N + 255) / 256 * 256 > rows_max)
        return fail(ABM_EINVAL, "N=%lld too long for the %splain path (at most %lld steps of %d components on %d CUs)",
                    (long long)p.N, dd ? "double-double " : "", (long long)rows_max, d, gcap);
    const bool pc = orders_differ(p);
    const int64_t chunks = (p.N + kPlainBlock - 1) / kPlainBlock;
    const int forced = env_int("ABM_PLAIN_G", 0);
    const bool fits = (dd ? plain_dd_chain_lds(d, pc, chunks, true) : plain_chain_lds(d, pc, chunks, true)) <= kPlainLds;
    PlainShape sh{};
    if (fits && (forced == 1 || (forced <= 0 && chunks <= (dd ? kAloneBlocksDd : kAloneBlocks)))) {
        *out = sh;
        return ABM_OK;
    }
    int others = forced > 0 ? std::max(forced, 2) - 1 : 0;      // workers and reducers
    if (others == 0) {
        const int W = (int)std::min<int64_t>((chunks + kWorkerChunks - 1) / kWorkerChunks, gcap);
        others = W <= kPlainFan ? W : W + (W + kPlainFan - 1) / kPlainFan;
    }
    others = std::max(1, std::min(others, gcap - 1));
    for (;; ++others) {
        // every reducer with workers of its own (18 others are 16 workers and none)
        sh.W = others <= kPlainFan ? others : others - (others + kPlainFan) / (kPlainFan + 1);
        sh.nred = sh.W <= kPlainFan ? 0 : (sh.W + kPlainFan - 1) / kPlainFan;
        size_workers(p, &sh);
        // a forced count is raised until what its workers spill fits the
        // slots of abm_solve_noalloc, which takes the shape as it is
        if (forced <= 0 || sh.work_doubles * sizeof(double) <= kPlainSlotBytes || others >= gcap - 1) break;
    }
    *out = sh;
    return ABM_OK;
}

PlainShape plain_shape_small(const abm_problem& p, const PlainShape& full)
{
    PlainShape sh = full;
    sh.W = std::min(full.W, kPlainFan);
    sh.nred = 0;
    size_workers(p, &sh);
    return sh;
}

PlainArgs plain_args(const abm_problem& prob, const PlainTables& T, const PlainShape& sh,
                     double* work, uint32_t* flags, uint32_t* status, double* y_out)
{
    PlainArgs A{};
    for (int i = 0; i < 4; ++i) {
        A.b[i] = T.b[i];
        A.a[i] = T.a[i];
        A.c[i] = T.c[i];
        A.gam[i] = T.gam[i];
        A.alpha[i] = T.alpha[i];
        A.x0[i] = prob.x0[i];
        A.x1[i] = prob.x1[i];
    }
    A.h = prob.h;
    for (int i = 0; i < 8; ++i) A.p[i] = prob.p[i];
    A.N = prob.N;
    A.W = sh.W;
    A.nred = sh.nred;
    A.nloc = sh.nloc;
    A.nspill = sh.nspill;
    if (sh.W > 0) {
        const size_t chunk = (size_t)prob.d * kPlainBlock * (prob.far_prec == ABM_FAR_DD ? 2 : 1);
        const size_t slot = 2 * chunk;
        A.ring = work;
        A.rpart = A.ring + kPlainRing * chunk;
        A.part = A.rpart + kPlainSlots * (size_t)sh.nred * slot;
        A.spill = A.part + kPlainSlots * (size_t)sh.W * slot;
    }
    A.flags = flags;
    A.y_out = y_out;
    A.out_stride = prob.out_stride;
    A.status = status;
    // test hooks for the device-side waits' failure path: a smaller bound
    // and an offset that no flag reaches (every wait then gives up)
    const int spin = env_int("ABM_SPIN_LIMIT", 0);
    A.spin_limit = spin > 0 ? (uint32_t)spin : kSpinLimit;
    A.wait_bias = (uint32_t)std::max(0, env_int("ABM_WAIT_BIAS", 0));
    return A;
}

hipError_t plain_enqueue(const PlainArgs& A, const PlainShape& sh, int kind, bool dd, hipStream_t st)
{
    if (sh.W > 0) {
        hipError_t e = launch_fill_u32(A.flags, 0, sh.flags, st);
        if (e != hipSuccess) return e;
    }
    return dd ? launch_plain_dd(A, kind, st) : launch_plain(A, kind, st);
}

// flags of a plan: the run's, the status word of a run that may be repeated,
// the repeated run's
static size_t flag_words(const abm_plan_s* pl) { return pl->plain.flags + 1 + pl->again.flags; }

hipError_t plain_run(abm_plan_s* pl, const abm_problem& prob, double* y_out, bool retry)
{
    PlainTables T{};
    for (int i = 0; i < 4; ++i) {
        const WeightTable& t = pl->tables[pl->table_of[i]];
        T.b[i] = t.b;
        T.a[i] = t.a;
        T.c[i] = t.c;
        T.gam[i] = t.gam;
        T.alpha[i] = t.alpha;
    }
    const hipStream_t st = pl->ctx->stream;
    const int kind = chain_kind(prob.rhs, orders_differ(prob));
    if (!retry || pl->plain.W == 0) {
        const PlainArgs A = plain_args(prob, T, pl->plain, pl->part, pl->flags, pl->status, y_out);
        return plain_enqueue(A, pl->plain, kind, pl->dd, st);
    }
    // The workgroups of the first run wait for each other and so need the chip
    // to themselves; where another process holds part of it past the bound on
    // the waits, they give up.  The second launch then takes the trajectory
    // again with at most kPlainFan workers, which up to 15 such processes can
    // hold side by side, and waits longer (oscillator, 200000 steps 50 ms for
    // 20, 10^6 steps 1.2 s for 0.14).  Otherwise it returns at once.
    uint32_t* const first = pl->flags + pl->plain.flags;
    hipError_t e = launch_fill_u32(pl->flags, 0, flag_words(pl), st);
    if (e != hipSuccess) return e;
    PlainArgs A = plain_args(prob, T, pl->plain, pl->part, pl->flags, first, y_out);
    if ((e = launch_plain(A, kind, st)) != hipSuccess) return e;
    A = plain_args(prob, T, pl->again, pl->part, first + 1, pl->status, y_out);
    A.gate = first;
    A.spin_limit = 8 * kSpinLimit;
    A.wait_bias = 0;
    return launch_plain(A, kind, st);
}

abm_status plain_setup(abm_plan_s* pl)
{
    abm_status st = plain_shape(pl->shape[0], pl->ctx->n_cu, &pl->plain);
    if (st != ABM_OK) return st;
    const PlainShape& sh = pl->plain;
    if (sh.W > 0) {
        // (the second run reuses the first one's workspace)
        size_t work = sh.work_doubles;
        if (pl->shape[0].far_prec == ABM_FAR_FP64) {
            pl->again = plain_shape_small(pl->shape[0], sh);
            work = std::max(work, pl->again.work_doubles);
        }
        st = dev_alloc((void**)&pl->part, work * sizeof(double), "plain workspace");
        if (st == ABM_OK) st = dev_alloc((void**)&pl->flags, flag_words(pl) * sizeof(uint32_t), "plain flags");
    }
    pl->plain_ok = st == ABM_OK;
    return st;
}

}  // namespace abm
