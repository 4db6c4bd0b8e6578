// K1 in double-double (ABM_FAR_DD): the library's counterpart of the paper's
// long-double runs (Section "Memory saving improves computing time": the same
// computation in a wider type, at a higher cost).  Every quantity of the
// scheme is a double-double (dd.h, about 106 significant bits): the weights
// b_k, a_k, c_k, Gamma(alpha+1), Gamma(alpha+2), h^alpha, t_s = s h, the history
// f_k, both history sums, the state and the right-hand side (with the forcing
// cos / sin).
//   * k_weights_dd: the cancellation-free binomial series of the double weight
//     kernel, u = 1/k, in double-double;
//   * the solve is plain_block.h on the arithmetic Num<dd> below.
// Tables and outputs are (hi, lo) pairs of doubles.
#include "abm_dev.h"
#include "abm_kernels.h"
#include "plain_block.h"
#include "dd.h"

namespace abm {

namespace {

// ------------------------------------------------------------------ weights
// C(al, j) u^(j-1) summed over j >= 1 (al as a pair: al + 1 need not be a double)
__host__ __device__ dd series_b_dd(dd al, dd u)
{
    dd coef = al, up = dd_make(1.0), s = dd_make(0.0);
    for (int j = 1; j < 400; ++j) {
        const dd term = dd_mul(coef, up);
        s = dd_add(s, term);
        if (fabs(term.hi) <= 1e-34 * fabs(s.hi)) break;
        coef = dd_div(dd_mul(coef, dd_add_d(al, -(double)j)), dd_make(j + 1.0));   // C(al, j+1)
        up = dd_mul(up, u);
    }
    return s;
}

// C(be, 2j) u^(2j-2) summed over j >= 1
__host__ __device__ dd series_a_dd(dd be, dd u)
{
    dd c2 = dd_ldexp(dd_mul(be, dd_add_d(be, -1.0)), -1);   // C(be, 2)
    const dd u2 = dd_mul(u, u);
    dd up = dd_make(1.0), s = dd_make(0.0);
    for (int j = 1; j < 400; ++j) {
        const dd term = dd_mul(c2, up);
        s = dd_add(s, term);
        if (fabs(term.hi) <= 1e-34 * fabs(s.hi) || c2.hi == 0.0) break;
        // C(be, 2j+2) = C(be, 2j) (be-2j)(be-2j-1) / ((2j+1)(2j+2))
        c2 = dd_div(dd_mul(c2, dd_mul(dd_add_d(be, -2.0 * j), dd_add_d(be, -2.0 * j - 1.0))),
                    dd_make((2.0 * j + 1.0) * (2.0 * j + 2.0)));
        up = dd_mul(up, u2);
    }
    return s;
}

// -(C(al, j) - al C(al, j-1)) u^(j-2) summed over j >= 2
__host__ __device__ dd series_c_dd(dd al, dd u)
{
    dd cj1 = al;                                             // C(al, 1)
    dd cj = dd_ldexp(dd_mul(al, dd_add_d(al, -1.0)), -1);    // C(al, 2)
    dd up = dd_make(1.0), s = dd_make(0.0);
    for (int j = 2; j < 400; ++j) {
        const dd term = dd_neg(dd_mul(dd_sub(cj, dd_mul(al, cj1)), up));
        s = dd_add(s, term);
        if (fabs(term.hi) <= 1e-34 * fabs(s.hi)) break;
        cj1 = cj;
        cj = dd_div(dd_mul(cj, dd_add_d(al, -(double)j)), dd_make(j + 1.0));
        up = dd_mul(up, u);
    }
    return s;
}

// Gamma(alpha+1), Gamma(alpha+2)
__host__ __device__ inline void gammas_dd(double alpha, dd* g1, dd* g2)
{
    const dd z = dd_add_d(dd_make(alpha), 1.0);
    *g1 = dd_gamma(z);
    *g2 = dd_mul(z, *g1);                                    // Gamma(a+2) = (a+1) Gamma(a+1)
}

// b_k Gamma(alpha+1), a_k Gamma(alpha+2), c_k Gamma(alpha+2) (Section 2's
// weights before their Gamma factors) by the binomial series in u = 1/k
__host__ __device__ inline void weights_dd_at(double alpha, int64_t k, dd* bk, dd* ak, dd* ck)
{
    const dd al = dd_make(alpha);
    const dd be = dd_add_d(al, 1.0);
    if (k <= 1) {
        const dd t2m1 = dd_expm1_series(dd_mul_d(dd_ln2(), alpha));   // 2^a - 1
        if (k == 0) {
            *bk = dd_make(1.0);
            *ak = dd_ldexp(t2m1, 1);                                   // 2^(a+1) - 2
            *ck = al;
        } else {
            *bk = t2m1;
            // 3^(a+1) - 2^(a+2) + 1 = 2^a * series in u = 1/2 around m = 2
            *ak = dd_mul(dd_add_d(t2m1, 1.0), series_a_dd(be, dd_make(0.5)));
            *ck = dd_sub(al, dd_mul(dd_add_d(dd_neg(al), 1.0), t2m1));  // a - (1-a)(2^a - 1)
        }
    } else {
        const dd kd = dd_make((double)k);
        const dd m = dd_make((double)(k + 1));
        const dd u = dd_div(dd_make(1.0), kd);
        // k^(a-1) as k^a / k (a - 1 would round)
        const dd pk = dd_div(dd_pow(kd, alpha), kd);
        const dd pm = dd_div(dd_pow(m, alpha), m);
        *bk = dd_mul(pk, series_b_dd(al, u));
        *ak = dd_ldexp(dd_mul(pm, series_a_dd(be, dd_div(dd_make(1.0), m))), 1);
        *ck = dd_mul(pk, series_c_dd(al, u));
    }
}

__device__ __forceinline__ void put(double* t, int64_t k, dd v)
{
    t[2 * k] = v.hi;
    t[2 * k + 1] = v.lo;
}

// gam: Gamma(alpha+1), Gamma(alpha+2) as pairs (4 doubles)
__global__ void k_gammas_dd(double alpha, double* gam)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        dd g1, g2;
        gammas_dd(alpha, &g1, &g2);
        put(gam, 0, g1);
        put(gam, 1, g2);
    }
}

__global__ __launch_bounds__(256) void k_weights_dd(double alpha, int64_t n, const double* gam,
                                                    double* b, double* a, double* c)
{
    const dd g1 = dd{gam[0], gam[1]}, g2 = dd{gam[2], gam[3]};
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += stride) {
        dd bk, ak, ck;
        weights_dd_at(alpha, k, &bk, &ak, &ck);
        put(b, k, dd_div(bk, g1));
        put(a, k, dd_div(ak, g2));
        put(c, k, dd_div(ck, g2));
    }
}

// ------------------------------------------------------------------ f(t, y)
// the part of f(t, y) that depends on t only
template <int R>
__device__ __forceinline__ dd forcing_dd(const double* __restrict__ p, dd t)
{
    dd sn, cs;
    if constexpr (R == ABM_RHS_DUFFING) {
        dd_sincos(dd_mul_d(t, p[2]), &sn, &cs);
        return dd_mul_d(cs, p[1]);
    } else if constexpr (R == ABM_RHS_LCR) {
        dd_sincos(dd_mul_d(t, p[1]), &sn, &cs);
        return dd_mul_d(sn, p[4]);
    } else if constexpr (R == ABM_RHS_POLY) {
        return dd_add_d(dd_mul_d(t, p[1]), p[0]);
    } else {
        return dd_make(0.0);
    }
}

// f(t, y) with that part given
template <int R, int D>
__device__ __forceinline__ void rhs_dd(const double* __restrict__ p, dd frc, const dd* y, dd* f)
{
    if constexpr (R == ABM_RHS_LINEAR) {
        f[0] = dd_mul_d(y[0], -p[0]);
    } else if constexpr (R == ABM_RHS_DUFFING) {
        f[0] = y[1];
        const dd cube = dd_mul(dd_mul(y[0], y[0]), y[0]);
        f[1] = dd_add(dd_sub(dd_sub(dd_mul_d(y[1], -p[0]), y[0]), cube), frc);
    } else if constexpr (R == ABM_RHS_LORENZ) {
        f[0] = dd_mul_d(dd_sub(y[1], y[0]), p[0]);
        f[1] = dd_sub(dd_mul(y[0], dd_add_d(dd_neg(y[2]), p[1])), y[1]);
        f[2] = dd_sub(dd_mul(y[0], y[1]), dd_mul_d(y[2], p[2]));
    } else if constexpr (R == ABM_RHS_POLY) {
        f[0] = frc;
    } else if constexpr (R == ABM_RHS_LCR) {
        const dd x = y[0];
        dd g;
        if (dd_le(x, -1.0))
            g = dd_add_d(dd_add_d(dd_mul_d(x, p[3]), -p[2]), p[3]);
        else if (dd_ge(x, 1.0))
            g = dd_add_d(dd_add_d(dd_mul_d(x, p[3]), p[2]), -p[3]);
        else
            g = dd_mul_d(x, p[2]);
        f[0] = dd_sub(y[1], g);
        f[1] = dd_add(dd_sub(dd_mul_d(y[1], -p[0]), y[0]), frc);
    } else if constexpr (R == ABM_RHS_DIAG) {
        f[0] = dd_add_d(dd_mul_d(y[0], -p[0]), p[2]);
        f[1] = dd_add_d(dd_mul_d(y[1], -p[1]), p[3]);
    }
}

}  // namespace

template <>
struct Num<dd> {
    static constexpr int LR = 16;
    static constexpr bool kUnroll = false;
    static __device__ __forceinline__ dd zero() { return dd_make(0.0); }
    // The history sums (older chunks) and the corrector round no worse than
    // dd_fma.  The shorter form takes the at most 127 newest terms, whose sum
    // is kept apart from the rest, and the predictor's newest term, whose
    // rounding reaches the state only through f.
    static __device__ __forceinline__ dd mac(dd w, dd f, dd acc) { return dd_mac(w, f, acc); }
    static __device__ __forceinline__ dd mac_near(dd w, dd f, dd acc) { return dd_mac15(w, f, acc); }
    static __device__ __forceinline__ dd mac_state(dd w, dd f, dd acc) { return dd_mac18(w, f, acc); }
    static __device__ __forceinline__ dd newest_weight(dd w) { return w; }
    static __device__ __forceinline__ dd newest_predictor(dd w, dd f, dd acc) { return dd_mac15(w, f, acc); }
    static __device__ __forceinline__ dd newest(dd w, dd f, dd acc) { return dd_mac18(w, f, acc); }
    static __device__ __forceinline__ dd mul_add(dd a, dd b, dd c) { return dd_fma(a, b, c); }
    static __device__ __forceinline__ dd add(dd a, dd b) { return dd_add(a, b); }
    static __device__ __forceinline__ dd mul(dd a, dd b) { return dd_mul(a, b); }
    static __device__ __forceinline__ dd of(double x) { return dd_make(x); }
    static __device__ __forceinline__ dd recip(dd x) { return dd_div(dd_make(1.0), x); }
    static __device__ __forceinline__ dd power(double h, double al) { return dd_pow(dd_make(h), al); }
    static __device__ __forceinline__ dd time(int64_t s, double h) { return two_prod((double)s, h); }
    static __device__ __forceinline__ bool finite(dd x) { return dd_isfinite(x); }
    static __device__ __forceinline__ dd nan() { return dd{__builtin_nan(""), __builtin_nan("")}; }
    static __device__ __forceinline__ dd lane(dd v, int l) { return dd{Num<double>::lane(v.hi, l), Num<double>::lane(v.lo, l)}; }
    static __device__ __forceinline__ dd swap(dd v, int mask) { return dd{Num<double>::swap(v.hi, mask), Num<double>::swap(v.lo, mask)}; }
    static __device__ __forceinline__ void exchange(dd& a, dd& b, int mask)
    {
        exchange_halves(a.hi, b.hi, mask);
        exchange_halves(a.lo, b.lo, mask);
    }
    static __device__ __forceinline__ dd get(const dd* p) { return dd{*as_global(&p->hi), *as_global(&p->lo)}; }
    static __device__ __forceinline__ void put(dd* p, dd v)
    {
        *as_global(&p->hi) = v.hi;
        *as_global(&p->lo) = v.lo;
    }
    static __device__ __forceinline__ dd ld_agent(const dd* p) { return dd{ld_relaxed(&p->hi), ld_relaxed(&p->lo)}; }
    static __device__ __forceinline__ void st_agent(dd* p, dd v)
    {
        Num<double>::st_agent(&p->hi, v.hi);
        Num<double>::st_agent(&p->lo, v.lo);
    }
    template <int R>
    static __device__ __forceinline__ dd force(const double* p, int64_t s, double h)
    {
        return forcing_dd<R>(p, time(s, h));
    }
    template <int R, int D>
    static __device__ __forceinline__ void rhs(const double* p, const dd* y, dd frc, dd* f)
    {
        rhs_dd<R, D>(p, frc, y, f);
    }
    template <int R, int D>
    static __device__ __forceinline__ void rhs0(const double* p, const dd* y, dd* f)
    {
        rhs_dd<R, D>(p, forcing_dd<R>(p, dd_make(0.0)), y, f);
    }
};

size_t plain_dd_chain_lds(int d, bool per_comp, int64_t chunks, bool alone)
{
    return plainblk::chain_lds<dd>(d, per_comp, chunks, alone);
}

int plain_dd_worker_chunks(int d) { return plainblk::worker_chunks<dd>(d); }

hipError_t launch_weights_dd(double alpha, int64_t n, double* gam, double* b, double* a, double* c,
                             hipStream_t st)
{
    hipLaunchKernelGGL(k_gammas_dd, dim3(1), dim3(64), 0, st, alpha, gam);
    if (n <= 0) return hipGetLastError();
    int64_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_weights_dd, dim3((unsigned)blocks), dim3(256), 0, st, alpha, n, gam, b, a, c);
    return hipGetLastError();
}

hipError_t launch_plain_dd(const PlainArgs& A, int kind, hipStream_t st)
{
    return plainblk::launch_kind<dd>(A, kind, st);
}

}  // namespace abm
