// Host build of the multiply-adds of csrc/dd.h: sums of n products of (hi, lo)
// pairs, the first `cut` terms by form `far`, the rest by form `near` into a
// second accumulator, the two added at the end.  Forms: 0 dd_fma, 1 dd_mac,
// 2 dd_mac18, 3 dd_mac15.
#include "dd.h"

using abm::dd;

static dd step(int form, dd w, dd f, dd acc)
{
    switch (form) {
    case 0: return abm::dd_fma(w, f, acc);
    case 1: return abm::dd_mac(w, f, acc);
    case 2: return abm::dd_mac18(w, f, acc);
    default: return abm::dd_mac15(w, f, acc);
    }
}

extern "C" void t_sum(int far, int near, int n, int cut, const double* w, const double* f, double* o)
{
    dd a{0.0, 0.0}, b{0.0, 0.0};
    for (int k = 0; k < cut; ++k) a = step(far, dd{w[2 * k], w[2 * k + 1]}, dd{f[2 * k], f[2 * k + 1]}, a);
    for (int k = cut; k < n; ++k) b = step(near, dd{w[2 * k], w[2 * k + 1]}, dd{f[2 * k], f[2 * k + 1]}, b);
    const dd r = cut < n ? abm::dd_add(a, b) : a;
    o[0] = r.hi;
    o[1] = r.lo;
}
