"""Rounding of the double-double path's multiply-adds (csrc/dd.h, built for the
host) in history sums: b_k-like weights, newest last, against histories of one
sign, oscillating and random.

The bar is dd_fma, a normalised product and an accurate sum: the forms that
take the history's sums (dd_mac) and the corrector's update (dd_mac18) leave
one rounding of the low part's size where it has two, so their rms error must
not be larger; nor must that of a sum whose 96 newest terms go through the
short form (dd_mac15) into an accumulator of their own."""
import ctypes
import os
import shutil
import subprocess

import mpmath as mp
import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1710_01133_amd", "csrc")
FMA, MAC, MAC18, MAC15 = range(4)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("ddmac") / "libddmac.so")
    subprocess.run([hipcc, "-x", "hip", "--offload-arch=gfx950", "-O2", "-fPIC", "-shared",
                    "-std=c++17", "-ffp-contract=off", "-I", CSRC,
                    os.path.join(HERE, "dd_mac_shim.hip"), "-o", out],
                   check=True, capture_output=True)
    return ctypes.CDLL(out)


def _pairs(hi, rng):
    """Pairs with populated low parts below half a unit of the heads."""
    lo = hi * rng.uniform(-0.49, 0.49, hi.shape) * 2.0 ** -53
    return np.ascontiguousarray(np.stack([hi, lo], axis=-1))


def _sums(lib, kind, forms, n=512, trials=400):
    """rms error of each (far, near, cut) form in units of 2^-106 of the scale."""
    rng = np.random.default_rng(["one sign", "oscillating", "random"].index(kind) + 11)
    dp = ctypes.POINTER(ctypes.c_double)
    err = np.zeros((len(forms), trials))
    k = np.arange(n)
    for t in range(trials):
        al, om, ph = rng.uniform(0.8, 0.94), rng.uniform(0.002, 0.022), rng.uniform(0, 2 * np.pi)
        w = _pairs((n - k + 1.0) ** al - (n - k) ** al, rng)
        f = {"one sign": 1 + 0.3 * np.sin(om * k + ph), "oscillating": np.sin(om * k + ph),
             "random": rng.uniform(-1, 1, n)}[kind]
        f = _pairs(f, rng)
        ref = mp.fdot((mp.mpf(a[0]) + mp.mpf(a[1]), mp.mpf(b[0]) + mp.mpf(b[1])) for a, b in zip(w.tolist(), f.tolist()))
        scale = abs(ref) if kind == "one sign" else mp.sqrt(n)
        for i, (far, near, cut) in enumerate(forms):
            o = (ctypes.c_double * 2)()
            lib.t_sum(far, near, n, cut, w.ctypes.data_as(dp), f.ctypes.data_as(dp), o)
            err[i, t] = float((mp.mpf(o[0]) + mp.mpf(o[1]) - ref) / scale) * 2.0 ** 106
    return np.sqrt((err ** 2).mean(axis=1))


@pytest.mark.parametrize("kind", ["one sign", "oscillating", "random"])
def test_history_sums_round_no_worse_than_the_accurate_form(lib, kind):
    mp.mp.dps = 50
    n = 512
    forms = [(FMA, FMA, n), (MAC, MAC, n), (MAC18, MAC18, n), (MAC, MAC15, n - 96)]
    rms = _sums(lib, kind, forms, n)
    print(kind, dict(zip(("fma", "mac", "mac18", "mac and newest by mac15"), rms.round(3).tolist())))
    assert (rms[1:] <= rms[0]).all()


def test_a_sum_is_exact_where_doubles_hold_it(lib):
    """Small integers: every form gives the exact sum."""
    rng = np.random.default_rng(2)
    w = np.zeros((64, 2))
    f = np.zeros((64, 2))
    w[:, 0], f[:, 0] = rng.integers(-1000, 1000, 64), rng.integers(-1000, 1000, 64)
    dp = ctypes.POINTER(ctypes.c_double)
    for form in (FMA, MAC, MAC18, MAC15):
        o = (ctypes.c_double * 2)()
        lib.t_sum(form, form, 64, 64, w.ctypes.data_as(dp), f.ctypes.data_as(dp), o)
        assert o[0] == float((w[:, 0] * f[:, 0]).sum()) and o[1] == 0.0
