"""The launch shape of the plain path, on the host (no device work): every
reducer has workers, the workers hold every chunk, the launch fits the chip,
and what abm_solve_noalloc takes fits its arrays, for any forced workgroup
count too."""
import ctypes

import pytest

from paper_1710_01133_amd import abm, inputs

FAN, BLOCK, SLOT_BYTES, FLAG_PAD = 16, 64, 4 << 20, 32
NOALLOC_MAX = 341952


class Shape(ctypes.Structure):
    _fields_ = [("W", ctypes.c_int32), ("nred", ctypes.c_int32), ("nloc", ctypes.c_int32),
                ("nspill", ctypes.c_int32), ("work_doubles", ctypes.c_size_t), ("flags", ctypes.c_int)]


@pytest.fixture(scope="module")
def shape():
    f = abm.load()["_ZN3abm11plain_shapeERK11abm_problemiPNS_10PlainShapeE"]
    f.restype = ctypes.c_int32

    def call(p, n_cu=256):
        out = Shape()
        c = abm.c_problem(p, 0)
        return f(ctypes.byref(c), ctypes.c_int(n_cu), ctypes.byref(out)), out
    return call


def _problem(d, N, prec="fp64", orders=1):
    if d == 1:
        return inputs.Problem("LINEAR", 0.8, 1e-3, N, (1.0,), (1.0,), prec)
    if d == 2:
        return inputs.Problem("DUFFING", 0.9 if orders == 1 else (0.9, 0.8), 1e-3, N, (0.1, 0.0),
                              inputs.DUFFING_P, prec)
    return inputs.Problem("LORENZ", 0.9 if orders == 1 else (0.9, 0.8, 0.85), 1e-3, N, (1.0, 1.0, 1.0),
                          inputs.LORENZ_P, prec)


def _check(sh, p, n_cu):
    chunks = -(-p.N // BLOCK)
    if sh.W == 0:
        assert sh.nred == 0 and sh.work_doubles == 0
        return
    assert 1 + sh.W + sh.nred <= max(2, min(n_cu, 256))
    assert sh.nred == (0 if sh.W <= FAN else -(-sh.W // FAN))       # none without workers
    assert (sh.nloc + sh.nspill) * sh.W >= chunks and sh.flags >= FLAG_PAD + sh.W + sh.nred


@pytest.mark.parametrize("prec", ["fp64", "dd"])
@pytest.mark.parametrize("d", [1, 2, 3])
def test_forced_workgroup_counts(shape, d, prec, monkeypatch):
    for G in list(range(1, 70)) + [100, 255, 256, 257, 1000]:
        monkeypatch.setenv("ABM_PLAIN_G", str(G))
        for N in (1, 64, 2500, 20000, 300000):
            p = _problem(d, N, prec)
            st, sh = shape(p)
            assert st == abm.ABM_OK
            _check(sh, p, 256)
            assert sh.work_doubles * 8 <= SLOT_BYTES or prec == "dd"


@pytest.mark.parametrize("n_cu", [2, 16, 32, 38, 64, 128, 256, 304])
@pytest.mark.parametrize("d,orders", [(1, 1), (2, 1), (2, 2), (3, 1), (3, 3)])
def test_default_shapes(shape, d, orders, n_cu):
    for N in (1, 63, 64, 2048, 2049, 17000, 17500, 100000, NOALLOC_MAX // orders, 10 ** 6, 2 * 10 ** 6):
        p = _problem(d, N, orders=orders)
        st, sh = shape(p, n_cu)
        if st != abm.ABM_OK:
            assert st == abm.ABM_EINVAL and N > 3000
            continue
        _check(sh, p, n_cu)
        if N * orders <= NOALLOC_MAX:
            assert sh.work_doubles * 8 <= SLOT_BYTES
