"""Forms of the plain path's launch that short runs do not take by themselves:
reducers with few workers, and chunks beyond the workers' LDS (119, 119 and 71
chunks of 64 rows are kept of one, two and three components, 39 and 18 of two
and three in double-double) with one worker and with 17 of them and two
reducers, in both arithmetics.

Bounds: TOL_FP64 and TOL_DD, the parity bars against the oracles; long runs
against the default shape of the same problem, which sums in another order."""
import numpy as np
import pytest

from paper_1710_01133_amd import inputs
from gpu_common import TOL_FP64, normerr, oracle_run, run_plain
from test_gpu_dd import TOL_DD, ctx, err_pairs, quad_run, run_dd  # noqa: F401

pytestmark = pytest.mark.gpu

LCR = (1.015, 0.55, -1.02, -0.58, 0.117)
SYSTEMS = {
    "LINEAR": lambda N: inputs.Problem("LINEAR", 0.7, 0.01, N, (1.0,), (1.3,)),
    "DUFFING": lambda N: inputs.duffing_single(N=N, h=2e-3),
    "LORENZ": lambda N: inputs.Problem("LORENZ", 0.9, 2.0 ** -10, N, (1.0, 1.0, 1.0), inputs.LORENZ_P),
    "LORENZ3": lambda N: inputs.Problem("LORENZ", (0.95, 0.9, 0.93), 2.0 ** -10, N, (1.0, 1.0, 1.0),
                                        inputs.LORENZ_P),
    "LCR2": lambda N: inputs.Problem("LCR", (0.9, 0.8), 2e-3, N, (1.2, -0.4), LCR),
}


# 16 workers (a 19th workgroup would be a reducer without any); 17 and 18
# workers (the second reducer sums one and two); 33 (the third sums one)
@pytest.mark.parametrize("rhs", ["LINEAR", "LORENZ3"])
@pytest.mark.parametrize("G", [19, 20, 21, 37])
def test_reducers_with_few_workers(ctx, rhs, G, monkeypatch):  # noqa: F811
    monkeypatch.setenv("ABM_PLAIN_G", str(G))
    p = SYSTEMS[rhs](2500)
    assert normerr(run_plain(ctx, p, 7), oracle_run(p, 7)) <= TOL_FP64
    assert err_pairs(run_dd(ctx, p, 7), quad_run(p, 7)) <= TOL_DD


@pytest.mark.parametrize("rhs,N", [("LINEAR", 9100), ("LORENZ", 5000), ("LORENZ3", 5000)])
def test_one_worker_spills(ctx, rhs, N, monkeypatch):  # noqa: F811
    monkeypatch.setenv("ABM_PLAIN_G", "2")
    p = SYSTEMS[rhs](N)
    assert normerr(run_plain(ctx, p, 1), oracle_run(p, 1)) <= TOL_FP64


@pytest.mark.parametrize("rhs,N", [("DUFFING", 3000), ("LCR2", 3001), ("LORENZ", 1500), ("LORENZ3", 1500)])
def test_one_worker_spills_in_double_double(ctx, rhs, N, monkeypatch):  # noqa: F811
    monkeypatch.setenv("ABM_PLAIN_G", "2")
    p = SYSTEMS[rhs](N)
    assert err_pairs(run_dd(ctx, p, 1), quad_run(p, 1)) <= TOL_DD


@pytest.mark.parametrize("rhs,N", [("DUFFING", 140000), ("LORENZ", 80000), ("LORENZ3", 80000)])
def test_workers_and_reducers_spill(ctx, rhs, N, monkeypatch):  # noqa: F811
    p = SYSTEMS[rhs](N)
    ref = run_plain(ctx, p, 50)
    monkeypatch.setenv("ABM_PLAIN_G", "20")
    y = run_plain(ctx, p, 50)
    assert not np.array_equal(y, ref) and normerr(y, ref) <= TOL_FP64


@pytest.mark.parametrize("rhs,N", [("DUFFING", 45000), ("LCR2", 45000), ("LORENZ", 21000)])
def test_workers_and_reducers_spill_in_double_double(ctx, rhs, N, monkeypatch):  # noqa: F811
    p = SYSTEMS[rhs](N)
    ref = run_dd(ctx, p, 50)
    monkeypatch.setenv("ABM_PLAIN_G", "20")
    y = run_dd(ctx, p, 50)
    assert not np.array_equal(y, ref) and err_pairs(y, ref) <= TOL_DD


def test_default_shape_spills_in_double_double(ctx):  # noqa: F811
    """640000 steps of two components, 240 workers of 42 chunks each, 39 of
    them in LDS: against the double path."""
    p = inputs.duffing_single(N=640000)
    y = run_dd(ctx, p, 1000)
    assert normerr(y[..., 0] + y[..., 1], run_plain(ctx, p, 1000)) <= TOL_FP64
