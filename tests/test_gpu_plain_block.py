"""The blocked plain kernel (abm_solve) where its dispatch and its blocks have
edges, against the CPU oracle: step counts around the 64-step blocks and
around the length from which several workgroups share the history; workgroup
counts around the 16 partials that one workgroup sums; a history that does
not fit its workers' LDS; per-component orders in each of these forms.

Bound: TOL_FP64, the parity bar of the double path (both sides sum the same
products in double in another order)."""
import numpy as np
import pytest

from paper_1710_01133_amd import abm, inputs
from gpu_common import TOL_FP64, normerr, oracle_run, run_plain

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.init()
    c = abm.Context(0)
    yield c
    c.close()


LCR = (1.015, 0.55, -1.02, -0.58, 0.117)
SYSTEMS = {
    "LINEAR": lambda N: inputs.Problem("LINEAR", 0.7, 0.01, N, (1.0,), (1.3,)),
    "DUFFING": lambda N: inputs.duffing_single(N=N, h=2e-3),
    "LORENZ": lambda N: inputs.Problem("LORENZ", (0.95, 0.9, 0.93), 2.0 ** -9, N, (1.0, 1.0, 1.0),
                                       inputs.LORENZ_P),
    "LCR": lambda N: inputs.Problem("LCR", (0.9, 0.8), 0.005, N, (1.2, -0.4), LCR),
    "DIAG": lambda N: inputs.Problem("DIAG", (0.6, 1.3), 1 / 256, N, (1.0, -0.5),
                                     (1.3, 0.7, 0.2, -0.1), x1=(0.0, 0.25)),
}


@pytest.mark.parametrize("rhs", list(SYSTEMS))
@pytest.mark.parametrize("N", [63, 64, 65, 128, 129, 192, 193, 2048, 2049, 4100])
def test_block_and_dispatch_edges(ctx, rhs, N):
    p = SYSTEMS[rhs](N)
    assert normerr(run_plain(ctx, p, 1), oracle_run(p, 1)) <= TOL_FP64


@pytest.mark.parametrize("rhs", ["DUFFING", "LORENZ"])
@pytest.mark.parametrize("G", [2, 16, 17, 18, 19, 35, 256])
def test_workers_and_reducers(ctx, rhs, G, monkeypatch):
    """One worker; 15, 16 workers summed by the stepping workgroup; 16, 17
    and 32 summed by one and two reducers; as many as the chip holds."""
    monkeypatch.setenv("ABM_PLAIN_G", str(G))
    p = SYSTEMS[rhs](2500)
    assert normerr(run_plain(ctx, p, 7), oracle_run(p, 7)) <= TOL_FP64


@pytest.mark.parametrize("rhs", ["DUFFING", "LCR"])
def test_history_beyond_the_workers_lds(ctx, rhs, monkeypatch):
    """One worker holds 119 chunks of 64 rows of two components in LDS: with
    9000 steps the rest lie in device memory."""
    monkeypatch.setenv("ABM_PLAIN_G", "2")
    p = SYSTEMS[rhs](9000)
    p.h = 2e-3
    assert normerr(run_plain(ctx, p, 1), oracle_run(p, 1)) <= TOL_FP64


def test_two_plans_in_turn_on_one_stream(ctx):
    """Two plans' solves in turn without a wait: each keeps its own flags and slots."""
    ps = [inputs.duffing_single(N=5000), inputs.duffing_single(N=7001, A=0.5)]
    plans = [abm.Plan(ctx, [p], out_stride=1) for p in ps]
    ys = [abm.alloc_out(p, 1) for p in ps]
    for _ in range(3):
        for p, plan, y in zip(ps, plans, ys):
            abm.solve(plan, p, y)
    for p, plan, y in zip(ps, plans, ys):
        plan.check()
        assert normerr(y.cpu().numpy(), oracle_run(p, 1)) <= TOL_FP64
        assert np.array_equal(y.cpu().numpy(), run_plain(ctx, p, 1))
        plan.close()
