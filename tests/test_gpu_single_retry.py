"""abm_solve_batch of one double trajectory where a device-side wait of its
first run gives up (forced from the host: the ABM_WAIT_BIAS hook raises every
awaited number of that run beyond reach, ABM_SPIN_LIMIT bounds its waits at 64
polls): the trajectory is taken again in a smaller shape and nothing is
reported; abm_solve still reports its own failures, and a non-finite state is
reported either way.

Bound: TOL_FP64, the parity bar of the double path."""
import numpy as np
import pytest

from paper_1710_01133_amd import abm, inputs
from gpu_common import TOL_FP64, normerr, oracle_run, run_plain

pytestmark = pytest.mark.gpu

LCR = (1.015, 0.55, -1.02, -0.58, 0.117)


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.init()
    c = abm.Context(0)
    yield c
    c.close()


def _hooks(monkeypatch, on):
    for name, v in (("ABM_SPIN_LIMIT", "64"), ("ABM_WAIT_BIAS", str(1 << 30))):
        monkeypatch.setenv(name, v) if on else monkeypatch.delenv(name, raising=False)


def _batch(ctx, p, stride):
    plan = abm.Plan(ctx, [p], out_stride=stride)
    y = abm.alloc_out(p, stride)
    st = abm.solve_batch(plan, [p], [y])
    assert st["far_launches"] == 0
    return plan, y


# one, three and 20 workers in the first run (the last with reducers, cut to 16)
@pytest.mark.parametrize("N", [2049, 3000, 20011])
@pytest.mark.parametrize("rhs", ["DUFFING", "LCR"])
def test_a_run_whose_waits_give_up_is_taken_again(ctx, rhs, N, monkeypatch):
    p = inputs.duffing_single(N=N, h=2e-3) if rhs == "DUFFING" else \
        inputs.Problem("LCR", (0.9, 0.8), 0.003, N, (1.2, -0.4), LCR)
    plain = run_plain(ctx, p, 7)
    _hooks(monkeypatch, True)
    plan, y = _batch(ctx, p, 7)
    plan.check()
    again = y.cpu().numpy()
    assert normerr(again, oracle_run(p, 7)) <= TOL_FP64
    if N <= 3000:
        assert np.array_equal(again, plain)      # the same shape
    # and without the hooks the same plan's first run stands
    _hooks(monkeypatch, False)
    abm.solve_batch(plan, [p], [y])
    plan.check()
    plan.close()
    assert np.array_equal(y.cpu().numpy(), plain)


def test_taken_again_with_a_history_beyond_the_lds(ctx, monkeypatch):
    """130000 steps: 16 workers keep 119 of their 127 chunks in LDS."""
    p = inputs.duffing_single(N=130000)
    plain = run_plain(ctx, p, 100)
    _hooks(monkeypatch, True)
    plan, y = _batch(ctx, p, 100)
    plan.check()
    plan.close()
    assert normerr(y.cpu().numpy(), plain) <= TOL_FP64


def test_failures_are_still_reported(ctx, monkeypatch):
    p = inputs.duffing_single(N=3000, h=2e-3)
    _hooks(monkeypatch, True)
    plan, y = _batch(ctx, p, 0)
    plan.check()
    z = abm.alloc_out(p, 0)
    abm.solve(plan, p, z)                        # abm_solve's own waits
    abm.solve_batch(plan, [p], [y])
    with pytest.raises(abm.AbmError) as e:
        plan.check()
    assert e.value.code == abm.ABM_EDEVICE
    assert np.isnan(z.cpu().numpy()).all() and np.isfinite(y.cpu().numpy()).all()
    plan.close()


@pytest.mark.parametrize("hooks", [False, True])
def test_a_nonfinite_state_is_reported(ctx, hooks, monkeypatch):
    p = inputs.Problem("DUFFING", 0.95, 2 ** -8, 4000, (1e3, 0.0), inputs.DUFFING_P)
    _hooks(monkeypatch, hooks)
    plan, y = _batch(ctx, p, 0)
    with pytest.raises(abm.AbmError) as e:
        plan.check()
    assert e.value.code == abm.ABM_EDEVICE
    plan.check()                                 # cleared by the report
    plan.close()
