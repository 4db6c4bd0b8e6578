"""abm_solve_batch of one double trajectory: without a blocking it runs as
abm_solve (the same bits), with one it runs the blocked method at that
blocking; the plan reports which, and the autotuner compares the two.

Bound: TOL_FP64, the parity bar of the double path."""
import numpy as np
import pytest

from paper_1710_01133_amd import abm, inputs
from gpu_common import TOL_FP64, normerr, oracle_run, run_plain

pytestmark = pytest.mark.gpu

NONE = dict(block_L=0, kchunk=0, max_split=0, column_tiles_only=0)


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.init()
    c = abm.Context(0)
    yield c
    c.close()


def _solve(ctx, p, stride, tuning):
    plan = abm.Plan(ctx, [p], out_stride=stride, tuning=tuning)
    y = abm.alloc_out(p, stride)
    st = abm.solve_batch(plan, [p], [y])
    plan.check()
    cfg = plan.config()
    plan.close()
    return y.cpu().numpy(), st, cfg


@pytest.mark.parametrize("N", [700, 5000])
@pytest.mark.parametrize("given", [dict(block_L=128), dict(block_L=256), dict(max_split=4), dict(kchunk=512)])
def test_a_given_blocking_is_used(ctx, N, given):
    p = inputs.duffing_single(N=N, h=2e-3)
    y, st, cfg = _solve(ctx, p, 1, dict(NONE, **given))
    assert st["far_launches"] > 0 and st["chain_launches"] == -(-N // cfg["block_L"])
    assert all(cfg[k] == v for k, v in given.items())
    assert normerr(y, oracle_run(p, 1)) <= TOL_FP64


def test_a_blocking_of_the_environment_is_used(ctx, monkeypatch):
    p = inputs.duffing_single(N=3000, h=2e-3)
    monkeypatch.setenv("ABM_BLOCK_L", "64")
    y, st, cfg = _solve(ctx, p, 1, None)
    assert st["far_launches"] > 0 and cfg["block_L"] == 64
    assert normerr(y, oracle_run(p, 1)) <= TOL_FP64


@pytest.mark.parametrize("tuning", [None, NONE])
def test_without_a_blocking_as_abm_solve(ctx, tuning):
    p = inputs.duffing_single(N=5000, h=2e-3)
    y, st, cfg = _solve(ctx, p, 1, tuning)
    assert st["far_launches"] == 0 and st["chain_launches"] == 1 and cfg == NONE
    assert np.array_equal(y, run_plain(ctx, p, 1))


@pytest.mark.parametrize("budget", [0.0, 60.0])
def test_autotune_compares_the_two(ctx, budget):
    p = inputs.duffing_single(N=6000)
    best, trials = abm.autotune(ctx, [p], out_stride=10, budget_s=budget)
    assert trials[0]["cfg"] == NONE
    if budget:
        assert {t["cfg"]["block_L"] for t in trials[1:]} >= {64, 128, 256, 512}
    y, st, cfg = _solve(ctx, p, 10, best)
    assert cfg == best and (st["far_launches"] == 0) == (best == NONE)
    assert normerr(y, oracle_run(p, 10)) <= TOL_FP64


def test_autotune_of_a_reduced_precision_tries_blockings_only(ctx):
    p = inputs.duffing_single(N=3000)
    p.far_prec = "fp32"
    _, trials = abm.autotune(ctx, [p], out_stride=10, budget_s=60.0)
    assert all(t["cfg"]["block_L"] > 0 for t in trials)
