"""The blocked convolution of one double trajectory (a blocking given: without
one abm_solve_batch runs it as abm_solve), against the plain path, the oracle
and column tiles.  abm_stats shows the route: far_launches is 0 on the plain
one.

Bounds: TOL_FP64 against the oracle; 1e-12 between the two paths over 2e5 and
1e6 steps and 1e-13 against column tiles, as where the routes were first
compared; single steps recomputed by the oracle from the GPU's own states
within gpu_common.check_steps_fp64's rounding bound."""
import numpy as np
import pytest

from paper_1710_01133_amd import abm, inputs
from gpu_common import TOL_FP64, check_steps_fp64, normerr, oracle_run, run_batch, run_plain, sampled_steps

pytestmark = pytest.mark.gpu

BLOCKED = dict(block_L=256, kchunk=0, max_split=0, column_tiles_only=0)
LCR = (1.015, 0.55, -1.02, -0.58)


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.init()
    c = abm.Context(0)
    yield c
    c.close()


def run_blocked(ctx, p, stride, **tuning):
    plan = abm.Plan(ctx, [p], out_stride=stride, tuning=dict(BLOCKED, **tuning))
    y = abm.alloc_out(p, stride)
    st = abm.solve_batch(plan, [p], [y])
    plan.check()
    plan.close()
    assert st["far_launches"] > 0
    assert st["narrow_groups"] == (0 if tuning.get("column_tiles_only") else 1)
    return y.cpu().numpy()


@pytest.mark.parametrize("N,stride", [(200000, 100), (1000000, 1000)])
def test_blocked_matches_plain(ctx, N, stride):
    p = inputs.duffing_single(N=N, h=200.0 / N)
    a, b = run_blocked(ctx, p, stride), run_plain(ctx, p, stride)
    assert np.all(np.isfinite(a)) and np.max(np.abs(a)) < 10
    assert not np.array_equal(a, b) and normerr(a, b) <= 1e-12


@pytest.mark.parametrize("kind", ["lcr", "duffing"])
def test_million_steps_recomputed(ctx, kind):
    N = 1000000
    p = inputs.Problem("LCR", 0.9, 0.01, N, (0.1, 0.0), inputs.LCR_P + (0.117,)) if kind == "lcr" else \
        inputs.duffing_single(N=N)
    y = run_blocked(ctx, p, 1)
    assert np.all(np.isfinite(y))
    check_steps_fp64(p, y, sampled_steps(N))
    assert np.array_equal(run_blocked(ctx, p, 0)[0], y[-1])


@pytest.mark.parametrize("L", [64, 128, 256, 512])
def test_long_trajectory_vs_oracle(ctx, L):
    p = inputs.duffing_single(N=20000)
    assert normerr(run_blocked(ctx, p, 1, block_L=L), oracle_run(p, 1)) <= TOL_FP64


@pytest.mark.parametrize("i", [0, 3])
def test_a_member_alone_beside_its_batch(ctx, i):
    """The blocked convolution sums in another order than the batch's column
    tiles; alone in column tiles a member has the batch's bits."""
    probs = [inputs.Problem("DUFFING", 0.95, 2 ** -8, N, (0.1, 0.0), (0.1, A, 1.2))
             for N, A in ((7000, 0.2), (5200, 0.3), (2500, 0.5), (900, 0.6))]
    probs += [inputs.Problem("DUFFING", 0.95, 2 ** -8, 1000, (0.1, 0.0), (0.1, 0.4, 1.2))] * 12
    outs, st = run_batch(ctx, probs, 1)
    assert st["narrow_groups"] == 0
    assert normerr(run_blocked(ctx, probs[i], 1), outs[i]) <= 1e-13
    assert np.array_equal(run_blocked(ctx, probs[i], 1, column_tiles_only=1), outs[i])


def test_incommensurate_narrow_vs_tiles(ctx):
    p = inputs.Problem("LCR", (0.9, 0.8), 0.01, 3600, (1.2, -0.4), LCR + (0.117,))
    ref = oracle_run(p, 1)
    yn, yt = run_blocked(ctx, p, 1), run_blocked(ctx, p, 1, column_tiles_only=1)
    assert normerr(yn, ref) <= TOL_FP64 and normerr(yt, ref) <= TOL_FP64 and normerr(yn, yt) <= 1e-13
