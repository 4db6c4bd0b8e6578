"""The history chunk of double column tiles: the caller's is used and
reported, the default is what the plan reports, a reported blocking can be
given back, and the autotuner tries chunks that differ.

Bound: TOL_FP64, the parity bar of the double path."""
import numpy as np
import pytest

from paper_1710_01133_amd import abm, inputs
from gpu_common import TOL_FP64, normerr, oracle_run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.init()
    c = abm.Context(0)
    yield c
    c.close()


def _solve(ctx, probs, tuning, stride=3):
    plan = abm.Plan(ctx, probs, out_stride=stride, tuning=tuning)
    cfg = plan.config()
    ys = [abm.alloc_out(p, stride) for p in probs]
    abm.solve_batch(plan, probs, ys)
    plan.check()
    plan.close()
    return [y.cpu().numpy() for y in ys], cfg


# below and beyond the first superblock of 2048 rows
@pytest.mark.parametrize("N", [1900, 5000])
def test_the_callers_chunk_is_used(ctx, N):
    probs = inputs.duffing_sweep(B=24, N=N)
    outs = {}
    for kc in (0, 256, 512, 1024, 2048):
        t = dict(block_L=128, kchunk=kc, max_split=8, column_tiles_only=0)
        outs[kc], cfg = _solve(ctx, probs, t)
        assert cfg == dict(t, kchunk=kc or 256)
        for i in (0, 11, 23):
            assert normerr(outs[kc][i], oracle_run(probs[i], 3)) <= TOL_FP64, kc
    same = lambda a, b: all(np.array_equal(x, y) for x, y in zip(outs[a], outs[b]))
    assert same(0, 256)
    # other slices of the history: other roundings
    assert not same(256, 512) and not same(512, 1024) and not same(1024, 2048)


def test_chunks_refused_and_reported(ctx):
    double = inputs.duffing_sweep(B=24, N=1000)
    both = double + inputs.duffing_sweep(B=24, N=1000, far_prec="fp32")
    for probs, kc in ((double, 128), (double, 384), (both, 256)):
        with pytest.raises(abm.AbmError) as e:
            abm.Plan(ctx, probs, tuning=dict(block_L=0, kchunk=kc, max_split=0, column_tiles_only=0))
        assert e.value.code == abm.ABM_EINVAL, kc
    plan = abm.Plan(ctx, both)
    assert plan.config()["kchunk"] == 2048
    plan.close()


def test_autotune_tries_chunks_that_differ(ctx):
    probs = inputs.duffing_sweep(B=24, N=5000)
    best, trials = abm.autotune(ctx, probs, out_stride=3, budget_s=60.0)
    assert {t["cfg"]["kchunk"] for t in trials} == {256, 512, 1024, 2048}
    outs, cfg = _solve(ctx, probs, best)
    assert cfg == best
    for i in (0, 23):
        assert normerr(outs[i], oracle_run(probs[i], 3)) <= TOL_FP64


def test_autotune_of_narrow_groups_tries_no_chunks(ctx):
    probs = [inputs.Problem("LORENZ", 0.95, 2 ** -8, 2500, (1.0, 1.0, 1.0), inputs.LORENZ_P, "fp32")]
    _, trials = abm.autotune(ctx, probs, out_stride=0, budget_s=60.0)
    tiles = [t for t in trials if t["cfg"]["column_tiles_only"]]
    assert len({t["cfg"]["kchunk"] for t in trials}) == 1 and len(tiles) == 1
