"""Old history by transforms (double far field, column tiles): runs that end
around the superblocks of 2048 rows, every block length, ragged members,
per-component orders and orders above 1, against the CPU oracle; a member's
bits alone and in a batch; a non-finite member beside good ones.

Bound: TOL_FP64, the parity bar of the double path (a transform of 4096 points
rounds its sums by a few units of 1e-16 of their size)."""
import numpy as np
import pytest

from paper_1710_01133_amd import abm, inputs
from gpu_common import TOL_FP64, normerr, oracle_run, run_batch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    torch.cuda.init()
    c = abm.Context(0)
    yield c
    c.close()


LCR = (1.015, 0.55, -1.02, -0.58)


def _mixed(Ns, g):
    probs = []
    for i, N in enumerate(Ns):
        probs.append(inputs.Problem("DUFFING", 0.95, 2 ** -8, N, (0.1, 0.0),
                                    (0.1, float(g.uniform(0.1, 0.6)), 1.2)))
        probs.append(inputs.Problem("LORENZ", 0.93, 2 ** -9, N, tuple(g.uniform(0.8, 1.2, 3)), inputs.LORENZ_P))
        probs.append(inputs.Problem("LCR", (0.9, 0.8), 0.004, N, (0.1, 0.0), LCR + (0.02 * i,)))
        probs.append(inputs.Problem("DIAG", (0.6, 1.3), 1 / 512, N, (1.0, -0.5), (1.3, 0.7, 0.2, -0.1),
                                    x1=(0.0, 0.25)))
    return probs


@pytest.mark.parametrize("L", [64, 128, 256, 512])
def test_superblock_edges(ctx, L, monkeypatch):
    monkeypatch.setenv("ABM_BLOCK_L", str(L))
    monkeypatch.setenv("ABM_NARROW", "0")
    probs = _mixed([2047, 2048, 2049, 4096, 4097, 6300, 2048 + L, 2049 + L], np.random.default_rng(L))
    outs, st = run_batch(ctx, probs, 1)
    assert st["n_groups"] == 4
    for p, y in zip(probs, outs):
        assert normerr(y, oracle_run(p, 1)) <= TOL_FP64, (p.rhs, p.N)


def test_member_alone_has_the_same_bits(ctx, monkeypatch):
    monkeypatch.setenv("ABM_NARROW", "0")
    probs = _mixed([7000, 5200, 3000], np.random.default_rng(5))
    outs, _ = run_batch(ctx, probs, 3)
    for i in (0, 1, 2, 3, 4, 9):
        (alone,), _ = run_batch(ctx, [probs[i]], 3)
        assert np.array_equal(alone, outs[i]), probs[i].rhs


def test_nonfinite_member_stays_alone(ctx):
    probs = inputs.duffing_sweep(B=6, N=5000)
    bad = inputs.Problem("DUFFING", 0.95, 2 ** -8, 5000, (1e3, 0.0), inputs.DUFFING_P)
    mix = probs[:3] + [bad] + probs[3:]
    plan = abm.Plan(ctx, mix, out_stride=1)
    ys = [abm.alloc_out(p, 1) for p in mix]
    abm.solve_batch(plan, mix, ys)
    with pytest.raises(abm.AbmError) as e:
        plan.check()
    assert e.value.code == abm.ABM_EDEVICE
    for p, y in zip(mix, ys):
        if p is not bad:
            assert normerr(y.cpu().numpy(), oracle_run(p, 1)) <= TOL_FP64
    plan.close()
