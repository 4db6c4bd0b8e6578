"""Plans under a bound on their device memory (the ABM_PLAN_MEM_MIB test hook
fails allocations beyond it, as a full device does): a plan of double column
tiles fits wherever its direct products fit, whether or not the spectra of its
history do, and gives the same states to rounding in both forms.

Bound: TOL_FP64, the parity bar of the double path."""
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


def _problems(N):
    """Two groups (two orders) of 48 oscillators each, at two lengths."""
    probs = inputs.duffing_sweep(B=96, N=N)
    for i, p in enumerate(probs):
        p.alpha = 0.95 if i % 2 else 0.9
        p.N = N if i < 4 else N - 700
    return probs


def _scan(ctx, probs, bounds, stride, checked, monkeypatch):
    """Plans under rising bounds (MiB): refused up to some bound, accepted from
    it on; returns it.  Both forms are seen and solved."""
    seen = {}
    for mib in bounds:
        monkeypatch.setenv("ABM_PLAN_MEM_MIB", str(mib))
        try:
            plan = abm.Plan(ctx, probs, out_stride=stride)
        except abm.AbmError as e:
            assert e.code == abm.ABM_ENOMEM
            assert not seen, "refused at %d MiB, accepted at %d" % (mib, min(seen))
            continue
        ys = [abm.alloc_out(p, stride) for p in probs]
        far = abm.solve_batch(plan, probs, ys)["far_macs"]
        plan.check()
        plan.close()
        if far not in seen.values():
            for i, tol in checked:
                assert normerr(ys[i].cpu().numpy(), oracle_run(probs[i], stride)) <= tol, (mib, i)
        seen[mib] = far
    # the direct form at the smallest bounds, the spectra from some bound on
    forms = list(seen.values())
    assert len(set(forms)) == 2 and forms == sorted(forms, reverse=True), seen
    return min(seen)


@pytest.mark.parametrize("L", [64, 256])
def test_a_plan_fits_wherever_its_direct_products_fit(ctx, L, monkeypatch):
    monkeypatch.setenv("ABM_BLOCK_L", str(L))
    probs = _problems(6000)
    history = sum(8 * p.d * p.N for p in probs)
    least = _scan(ctx, probs, range(2, 74, 2), 500,
                  [(i, TOL_FP64) for i in (0, 3, 50, 95)], monkeypatch)
    assert least << 20 < 3 * history


def test_one_group_with_transforms_beside_short_and_reduced_ones(ctx, monkeypatch):
    """Groups that never reach a second superblock, or are not double, share
    the plan's schedule in both forms."""
    probs = inputs.duffing_sweep(B=16, N=5000) + inputs.duffing_sweep(B=16, N=1900, alpha=0.9) \
        + inputs.duffing_sweep(B=16, N=3000, far_prec="bf16x6")
    _scan(ctx, probs, range(1, 25), 100, [(2, TOL_FP64), (20, TOL_FP64), (40, 1e-6)], monkeypatch)
