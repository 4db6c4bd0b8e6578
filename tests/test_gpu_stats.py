"""abm_stats of a double sweep whose old history goes through transforms:
far_launches, far_ms and far_macs describe the direct products alone, so that
their quotient is a rate; the transforms have a count of their own."""
import pytest

from paper_1710_01133_amd import abm, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,L", [(2048, 256), (2049, 256), (9000, 256), (9000, 128)])
def test_transforms_are_counted_apart(N, L, monkeypatch):
    import torch
    assert torch.cuda.is_available()
    monkeypatch.setenv("ABM_BLOCK_L", str(L))
    ctx = abm.Context(0)
    probs = inputs.duffing_sweep(B=24, N=N)
    plan = abm.Plan(ctx, probs, out_stride=0)
    ys = [abm.alloc_out(p, 0) for p in probs]
    # blocks m >= 2 have history older than the block before; right after a
    # superblock of 2048 rows began all of it went through the transforms
    blocks = range(2, (N + L - 1) // L)
    rows = {m: (m - 1) * L - max(0, m * L // 2048 * 2048 - L) for m in blocks}
    macs = sum(p.d * min(L, N - m * L) * k for p in probs for m, k in rows.items())
    for mode in ("eager", "timed", "graph"):
        plan.timing(mode == "timed")
        plan.graph(mode == "graph")
        st = abm.solve_batch(plan, probs, ys)
        plan.check()
        assert st["far_launches"] <= len(blocks)
        assert st["transform_launches"] == 2 * ((N - 1) // 2048)
        assert st["far_macs"] == macs
        assert (st["far_ms"] > 0) == (mode == "timed")
    plan.close()
    ctx.close()
