"""Old history by transforms under every schedule: with the far field and the
chains on alternating or fixed streams or on one, eager or replayed from a
graph, every state has the same bits.  Wide groups, so that a superblock's
transforms outlast the first far fields that read their sums; members that end
inside, at and after the superblocks' starts."""
import numpy as np
import pytest

from paper_1710_01133_amd import abm, inputs
from gpu_common import TOL_FP64, normerr, oracle_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [64, 256, 512])
def test_schedules_give_the_same_bits(L, monkeypatch):
    import torch
    assert torch.cuda.is_available()
    torch.cuda.init()
    ctx = abm.Context(0)
    monkeypatch.setenv("ABM_BLOCK_L", str(L))
    probs = inputs.duffing_sweep(B=1000, N=7000)
    for i, p in enumerate(probs):
        p.N = (7000, 6144, 6145, 4096 + L, 4097, 5000)[i % 6]
    ref = None
    for alt, overlap, graph in ((0, 0, False), (1, 1, False), (0, 1, False), (1, 1, True), (0, 1, True)):
        monkeypatch.setenv("ABM_ALT_STREAMS", str(alt))
        monkeypatch.setenv("ABM_OVERLAP", str(overlap))
        plan = abm.Plan(ctx, probs, out_stride=500)
        plan.graph(graph)
        sizes = [abm.n_out(p.N, 500) * 2 for p in probs]
        at = np.concatenate([[0], np.cumsum(sizes)])
        buf = torch.zeros(int(at[-1]), dtype=torch.float64, device="cuda")
        ys = [buf[a:b] for a, b in zip(at[:-1], at[1:])]
        torch.cuda.synchronize()
        for _ in range(3 if graph else 2):       # capture and replays
            buf.fill_(np.nan)
            torch.cuda.synchronize()
            assert abm.solve_batch(plan, probs, ys)["transform_launches"] == 6
            plan.check()
            got = buf.cpu().numpy()
            ref = got if ref is None else ref
            assert np.array_equal(got, ref), (alt, overlap, graph)
        plan.close()
    for i in (0, 1, 2, 3, 4, 999):
        y = ref[at[i]:at[i + 1]].reshape(-1, 2)
        assert normerr(y, oracle_run(probs[i], 500)) <= TOL_FP64
    ctx.close()
