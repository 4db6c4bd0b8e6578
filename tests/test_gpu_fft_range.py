"""Old history by transforms near the ends of the double range: the linear
equation scaled by a power of two gives every state scaled by it, bit for bit,
as the direct products do as long as no product under- or overflows."""
import numpy as np
import pytest

from paper_1710_01133_amd import abm, inputs
from gpu_common import TOL_FP64, normerr, oracle_run, run_batch

pytestmark = pytest.mark.gpu


# the direct sums of the 9000 steps stay below 2^(e + 18)
@pytest.mark.parametrize("alpha,e", [(0.6, -960), (0.95, -960), (1.4, -960), (0.6, 1005), (0.95, 1005), (1.4, 1004)])
def test_states_scale_by_powers_of_two(alpha, e, monkeypatch):
    import torch
    assert torch.cuda.is_available()
    torch.cuda.init()
    ctx = abm.Context(0)
    monkeypatch.setenv("ABM_NARROW", "0")
    lam = np.random.default_rng(9).uniform(0.5, 1.5, 40)
    x1 = (0.0,) if alpha > 1 else None

    def probs(scale):
        return [inputs.Problem("LINEAR", alpha, 2.0 ** -9, 9000 - 130 * i, (scale,), (float(v),), x1=x1)
                for i, v in enumerate(lam)]
    base, st = run_batch(ctx, probs(1.0), 1)
    assert st["transform_launches"] > 0
    far, _ = run_batch(ctx, probs(2.0 ** e), 1)
    for p, y, z in zip(probs(1.0), base, far):
        assert np.array_equal(np.ldexp(y, e), z), p.p
    for i in (0, 39):
        assert normerr(base[i], oracle_run(probs(1.0)[i], 1)) <= TOL_FP64
    ctx.close()
