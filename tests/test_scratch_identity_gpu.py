"""Just below the size of the scratch array, where the default tiles would leave
too many sums, every entry point takes the same deeper tiles: equal bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# Sums some ten thousand bytes too many at the default depth, and as many to
# spare at the depth taken instead.
@pytest.mark.parametrize("shape,C", [((206, 348, 55), 16), ((65, 1403, 147), 4), ((69, 961, 337), 2)])
@pytest.mark.parametrize("steps,eps", [(1, 0.0), (6, 1e-4)])
def test_every_call_has_the_bits_of_the_scratch_solve(shape, C, steps, eps):
    import torch
    from paper_2002_01981_amd import PIFCM_SWARM_BATCHED, PIFCM_SWARM_PLAIN, Context, Params
    ctx = Context(0)
    g = torch.Generator(device="cuda").manual_seed(91)
    x = torch.rand(shape, generator=g, device="cuda")
    U0 = torch.rand((x.numel(), C), generator=g, device="cuda") + 0.1
    U0 /= U0.sum(1, keepdim=True)
    c0 = np.linspace(0.05, 0.95, C).astype(np.float32)
    p = Params(C=C, m=2.0, eps=eps, max_iter=steps)
    a = ctx.ifcm_solve_noalloc(x, p, 0.3, 0.4, c0, U_in=U0, labels=True, want_hist=True)
    b = ctx.ifcm_solve(x, p, 0.3, 0.4, c0, U_in=U0, labels=True, want_hist=True)
    assert a["iters"] == b["iters"] and a["J"] == b["J"] and np.array_equal(a["c"], b["c"])
    assert np.array_equal(a["J_hist"], b["J_hist"])
    assert torch.equal(a["U"], b["U"]) and torch.equal(a["labels"], b["labels"])
    parts = np.tile(np.array([0.3, 0.4], np.float32), (1, 2, 1))
    for mode in (PIFCM_SWARM_BATCHED, PIFCM_SWARM_PLAIN):
        s = ctx.swarm_evaluate([x], p, parts, c0[None], [U0], mode=mode)
        assert np.all(s["fitness"] == a["J"]) and np.all(s["iters"] == a["iters"])
        assert all(np.array_equal(c, a["c"]) for c in s["centres"][0])
    ctx.close()
