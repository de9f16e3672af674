"""Swarms on both sides of eight rounds of work items, where the grid of the
fused step turns persistent (two waves per SIMD at C = 6): every particle has
the bits of its own solve."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# 605 tiles a particle on up to 3072 wave slots: 8 rounds are 40.6 particles.
@pytest.mark.parametrize("C,m", [(6, 2.0), (6, 2.5), (5, 2.0)])
@pytest.mark.parametrize("P", [40, 41, 55])
def test_swarm_equals_solves(C, m, P):
    import torch
    from paper_2002_01981_amd import Context, Params
    ctx = Context(0)
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.rand((12, 217, 164), generator=g, device="cuda")
    U0 = torch.rand((x.numel(), C), generator=g, device="cuda") + 0.1
    U0 /= U0.sum(1, keepdim=True)
    c0 = np.linspace(0.1, 0.9, C).astype(np.float32)
    parts = (np.random.default_rng(P).random((P, 2)) * 0.45).astype(np.float32)
    p = Params(C=C, m=m, eps=0.0, max_iter=3)
    r = ctx.swarm_evaluate([x], p, parts, c0[None], [U0])
    for q in (0, 1, P // 2, P - 2, P - 1):
        s = ctx.ifcm_solve(x, p, float(parts[q, 0]), float(parts[q, 1]), c0, U_in=U0)
        assert s["J"] == r["fitness"][0, q] and np.array_equal(s["c"], r["centres"][0, q])
    ctx.close()
