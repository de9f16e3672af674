"""ifcm_solve_noalloc where it runs kernel instances of its own, without spilled
registers (C = 6 with m != 2, C = 11 and 12), and where the sums of many slots
are added with fewer loads in flight (C >= 10): the bits of ifcm_solve, which is
held to the oracle over one step."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import TOL, dev, host, random_memberships_f32, rel

pytestmark = pytest.mark.gpu


# More than 1024 slots of sums and fewer than 256.
@pytest.mark.parametrize("shape", [(9, 131, 260), (6, 20, 33)])
@pytest.mark.parametrize("C,m", [(6, 2.5), (6, 2.0), (9, 2.0), (10, 2.0), (11, 2.0), (11, 1.7), (12, 2.0), (12, 2.5),
                                 (13, 2.0), (14, 2.0), (16, 2.0)])
def test_same_bits(shape, C, m):
    import torch
    from paper_2002_01981_amd import Context, Params
    ctx = Context(0)
    raw, _ = synth.random_ellipsoids(shape=shape, seed=70 + C, sigma=0.07, count=12)
    x = oracle.normalize(raw)
    U0 = random_memberships_f32(np.random.default_rng(C), x.size, C)
    c0 = np.linspace(0.05, 0.95, C).astype(np.float32)
    xg, Ug = dev(x), dev(U0)
    for hist, T in ((False, 1), (False, 4), (True, 3)):
        p = Params(C=C, m=m, eps=0.0, max_iter=T)
        a = ctx.ifcm_solve_noalloc(xg, p, 0.3, 0.4, c0, U_in=Ug, want_hist=hist)
        b = ctx.ifcm_solve(xg, p, 0.3, 0.4, c0, U_in=Ug, want_hist=hist)
        assert a["J"] == b["J"] and np.array_equal(a["c"], b["c"]) and torch.equal(a["U"], b["U"])
        if hist:
            assert np.array_equal(a["J_hist"], b["J_hist"])
        if T == 1:
            o = oracle.solve(x, c0.astype(np.float64), oracle.Params(C=C, m=m, eps=0.0, max_iter=1), 0.3, 0.4,
                             U0=U0.astype(np.float64))
            assert rel(host(b["U"]), o["U"]) <= TOL and rel(b["c"], o["c"]) <= TOL
    ctx.close()
