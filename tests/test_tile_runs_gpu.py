"""Tile depth by launch: sums are kept per run of a volume's default planes, so
a batched launch whose tiles hold several runs, and launches of other depths,
give the bits of a lone solve.  The lone solve is held to the oracle."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import TOL, dev, host, rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "the GPU tests need a GPU"
    from paper_2002_01981_amd import Context
    c = Context(0)
    yield c
    c.close()


def _P(**kw):
    from paper_2002_01981_amd import Params
    return Params(**kw)


# One plane; fewer, as many and more planes than a group of three; a last run
# shorter than the others; a volume of many columns beside small ones.
@pytest.mark.parametrize("shapes,P", [([(1, 9, 20)], 700), ([(2, 33, 47), (3, 20, 70)], 300), ([(4, 64, 64)], 120),
                                      ([(23, 17, 66), (8, 32, 32), (7, 5, 18)], 200), ([(37, 130, 190)], 24)])
@pytest.mark.parametrize("C,m", [(4, 2.0), (3, 1.7)])
def test_batched_launch_equals_lone_solves(ctx, shapes, P, C, m):
    xs, c0, U0, xo = [], [], [], []
    for i, sh in enumerate(shapes):
        raw, _ = synth.random_ellipsoids(shape=sh, seed=700 + i, sigma=0.07, count=12)
        xo.append(oracle.normalize(raw))
        xs.append(dev(xo[-1]))
        c, U, _ = ctx.pifcm_fcm_init(xs[-1], _P(C=C, m=m, eps=0.0, max_iter=4))
        c0.append(c)
        U0.append(U)
    parts = synth.uniform_particles(33, P) * np.float32(0.5)
    p = _P(C=C, m=m, eps=0.0, max_iter=2)
    bat = ctx.swarm_evaluate(xs, p, parts, np.stack(c0), U0)
    for b in range(len(shapes)):
        for q in (0, P // 2, P - 1):
            lam, xi = (float(v) for v in parts[q])
            s = ctx.ifcm_solve(xs[b], p, lam, xi, c0[b], U_in=U0[b])
            assert s["J"] == bat["fitness"][b, q] and np.array_equal(s["c"], bat["centres"][b, q])
        one = ctx.ifcm_solve(xs[b], _P(C=C, m=m, eps=0.0, max_iter=1), lam, xi, c0[b], U_in=U0[b])
        o = oracle.solve(xo[b], c0[b].astype(np.float64), oracle.Params(C=C, m=m, eps=0.0, max_iter=1), lam, xi,
                         U0=host(U0[b]).astype(np.float64))
        assert rel(host(one["U"]), o["U"]) <= TOL and rel(one["c"], o["c"]) <= TOL
