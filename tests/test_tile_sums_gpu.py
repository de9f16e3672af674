"""The sums over a pair's tile slots (centres and objective).

Pairs of at most 256 slots may be added by 256 threads, others by 1024; both
add in the same order, so a pair's results do not depend on which one its
launch takes.
"""
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


def _volume(ctx, shape, seed, C):
    raw, _ = synth.random_ellipsoids(shape=shape, seed=seed, sigma=0.07, count=12)
    x = oracle.normalize(raw)
    c, U, _ = ctx.pifcm_fcm_init(dev(x), _P(C=C, m=2.0, eps=0.0, max_iter=6))
    return x, dev(x), c, U


# 16 x 4 columns and zc planes per tile: 16, 255 (= 3 x 17 x 5), 256, 257 and
# 2 x 1028 slots, C on both sides of a register of four sums.
@pytest.mark.parametrize("shape,zc", [((8, 32, 32), 8), ((10, 66, 40), 2), ((16, 64, 64), 4), ((257, 4, 9), 1),
                                      ((40, 211, 300), 20)])
@pytest.mark.parametrize("C", [3, 4, 7])
def test_slot_counts(ctx, shape, zc, C):
    x, xg, c0, U0 = _volume(ctx, shape, 11, C)
    other = _volume(ctx, (9, 90, 200), 12, C)  # 9 x 23 x 13 slots at one plane per tile
    p = _P(C=C, m=2.0, eps=0.0, max_iter=1)
    ctx.pifcm_set_decomposition([xg], p, 4, zc, 1)
    ctx.pifcm_set_decomposition([other[1]], p, 4, 1, 1)
    lone = ctx.ifcm_solve(xg, p, 0.3, 0.4, c0, U_in=U0, want_hist=True)
    both = ctx.swarm_evaluate([xg, other[1]], p, np.array([[0.3, 0.4]], np.float32), np.stack([c0, other[2]]),
                              [U0, other[3]])
    assert lone["J"] == both["fitness"][0, 0] and np.array_equal(lone["c"], both["centres"][0, 0])
    o = oracle.solve(x, c0.astype(np.float64), oracle.Params(C=C, m=2.0, eps=0.0, max_iter=1), 0.3, 0.4,
                     U0=host(U0).astype(np.float64))
    assert rel(lone["c"], o["c"]) <= TOL and abs(lone["J"] - o["J"]) <= TOL * abs(o["J"])
    assert rel(host(lone["U"]), o["U"]) <= TOL
