"""The two-ring kernels (V = 2, C <= 4) where their tiles end: the step's tiles
of 16 x 4 columns with a halo of two, the invariants' tiles of 60 x 2 columns
and runs of planes, volumes smaller than the neighbourhood, flat rings, both
eq (7) weightings; and tile depth by launch for every general neighbourhood.

Bounds: TOL of gpu_util against the FP64 oracle after one iteration from given
float32 memberships and centres (the bound of test_ring_gpu.py).  Sums are kept
per run of a volume's default planes, so a swarm has the bits of lone solves.
"""
import numpy as np
import pytest

import oracle
from gpu_util import TOL, dev, host, random_memberships_f32, rel

pytestmark = pytest.mark.gpu

Q2 = 2


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "the GPU tests need a GPU"
    from paper_2002_01981_amd import Context
    c = Context(0)
    yield c
    c.close()


def _volume(shape, seed, flat):
    rng = np.random.default_rng(seed)
    x = rng.random(shape, dtype=np.float32)
    if flat:  # rings of equal intensity, with and without the voxel itself
        z, y, w = (s // 2 for s in shape)
        x[:, : y + 1, : w + 1] = 0.25
        x[z, y // 2, w // 2] = 0.75
    return x


@pytest.mark.parametrize("shape,C,m,flags,flat", [
    ((1, 1, 2), 2, 2.0, 0, False),
    ((2, 3, 2), 4, 2.0, Q2, False),
    ((5, 2, 59), 4, 2.0, 0, False),
    ((4, 3, 60), 4, 2.0, Q2, False),
    ((3, 4, 61), 3, 2.0, 0, False),
    ((7, 5, 62), 4, 2.5, 0, False),
    ((6, 4, 16), 4, 2.0, 0, True),
    ((5, 9, 17), 2, 2.0, Q2, True),
    ((33, 5, 18), 4, 2.0, 0, False),
    ((67, 6, 15), 3, 2.5, Q2, True),
])
def test_steps_at_tile_edges(ctx, shape, C, m, flags, flat):
    from paper_2002_01981_amd import Params
    lam, xi, steps = 0.35, 0.4, 1
    x = _volume(shape, 71, flat)
    U0 = random_memberships_f32(np.random.default_rng(72), x.size, C)
    c0 = np.linspace(0.15, 0.85, C).astype(np.float32)
    g = ctx.ifcm_solve(dev(x), Params(C=C, m=m, V=2, eps=0.0, max_iter=steps, flags=flags), lam, xi,
                       c0, U_in=dev(U0), want_hist=True)
    o = oracle.solve(x, c0.astype(np.float64),
                     oracle.Params(C=C, m=m, V=2, eps=0.0, max_iter=steps, flags=flags),
                     lam, xi, U0=U0.astype(np.float64), want_hist=True)
    assert rel(host(g["U"]), o["U"]) <= TOL
    assert rel(g["c"], o["c"]) <= TOL
    assert abs(g["J"] - o["J"]) <= TOL * abs(o["J"])
    assert rel(g["J_hist"], o["J_hist"]) <= TOL


# One plane; a last run shorter than the others; tiles of several runs beside
# volumes of one tile.
@pytest.mark.parametrize("shapes,P", [([(1, 9, 20)], 300), ([(23, 17, 66), (8, 32, 32), (7, 5, 18)], 70),
                                      ([(37, 60, 90)], 24)])
@pytest.mark.parametrize("C,V,flags", [(4, 2, 0), (3, 2, Q2), (5, 2, 0), (4, 3, 1)])
def test_swarm_equals_lone_solves(ctx, shapes, P, C, V, flags):
    from paper_2002_01981_amd import Params
    rng = np.random.default_rng(73)
    xs = [dev(_volume(sh, 74 + i, False)) for i, sh in enumerate(shapes)]
    U0 = [dev(random_memberships_f32(rng, int(np.prod(sh)), C)) for sh in shapes]
    c0 = np.stack([np.linspace(0.15, 0.85, C).astype(np.float32)] * len(shapes))
    parts = (rng.random((P, 2)) * 0.5).astype(np.float32)
    p = Params(C=C, V=V, eps=0.0, max_iter=2, flags=flags)
    bat = ctx.swarm_evaluate(xs, p, parts, c0, U0)
    for b in range(len(shapes)):
        for q in (0, P // 2, P - 1):
            s = ctx.ifcm_solve(xs[b], p, float(parts[q][0]), float(parts[q][1]), c0[b], U_in=U0[b])
            assert s["J"] == bat["fitness"][b, q] and np.array_equal(s["c"], bat["centres"][b, q])
