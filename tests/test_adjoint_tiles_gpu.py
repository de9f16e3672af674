"""The transpose of the adjoint at the edges of its tiles.

A tile whose cells and halo all lie off the x and y faces takes one eq (7)
normalisation for its planes off the z faces and a formed one elsewhere.  With
tiles of 16 x 4 columns the tile at (16, 4) is the first that can: it does from
34 x 10 columns on.  The sizes here are one below, at and above that line, with
one to four planes (no plane, and some planes, off the z faces), and volumes
deeper than one tile of the forward pass.

Bounds: the gradient against central differences of the FP64 oracle to 1e-3 of
its largest component (the bound of test_adjoint_gpu.py: the step of 1e-4 and
float32 passes); a wrong normalisation in one column of 34 moves it by about a
percent.
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "the GPU tests need a GPU"
    from paper_2002_01981_amd import Context
    c = Context(0)
    yield c
    c.close()


def _case(shape, C, m, seed):
    raw, _ = synth.random_ellipsoids(shape=shape, seed=seed, sigma=0.07)
    x = oracle.normalize(raw)
    c0, U0, _ = oracle.fcm_init(x, oracle.Params(C=C, m=m, eps=0.0, max_iter=8))
    return x, c0.astype(np.float32), U0.astype(np.float32)


@pytest.mark.parametrize("shape,C,m,sq", [
    ((4, 9, 34), 4, 2.0, False),
    ((4, 10, 33), 4, 2.0, False),
    ((4, 10, 34), 4, 2.0, False),
    ((3, 10, 34), 3, 2.5, True),
    ((2, 11, 35), 4, 2.0, False),
    ((1, 10, 34), 4, 2.0, False),
    ((4, 14, 50), 5, 2.0, True),
])
def test_gradient_at_the_edges_of_inner_tiles(ctx, shape, C, m, sq):
    from paper_2002_01981_amd import PIFCM_Q2_SQDIST, Params
    flags = PIFCM_Q2_SQDIST if sq else 0
    lam, xi, K = 0.15, 0.55, 3
    x, c0, U0 = _case(shape, C, m, seed=61)
    g = ctx.ifcm_backward(dev(x), Params(C=C, m=m, flags=flags), lam, xi, c0, dev(U0), K, 2)
    Jo, go = oracle.fd_grad(x, c0.astype(np.float64), U0.astype(np.float64),
                            oracle.Params(C=C, m=m, flags=flags), lam, xi, K=K, step=1e-4)
    gg = np.concatenate([[g["dlam"], g["dxi"]], g["dc"]])
    assert abs(g["J"] - Jo) <= 1e-4 * abs(Jo)
    assert np.max(np.abs(gg - go)) / np.max(np.abs(go)) <= 1e-3, (gg, go)


@pytest.mark.parametrize("shape", [(33, 6, 18), (70, 5, 17)])
def test_recomputed_steps_at_another_tile_depth_give_the_same_gradient(ctx, shape):
    """Strides above 1 recompute states at the depth of a lone solve, stride 1
    reads the forward pass's own: a voxel's update does not depend on the tile
    that holds it, so the gradients agree bit for bit."""
    from paper_2002_01981_amd import Params
    x, c0, U0 = _case(shape, 4, 2.0, seed=62)
    ref = ctx.ifcm_backward(dev(x), Params(C=4, m=2.0), 0.3, 0.2, c0, dev(U0), 10, 1)
    for s in (3, 4):
        g = ctx.ifcm_backward(dev(x), Params(C=4, m=2.0), 0.3, 0.2, c0, dev(U0), 10, s)
        assert g["J"] == ref["J"] and g["dlam"] == ref["dlam"] and g["dxi"] == ref["dxi"]
        assert np.array_equal(g["dc"], ref["dc"])
