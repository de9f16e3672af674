"""An iteration forms J of its input state only under a stop rule or for a
history; a run without either has the same memberships, centres and final
objective bit for bit."""
import numpy as np
import pytest

import synth
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "the GPU tests need a GPU"
    from paper_2002_01981_amd import Context
    c = Context(0)
    yield c
    c.close()


# One voxel, one column, one plane, and tiles with ragged ends.
@pytest.mark.parametrize("shape", [(1, 1, 1), (5, 1, 1), (1, 6, 19), (13, 37, 29)])
@pytest.mark.parametrize("C,m", [(2, 2.0), (3, 2.5), (4, 2.0), (8, 2.0), (13, 1.6)])
def test_history_changes_nothing(ctx, shape, C, m):
    from paper_2002_01981_amd import Params
    raw, _ = synth.random_ellipsoids(shape=shape, seed=5, sigma=0.07, count=9)
    x = ctx.pifcm_normalize(dev(raw))
    c0 = np.linspace(0.1, 0.9, C).astype(np.float32)
    p = Params(C=C, m=m, eps=0.0, max_iter=4)
    a = ctx.ifcm_solve(x, p, 0.3, 0.4, c0, want_hist=True)
    b = ctx.ifcm_solve(x, p, 0.3, 0.4, c0, want_hist=False)
    # a threshold that no relative change reaches, on the path with a stop rule
    s = ctx.ifcm_solve(x, Params(C=C, m=m, eps=1e-30, max_iter=4), 0.3, 0.4, c0)
    for o in (b,) + ((s,) if s["iters"] == 4 else ()):
        assert np.array_equal(host(a["U"]), host(o["U"])) and np.array_equal(a["c"], o["c"]) and a["J"] == o["J"]
    sw = ctx.swarm_evaluate([x], p, np.array([[0.3, 0.4], [0.1, 0.2], [0.3, 0.4]], np.float32), c0[None], [_u0(ctx, x, c0, C, m)])
    assert sw["fitness"][0, 0] == sw["fitness"][0, 2] == a["J"]


def _u0(ctx, x, c0, C, m):
    from paper_2002_01981_amd import Params
    return ctx.ifcm_solve(x, Params(C=C, m=m, eps=0.0, max_iter=0), 0.3, 0.4, c0)["U"]
