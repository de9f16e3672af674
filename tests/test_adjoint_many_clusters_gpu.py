"""The adjoint on both sides of C = 12, from where on a voxel's centre value is
read back from LDS, with a block of one intensity (whose centre value is
shifted).  Gradient against central differences of the FP64 oracle, 1e-3 of its
largest component: the bound of test_adjoint_gpu.py."""
import numpy as np
import pytest

import oracle
from gpu_util import dev, random_memberships_f32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,m", [(11, 2.0), (12, 2.0), (12, 2.5), (13, 2.0), (16, 2.0)])
def test_gradient(C, m):
    from paper_2002_01981_amd import Context, Params
    rng = np.random.default_rng(C)
    x = rng.random((5, 9, 37)).astype(np.float32)
    x[1:4, 2:7, 6:20] = 0.4
    U0, c0 = random_memberships_f32(rng, x.size, C), np.linspace(0.05, 0.95, C).astype(np.float32)
    ctx = Context(0)
    g = ctx.ifcm_backward(dev(x), Params(C=C, m=m), 0.2, 0.3, c0, dev(U0), 2, 1)
    Jo, go = oracle.fd_grad(x, c0.astype(np.float64), U0.astype(np.float64), oracle.Params(C=C, m=m), 0.2, 0.3, K=2,
                            step=1e-4)
    gg = np.concatenate([[g["dlam"], g["dxi"]], g["dc"]])
    assert abs(g["J"] - Jo) <= 1e-4 * abs(Jo)
    assert np.max(np.abs(gg - go)) / np.max(np.abs(go)) <= 1e-3, (gg, go)
    ctx.close()
