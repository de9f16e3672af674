"""Plain FCM where a thread takes many voxels: its sums stay those of short
float32 chains.

In units of 2^-24, for m = 2: a squared distance carries 3 (difference, doubled
by the square, and the square's own), the product of C - 1 of them
4 (C - 1) - 1, their sum C - 1 more, the reciprocal 2 and its product 1; a
membership is off by at most 9 C - 8 in all, its square by twice that and 1, a
term of a sum by 4 more (J's squared distance and product).  A thread's run of
eight terms adds 7, its sum of at most eight runs 7, the tree over the wave and
its work group 9.  A centre is a ratio of two such sums, and is rounded once.
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import TOL, dev, host, random_memberships_f32, rel

pytestmark = pytest.mark.gpu


def bound(C):
    return (2 * (2 * (9 * C - 8) + 5 + 23) + 1) * 2.0 ** -24


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


# 3, 4, 5, 8 and 9 voxels per thread: remainders of the groups of four that are
# loaded together and of the runs of eight.
@pytest.mark.parametrize("shape", [(3, 512, 500), (16, 256, 256), (17, 256, 256), (8, 512, 512), (33, 256, 257)])
@pytest.mark.parametrize("C,m", [(4, 2.0), (3, 1.7)])
def test_a_step_matches_the_oracle(ctx, shape, C, m):
    raw, _ = synth.random_ellipsoids(shape=shape, seed=40 + C, sigma=0.07, count=12)
    x = oracle.normalize(raw)
    xg = dev(x)
    U0 = random_memberships_f32(np.random.default_rng(C), x.size, C)
    c0 = np.linspace(0.1, 0.9, C).astype(np.float32)
    po = oracle.Params(C=C, m=m, eps=0.0, max_iter=1)
    r = ctx.ifcm_solve(xg, _P(C=C, m=m, eps=0.0, max_iter=1), 0.0, 0.0, c0, U_in=dev(U0), want_hist=True)
    Uo, co, Jo = oracle.step(x, U0.astype(np.float64), c0.astype(np.float64), po, 0.0, 0.0)
    assert rel(host(r["U"]), Uo) <= TOL
    tol = bound(C) if m == 2.0 else TOL
    assert np.all(np.abs(r["c"] / co - 1.0) <= tol) and abs(r["J_hist"][0] / Jo - 1.0) <= tol


@pytest.mark.parametrize("how", ["solve", "adjoint"])
def test_regions_of_one_intensity(ctx, how):
    """2^30 voxels of three intensities: equal terms, whose roundings all go the
    same way."""
    import torch
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 100 GB of free device memory")
    nz, plane, C = 1024, 1024 * 1024, 2
    vals, ends = np.array([0.03, 0.41, 0.77], np.float32), [614, 870, nz]
    x = torch.empty((nz, 1024, 1024), device="cuda")
    n, lo = np.zeros(3), 0
    for k, hi in enumerate(ends):
        x[lo:hi] = float(vals[k])
        n[k], lo = (hi - lo) * plane, hi
    c0 = np.array([0.2, 0.6], np.float32)
    v = vals.astype(np.float64)[:, None]

    def u_of(c):
        w = 1.0 / (v - c.astype(np.float64)) ** 2
        return w / w.sum(1, keepdims=True)

    w = n[:, None] * u_of(c0) ** 2
    c1 = (w * v).sum(0) / w.sum(0)
    if how == "solve":
        r = ctx.ifcm_solve(x, _P(C=C, m=2.0, eps=0.0, max_iter=1), 0.0, 0.0, c0, want_hist=True)
        assert np.all(np.abs(r["c"] / c1 - 1.0) <= bound(C))
        J0 = (w * (v - c0.astype(np.float64)) ** 2).sum()
        assert abs(r["J_hist"][0] / J0 - 1.0) <= bound(C)
        c, J = r["c"], r["J"]
    else:
        U0 = torch.empty((nz, plane, C), device="cuda")
        lo = 0
        for k, hi in enumerate(ends):
            U0[lo:hi] = torch.tensor([0.25, 0.75], device="cuda")
            lo = hi
        r = ctx.ifcm_backward(x, _P(C=C, m=2.0, eps=0.0, max_iter=1), 0.0, 0.0, c0, U0.view(-1, C), 1, 1)
        c, J = c1.astype(np.float32), r["J"]
    J1 = (w * (v - c.astype(np.float64)) ** 2).sum()
    assert abs(J / J1 - 1.0) <= bound(C)
    del r
    torch.cuda.empty_cache()
