"""The single-slice mode's one pass over the context: every output row and
label, and every refusal, wherever the slab lies in the volume and however far
the neighbourhood reaches beyond it.

One step from a float32 state at lambda + xi = 0.7: the parity bar (a factor
of eq (4) is at least 0.3, rounding moves a membership by less than 1e-5).
"""
import numpy as np
import pytest

import oracle
from gpu_util import TOL, dev, host, random_memberships_f32, rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "the GPU tests need a GPU"
    from paper_2002_01981_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("shape,slab", [((1, 9, 17), (0, 1)), ((9, 13, 37), (0, 1)), ((9, 13, 37), (8, 9)),
                                        ((9, 13, 37), (4, 5)), ((9, 13, 37), (1, 8)), ((40, 6, 70), (17, 37))])
@pytest.mark.parametrize("C,V,flags", [(4, 1, 0), (3, 1, 0), (5, 2, 0), (4, 2, 0), (4, 3, 0), (4, 4, 1)])
def test_rows_and_labels(ctx, shape, slab, C, V, flags):
    from paper_2002_01981_amd import Params
    rng = np.random.default_rng(sum(shape) + C + V)
    x = rng.random(shape).astype(np.float32)
    U0 = random_memberships_f32(rng, x.size, C)
    c0 = np.linspace(0.1, 0.9, C).astype(np.float32)
    k = shape[1] * shape[2]
    # The state is in either iteration buffer, or still the caller's.
    for T in (0, 1, 2, 3):
        p = Params(C=C, m=2.0, V=V, eps=0.0, max_iter=T, flags=flags)
        g = ctx.ifcm_solve_slab(dev(x), *slab, p, 0.4, 0.3, c0, dev(U0), labels=True)
        U = host(g["U"])
        assert np.array_equal(U[: slab[0] * k], U0[: slab[0] * k])
        assert np.array_equal(U[slab[1] * k:], U0[slab[1] * k:])
        assert np.array_equal(host(g["labels"]), np.argmax(U, axis=1))
        if T == 0:
            assert np.array_equal(U, U0)
        else:  # one oracle step from the library's own state before it
            o = oracle.solve_slab(x, prev[1], oracle.Params(C=C, m=2.0, V=V, eps=0.0, max_iter=1, flags=flags), 0.4,
                                  0.3, prev[0], *slab)
            assert rel(U, o["U"]) <= TOL and rel(g["c"], o["c"]) <= TOL
        prev = (U.astype(np.float64), g["c"].astype(np.float64))


@pytest.mark.parametrize("lam,xi", [(0.3, 0.2), (0.0, 0.0)])
def test_refused_outside_the_slab_too(ctx, lam, xi):
    from paper_2002_01981_amd import Params, PifcmError
    from paper_2002_01981_amd.abi import PIFCM_E_INVALID, PIFCM_E_NONFINITE
    rng = np.random.default_rng(1)
    shape, C = (7, 8, 20), 4
    x = rng.random(shape).astype(np.float32)
    U0 = random_memberships_f32(rng, x.size, C)
    c0 = np.linspace(0.1, 0.9, C).astype(np.float32)
    p = Params(C=C, m=2.0, eps=0.0, max_iter=2)
    for z in (0, 3, 6):
        bx, bu = x.copy(), U0.copy()
        bx[z, 7, 19] = np.nan
        bu[z * 160 + 159, 3] = 1.5
        for a, b, status in ((bx, U0, PIFCM_E_NONFINITE), (x, bu, PIFCM_E_INVALID)):
            with pytest.raises(PifcmError) as e:
                ctx.ifcm_solve_slab(dev(a), 3, 4, p, lam, xi, c0, dev(b))
            assert e.value.status == status
    ctx.ifcm_solve_slab(dev(x), 3, 4, p, lam, xi, c0, dev(U0))
