"""A context allocates a table when a call needs it: a fresh one holds a few
kilobytes, and the adjoint, as the first call, finds its own."""
import numpy as np
import pytest

from gpu_util import dev, random_memberships_f32

pytestmark = pytest.mark.gpu


def test_a_fresh_context_is_small_and_serves_the_adjoint():
    from paper_2002_01981_amd import Context, Params
    rng = np.random.default_rng(2)
    x, C, K = rng.random((5, 9, 20)).astype(np.float32), 3, 4
    U0, c0 = random_memberships_f32(rng, x.size, C), np.array([0.2, 0.5, 0.8], np.float32)
    ctx = Context(0)
    assert ctx.workspace_bytes() <= 64 << 10
    r = ctx.ifcm_backward(dev(x), Params(C=C, m=2.0, eps=0.0, max_iter=K), 0.3, 0.2, c0, dev(U0), K, 2)
    s = ctx.ifcm_solve(dev(x), Params(C=C, m=2.0, eps=0.0, max_iter=K), 0.3, 0.2, c0, U_in=dev(U0))
    assert abs(r["J"] - s["J"]) <= 1e-5 * abs(s["J"])
    assert np.isfinite([r["dlam"], r["dxi"], *r["dc"]]).all()
    ctx.close()
