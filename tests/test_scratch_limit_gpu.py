"""ifcm_solve_noalloc just below the size of its scratch array: a volume whose
default tiles would leave sums for a little more than the array is solved on
deeper tiles instead of being refused.

A voxel's update does not depend on its tile, so the memberships of one
iteration have the bits of ifcm_solve; the centres and J are float32 sums of
the same terms in another order (bound 1e-5: 2^-24 times the square root of the
some thousand terms a lane and its wave add, with room to spare).
"""
import numpy as np
import pytest

from gpu_util import rel

pytestmark = pytest.mark.gpu


def test_a_solve_at_the_limit_of_the_scratch():
    import torch
    from paper_2002_01981_amd import Context, Params
    ctx = Context(0)
    shape, C = (39, 4586, 22), 16
    x = torch.rand(shape, generator=torch.Generator().manual_seed(91)).cuda()
    c0 = np.linspace(0.05, 0.95, C).astype(np.float32)
    p = Params(C=C, m=2.0, eps=0.0, max_iter=1)
    a = ctx.ifcm_solve_noalloc(x, p, 0.3, 0.4, c0)
    b = ctx.ifcm_solve(x, p, 0.3, 0.4, c0)
    assert torch.equal(a["U"], b["U"])
    assert rel(a["c"], b["c"]) <= 1e-5 and abs(a["J"] - b["J"]) <= 1e-5 * abs(b["J"])
    ctx.close()
