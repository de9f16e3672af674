"""A volume of more than 2^31 voxels (69 GB at C = 2): counts and offsets that
do not fit 32 bits.

Its planes repeat with a period of seven, so the memberships of one iteration
must have the bits of those of a small volume of the same planes (a voxel's
update depends on its neighbours and not on its tile); the small volumes'
sizes are held to the oracle elsewhere.  The centres are held to float64 sums
over the memberships returned: a lane adds the planes of its tile in float32
before the float64 sums, at most DEEPEST of them (a tile's 32-bit byte offsets
reach that far), so numerator and denominator move by at most DEEPEST * 2^-24
each, and the wave's sum over 64 lanes by 6 * 2^-24 more.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPE, C, PERIOD = (2049, 1024, 1024), 2, 7
DEEPEST = 2 ** 31 // (SHAPE[1] * SHAPE[2] * C * 4) - 3


@pytest.fixture(scope="module")
def huge():
    import torch
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 100 GB of free device memory")
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.rand((PERIOD, *SHAPE[1:]), generator=g, device="cuda")
    u = torch.rand((PERIOD, SHAPE[1] * SHAPE[2], 1), generator=g, device="cuda") * 0.98 + 0.01
    U = torch.cat([u, 1.0 - u], 2)
    n = SHAPE[0] // PERIOD + 1
    yield x, U, x.repeat(n, 1, 1)[: SHAPE[0]], U.repeat(n, 1, 1)[: SHAPE[0]].view(-1, C)
    torch.cuda.empty_cache()


def _centres(x, U, m=2.0):
    """eq (3) in float64, plane by plane."""
    import torch
    num, den = torch.zeros(C, dtype=torch.float64, device="cuda"), torch.zeros(C, dtype=torch.float64, device="cuda")
    for xp, up in zip(x, U.view(x.shape[0], -1, C)):
        w = up.double() ** m
        num += (w * xp.reshape(-1, 1).double()).sum(0)
        den += w.sum(0)
    return (num / den).cpu().numpy()


def test_one_iteration(huge):
    import torch
    from paper_2002_01981_amd import Context, Params
    x7, U7, x, U0 = huge
    c0, p = np.array([0.3, 0.7], np.float32), Params(C=C, m=2.0, eps=0.0, max_iter=1)
    ctx = Context(0)
    r = ctx.ifcm_solve(x, p, 0.3, 0.4, c0, U_in=U0)
    U = r["U"].view(SHAPE[0], -1, C)
    for first in (0, SHAPE[0] - 14):
        idx = torch.arange(first, first + 14, device="cuda") % PERIOD
        s = ctx.ifcm_solve(x7[idx].contiguous(), p, 0.3, 0.4, c0, U_in=U7[idx].reshape(-1, C).contiguous())
        lo, hi = (0, 13) if first == 0 else (1, 14)  # the other end has a cut neighbourhood
        assert torch.equal(U[first + lo:first + hi], s["U"].view(14, -1, C)[lo:hi])
    assert np.all(np.abs(r["c"] / _centres(x, r["U"]) - 1.0) <= 2 * (DEEPEST + 6) * 2.0 ** -24)
    ctx.close()
