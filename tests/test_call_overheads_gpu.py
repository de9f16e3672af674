"""Calls that check their inputs while they run: refusals, and the calls after
them, are what they would be with a check up front."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import dev, host, random_memberships_f32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "the GPU tests need a GPU"
    from paper_2002_01981_amd import Context
    c = Context(0)
    yield c
    c.close()


def _inputs(shape=(6, 9, 20), C=4):
    rng = np.random.default_rng(3)
    x = rng.random(shape).astype(np.float32)
    return x, random_memberships_f32(rng, x.size, C), np.linspace(0.1, 0.9, C).astype(np.float32)


@pytest.mark.parametrize("eps", [0.0, 1e-5])
@pytest.mark.parametrize("max_iter", [0, 3, 60_000])  # short runs wait once at the end, long ones early
def test_refused_input_then_good_input(ctx, eps, max_iter):
    from paper_2002_01981_amd import Params, PifcmError
    from paper_2002_01981_amd.abi import PIFCM_E_INVALID, PIFCM_E_NONFINITE
    x, U0, c0 = _inputs()
    bx, bu = x.copy(), U0.copy()
    bx[5, 8, 19], bu[7, 2] = np.inf, -0.25
    p, good = Params(C=4, m=2.0, eps=eps, max_iter=max_iter), Params(C=4, m=2.0, eps=0.0, max_iter=3)
    part = np.array([[0.3, 0.4], [0.2, 0.1]], np.float32)
    ref = ctx.ifcm_solve(dev(x), good, 0.3, 0.4, c0, U_in=dev(U0), want_hist=True)
    for name in ("ifcm_solve", "ifcm_solve_noalloc", "swarm", "plain"):
        for a, b, status in ((bx, U0, PIFCM_E_NONFINITE), (x, bu, PIFCM_E_INVALID), (bx, bu, PIFCM_E_NONFINITE)):
            with pytest.raises(PifcmError) as e:
                if name in ("swarm", "plain"):
                    ctx.swarm_evaluate([dev(x), dev(a)], p, part, np.stack([c0, c0]), [dev(U0), dev(b)],
                                       mode=int(name == "plain"))
                else:
                    getattr(ctx, name)(dev(a), p, 0.3, 0.4, c0, U_in=dev(b), want_hist=True, labels=True)
            assert e.value.status == status
        if name == "plain" or name == "swarm":
            r = ctx.swarm_evaluate([dev(x)], good, part, c0[None], [dev(U0)], mode=int(name == "plain"))
            assert r["fitness"][0, 0] == ref["J"] and np.array_equal(r["centres"][0, 0], ref["c"])
        else:
            r = getattr(ctx, name)(dev(x), good, 0.3, 0.4, c0, U_in=dev(U0), want_hist=True, labels=True)
            assert np.array_equal(host(r["U"]), host(ref["U"])) and np.array_equal(r["J_hist"], ref["J_hist"])
            assert np.array_equal(host(r["labels"]), np.argmax(host(r["U"]), axis=1))


def test_normalisations_in_turn(ctx):
    """Calls with different ranges, refusals between them, and outputs left
    alone by a refusal (in place too)."""
    import torch
    from paper_2002_01981_amd import PifcmError
    rng = np.random.default_rng(8)
    for k in range(12):
        raw = (rng.random((3, 5, 7)) * 10.0 ** (k % 5) - 3.0 * k).astype(np.float32)
        if k % 3 == 2:
            bad = raw.copy()
            bad[2, 4, 6] = (np.nan, np.inf, -np.inf)[k % 3 - 1]
            out = torch.full((3, 5, 7), 4.0, device="cuda")
            t = dev(bad)
            for o in (out, t):
                with pytest.raises(PifcmError):
                    ctx.pifcm_normalize(t, out=o)
            assert torch.all(out == 4.0) and np.array_equal(host(t), bad, equal_nan=True)
        assert np.array_equal(host(ctx.pifcm_normalize(dev(raw))), oracle.normalize(raw))


def test_outputs_are_ready_for_the_callers_stream(ctx):
    """Work the caller queues on its own stream right after a call reads what
    the call wrote."""
    import torch
    from paper_2002_01981_amd import Context, Params
    raw, _ = synth.random_ellipsoids(shape=(20, 60, 70), seed=4, sigma=0.07)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        c = Context(0)
        try:
            sums = []
            for _ in range(3):
                x = c.pifcm_normalize(torch.from_numpy(raw).cuda())
                copy = x.clone()
                c0, U0, _ = c.pifcm_fcm_init(x, Params(C=4, m=2.0, eps=0.0, max_iter=3))
                r = c.ifcm_solve(x, Params(C=4, m=2.0, eps=0.0, max_iter=3), 0.3, 0.4, c0, U_in=U0, labels=True)
                sums.append((copy.double().sum().item(), r["U"].double().sum().item(), r["labels"].long().sum().item()))
            assert len(set(sums)) == 1
            assert abs(sums[0][0] - oracle.normalize(raw).astype(np.float64).sum()) < 1e-6
        finally:
            c.close()
