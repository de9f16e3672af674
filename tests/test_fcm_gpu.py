"""Plain FCM (lambda = xi = 0): the passes that keep no memberships between
iterations, against the oracle.

One step at a time: the oracle continues from the library's own state after
T iterations (float32 numbers are exact in its 64 bits), so x - c carries one
rounding, a membership moves by less than 1e-5, and the parity bar (1e-4)
applies.  Over several steps it would not: the float32 rounding of a centre
is amplified without bound at a voxel whose intensity meets it.
"""
import numpy as np
import pytest

import oracle
import synth
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


def _P(**kw):
    from paper_2002_01981_amd import Params
    return Params(**kw)


def _volume(ctx, shape, seed):
    raw, _ = synth.random_ellipsoids(shape=shape, seed=seed, sigma=0.07, count=12)
    x = oracle.normalize(raw)
    return x, dev(x)


# 262144 = 1024 work groups of 256 threads: one voxel per thread up to there.
@pytest.mark.parametrize("shape", [(1, 1, 3), (3, 5, 17), (1, 2, 128), (64, 64, 64), (8, 181, 182), (65, 64, 64)])
@pytest.mark.parametrize("C,m", [(2, 2.0), (3, 1.7), (4, 2.0), (7, 2.0), (16, 2.5)])
def test_every_iteration_matches_oracle(ctx, shape, C, m):
    x, xg = _volume(ctx, shape, 30 + C)
    U0 = random_memberships_f32(np.random.default_rng(C), x.size, C)
    c0 = np.linspace(0.1, 0.9, C).astype(np.float32)
    po = oracle.Params(C=C, m=m, eps=0.0, max_iter=1)

    def run(T, U):
        return ctx.ifcm_solve(xg, _P(C=C, m=m, eps=0.0, max_iter=T), 0.0, 0.0, c0,
                              U_in=None if U is None else dev(U), labels=True, want_hist=True)

    def step(r):
        return oracle.step(x, host(r["U"]).astype(np.float64), r["c"].astype(np.float64), po, 0.0, 0.0)

    for U in (U0, None):
        a = run(0, U)
        Us = U0 if U is not None else oracle.init_memberships(x, c0.astype(np.float64), po)
        assert rel(host(a["U"]), Us) <= (0.0 if U is not None else TOL)
        for T in (1, 2, 3, 5):
            b = run(T, U)
            if T <= 3:
                Uo, co, Jo = step(a)
                assert rel(host(b["U"]), Uo) <= TOL and rel(b["c"], co) <= TOL
                assert abs(b["J_hist"][T - 1] - Jo) <= TOL * abs(Jo)
            Jb = step(b)[2]
            assert b["iters"] == T and abs(b["J"] - Jb) <= TOL * abs(Jb)
            assert np.array_equal(host(b["labels"]), np.argmax(host(b["U"]), axis=1))
            a = b


@pytest.mark.parametrize("C,m", [(4, 2.0), (5, 2.0), (3, 2.5)])
def test_stop_rule_and_history_change_nothing_else(ctx, C, m):
    """The runs that form J of every iteration and those that do not agree bit
    for bit; the stop rule ends where the oracle's does."""
    x, xg = _volume(ctx, (9, 40, 70), 7)
    c0 = np.linspace(0.1, 0.9, C).astype(np.float32)
    o = oracle.solve(x, c0.astype(np.float64), oracle.Params(C=C, m=m, eps=1e-3, max_iter=40), 0.0, 0.0)
    a = ctx.ifcm_solve(xg, _P(C=C, m=m, eps=1e-3, max_iter=40), 0.0, 0.0, c0)
    assert a["iters"] == o["iters"] < 40
    for hist in (False, True):
        b = ctx.ifcm_solve(xg, _P(C=C, m=m, eps=0.0, max_iter=a["iters"]), 0.0, 0.0, c0, want_hist=hist)
        assert np.array_equal(host(a["U"]), host(b["U"])) and np.array_equal(a["c"], b["c"]) and a["J"] == b["J"]


def test_swarm_slab_and_scratch_agree(ctx):
    """Zero weights in every mode: batched, one launch per particle, a lone
    solve, the no-allocation solve, a carried state, and a slab."""
    from paper_2002_01981_amd import PIFCM_SWARM_BATCHED, PIFCM_SWARM_PLAIN
    C, T = 4, 6
    vols = [_volume(ctx, s, 50 + i) for i, s in enumerate(((6, 33, 47), (11, 20, 64)))]
    U0 = [random_memberships_f32(np.random.default_rng(i), x.size, C) for i, (x, _) in enumerate(vols)]
    Ug = [dev(u) for u in U0]
    c0 = np.tile(np.linspace(0.1, 0.9, C).astype(np.float32), (2, 1))
    xs = [g for _, g in vols]
    p = _P(C=C, m=2.0, eps=0.0, max_iter=T)
    zero = np.zeros((2, 3, 2), np.float32)
    a = ctx.swarm_evaluate(xs, p, zero, c0, Ug, mode=PIFCM_SWARM_BATCHED)
    b = ctx.swarm_evaluate(xs, p, zero, c0, Ug, mode=PIFCM_SWARM_PLAIN)
    assert np.array_equal(a["fitness"], b["fitness"]) and np.array_equal(a["centres"], b["centres"])
    st = {k: np.zeros(s) for k, s in (("x0", (3, 2)), ("v0", (3, 2)), ("r1", (2, 3, 2)), ("r2", (2, 3, 2)))}
    car = ctx.pifcm_pso_interleaved(xs, p, st, c0, Ug, steps=T // 2)
    for i in range(2):
        s = ctx.ifcm_solve(xs[i], p, 0.0, 0.0, c0[i], U_in=Ug[i], labels=True)
        n = ctx.ifcm_solve_noalloc(xs[i], p, 0.0, 0.0, c0[i], U_in=Ug[i], labels=True)
        assert s["J"] == a["fitness"][i, 1] and np.array_equal(s["c"], a["centres"][i, 2])
        assert s["J"] == n["J"] and np.array_equal(host(s["U"]), host(n["U"]))
        assert np.array_equal(host(s["U"]), host(car["U_best"][i])) and np.array_equal(s["c"], car["centres_best"][i])
        assert car["fit_hist"][i, 1, 0] == s["J"]
        z0, z1 = 2, 5
        sl = ctx.ifcm_solve_slab(xs[i], z0, z1, _P(C=C, m=2.0, eps=0.0, max_iter=1), 0.0, 0.0, c0[i], Ug[i])
        po = oracle.Params(C=C, m=2.0, eps=0.0, max_iter=1)
        o = oracle.solve_slab(vols[i][0], c0[i].astype(np.float64), po, 0.0, 0.0, U0[i].astype(np.float64), z0, z1)
        assert rel(host(sl["U"]), o["U"]) <= TOL and rel(sl["c"], o["c"]) <= TOL
        k = int(np.prod(vols[i][0].shape[1:]))
        assert np.array_equal(host(sl["U"])[: z0 * k], U0[i][: z0 * k])
        assert np.array_equal(host(sl["U"])[z1 * k:], U0[i][z1 * k:])


@pytest.mark.parametrize("C", [2, 4, 9])
def test_start_is_sorted(ctx, C):
    """The columns of the FCM start follow its ascending centres."""
    x, xg = _volume(ctx, (7, 30, 41), 90 + C)
    c, U, it = ctx.pifcm_fcm_init(xg, _P(C=C, m=2.0, eps=0.0, max_iter=12))
    co, Uo, ito = oracle.fcm_init(x, oracle.Params(C=C, m=2.0, eps=0.0, max_iter=12))
    assert it == ito and np.all(np.diff(c) >= 0) and rel(c, co) <= TOL and rel(host(U), Uo) <= TOL
