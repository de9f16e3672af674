"""CPU replay of the fused step's runs of planes: for every plane count, run
length, runs per tile and slab, each slot of sums receives exactly the planes
of its run, once, and no slot is left out (k_ifcm_gather's `finished`)."""
import pytest


def slots_of(nact, sc, runs, forget_tail=False):
    """{slot: [planes]} as the kernel's walk fills them (one column)."""
    sc = max(1, min(sc, nact))
    zc = min(sc * runs, (nact + sc - 1) // sc * sc)
    out = {}
    for tz in range((nact + zc - 1) // zc):
        zlo, zhi = tz * zc, min(tz * zc + zc, nact)
        run, left, acc = tz * (zc // sc), sc, []
        for z in range(zlo, zhi):
            acc.append(z)
            left -= 1
            if left > 0 and (z + 1 < zhi or forget_tail):
                continue
            assert run not in out
            out[run] = acc
            run, left, acc = run + 1, sc, []
    return sc, out


def check(nact, sc, runs, **kw):
    sc, got = slots_of(nact, sc, runs, **kw)
    want = {r: list(range(r * sc, min((r + 1) * sc, nact))) for r in range((nact + sc - 1) // sc)}
    return got == want


@pytest.mark.parametrize("runs", [1, 2, 3, 7, 200])
def test_every_plane_in_its_run(runs):
    for nact in list(range(1, 40)) + [75, 120, 181]:
        for sc in (1, 2, 3, 4, 5, 8, 11, 46, 200):
            assert check(nact, sc, runs), (nact, sc, runs)


def test_a_lost_last_run_is_caught():
    assert not check(23, 5, 2, forget_tail=True)
