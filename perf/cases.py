"""Timed cases of the library: what a program that segments volumes has it do.

Each case goes through the public entry points of paper_2002_01981_amd.Context
the way pipeline.py, quality.py and bench.py call them: normalisation, the FCM
start, IFCM solves, swarm evaluations, the single-slice mode and the adjoint.
Sizes are those of the repository's workloads (synth/phantoms.py) and tests.

A case is a dict of plain values:
  kind     entry point: normalize, fcm, solve, swarm, slab, adjoint
  volumes  "ZxYxX" shapes, blank-separated (one, but for swarm)
  C, m, V, sq   clusters, fuzziness, rings, rings by squared distance
  iters, eps    iteration cap and stop rule (eps 0: exactly iters)
  P, plain      particles per volume; one launch per particle instead of batched
  labels        the segmentation is asked for too

Particles are drawn with lambda + xi <= 0.95, where the attraction factor of
the distance stays positive: beyond it the iteration amplifies rounding
without bound and no two summation orders agree.
"""
import math

import numpy as np
import torch

from paper_2002_01981_amd import PIFCM_SHELL_SQDIST, PIFCM_SWARM_BATCHED, PIFCM_SWARM_PLAIN, Context, Params

BRAIN = "181x217x181"
RAGGED = "104x251x204 116x79x246 101x151x234 75x181x162 107x118x245 120x136x252"
CKPT = 5  # iterations between the adjoint's checkpoints


def _case(kind, volumes, C=4, m=2.0, V=1, sq=False, iters=20, eps=0.0, P=0, plain=False, labels=False):
    return dict(kind=kind, volumes=volumes, C=C, m=m, V=V, sq=sq, iters=iters, eps=eps, P=P, plain=plain,
                labels=labels)


def listed():
    return [
        # Every volume enters through the min-max normalisation.
        dict(_case("normalize", BRAIN), name="normalize-brain"),
        # The FCM start of a search, with its stop rule.
        dict(_case("fcm", BRAIN, iters=50, eps=1e-5), name="fcm-brain"),
        # The smallest volume of the paper's size series: launches and latency count.
        dict(_case("solve", "8x32x32", iters=50, labels=True), name="solve-32x32x8"),
        # The final solve of a search on the brain-sized volume.
        dict(_case("solve", BRAIN, iters=30), name="solve-brain"),
        # Three classes and a general fuzziness on an odd-sized volume.
        dict(_case("solve", "75x181x162", C=3, m=2.5), name="solve-162x181x75-c3-m2.5"),
        # More classes than one row of four.
        dict(_case("solve", "120x136x252", C=8, iters=10), name="solve-252x136x120-c8"),
        # One generation over a ragged batch: the benchmark's volumes and swarm.
        dict(_case("swarm", RAGGED, iters=4, P=64), name="swarm-ragged6"),
        # One generation of the search on the smallest volume, with its stop rule.
        dict(_case("swarm", "8x32x32", iters=50, eps=1e-5, P=8), name="swarm-32x32x8"),
        # The largest image of the paper's size series, one launch per particle.
        dict(_case("swarm", "16x854x854", iters=10, P=4, plain=True), name="swarm-854x854x16-plain"),
        # One slice of a volume with its 3D neighbours, the unit of Algorithm 1.
        dict(_case("slab", BRAIN, iters=30, labels=True), name="slab-brain"),
        # Gradient of the objective after some iterations (refinement of a particle).  Ten: the
        # gradient at the initial centres fades with every iteration until only rounding is left.
        dict(_case("adjoint", BRAIN, iters=10), name="adjoint-brain"),
        # Two rings: the 5x5x5 neighbourhood.
        dict(_case("swarm", "104x251x204", V=2, iters=5, P=8), name="ring2-204x251x104"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng, most):
    while True:
        z, y, x = _log(rng, 4, 190), _log(rng, 16, 400), _log(rng, 16, 400)
        if 4000 <= z * y * x <= most:
            return z, y, x


def draw(rng):
    what = rng.choice(["normalize", "fcm", "solve", "solve", "solve", "swarm", "swarm", "swarm", "slab", "adjoint",
                       "ring"])
    z, y, x = _shape(rng, 12_000_000)
    n, vol = z * y * x, "%dx%dx%d" % (z, y, x)
    eps = rng.choice([0.0, 0.0, 1e-5])
    C, m = rng.choice([2, 3, 4, 4, 4, 4, 5, 6, 8, 11, 16]), rng.choice([2.0, 2.0, 2.0, 1.5, 2.5])
    if what == "normalize":
        return _case(what, vol)
    if what == "fcm":
        return _case(what, vol, C=C, m=m, iters=50, eps=rng.choice([0.0, 1e-5]))
    if what == "solve":
        its = max(3, min(_log(rng, 5, 50), int(1.6e9 / (n * C))))
        return _case(what, vol, C=C, m=m, iters=its, eps=eps, labels=n <= 100_000)
    if what == "slab":
        return _case(what, vol, C=rng.choice([3, 4, 4]), iters=_log(rng, 5, 50), labels=n <= 100_000)
    if what == "adjoint":
        return _case(what, vol, C=rng.choice([3, 4, 4, 5]), iters=_log(rng, 5, 12))
    if what == "ring":
        V, sq = rng.choice([(2, False), (2, False), (3, False), (3, True)])
        P, cells = rng.choice([1, 4, 8]), {(2, False): 124, (3, False): 342, (3, True): 26}[V, sq]
        its = max(2, min(10, int(2.0e10 / (n * P * cells))))
        P = max(1, min(P, int(2.0e10 / (n * its * cells))))
        return _case("swarm", vol, V=V, sq=sq, iters=its, P=P)
    B = rng.choice([1, 1, 2, 4])
    shapes = [_shape(rng, 3_000_000) for _ in range(B)] if B > 1 else [(z, y, x)]
    n = sum(a * b * c for a, b, c in shapes)
    P = max(1, min(_log(rng, 2, 64), int(3.0e8 / n)))
    its = max(2, min(_log(rng, 3, 40), int(1.5e9 / (n * P))))
    plain = B * P <= 16 and rng.random() < 0.25
    return _case("swarm", " ".join("%dx%dx%d" % s for s in shapes), C=4 if rng.random() < 0.7 else min(C, 6),
                 m=m if rng.random() < 0.3 else 2.0, iters=its, eps=eps, P=P, plain=plain)


# ------------------------------------------------------------------ inputs


def _shapes(case):
    return [tuple(int(v) for v in s.split("x")) for s in case["volumes"].split()]


def _raw(shape, seed):
    """A volume of three nested tissues and a dozen ellipsoids with noise."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = torch.rand(16, 8, generator=g, device="cuda").tolist()
    az, ay, ax = ((torch.arange(n, device="cuda", dtype=torch.float32) + 0.5) * (2.0 / n) - 1.0 for n in shape)
    az, ay, ax = az[:, None, None], ay[None, :, None], ax[None, None, :]
    v = torch.zeros(shape, device="cuda")
    for k, (rad, val) in enumerate(((0.85, 0.3), (0.65, 0.6), (0.4, 0.9))):
        d = ((ax - 0.1 * r[k][0]) ** 2 + (ay - 0.1 * r[k][1]) ** 2 + (az - 0.1 * r[k][2]) ** 2).sqrt()
        v.masked_fill_(d <= rad * (0.9 + 0.2 * r[k][3]), val)
    for k in range(3, 15):
        c, s = [1.8 * t - 0.9 for t in r[k][:3]], [0.05 + 0.25 * t for t in r[k][3:6]]
        d = ((ax - c[0]) / s[0]) ** 2 + ((ay - c[1]) / s[1]) ** 2 + ((az - c[2]) / (2 * s[2])) ** 2
        v.masked_fill_(d <= 1.0, (0.0, 0.3, 0.6, 0.9)[int(4 * r[k][6]) % 4])
    return v + 0.06 * torch.randn(shape, generator=g, device="cuda")


def _normalized(raw):
    lo, hi = raw.min().double(), raw.max().double()
    return ((raw.double() - lo) / (hi - lo)).float()


def _memberships64(x, c, m):
    """FCM memberships (N, C) of the flat volume x (float64) at centres c."""
    d2 = ((x[:, None] - c) ** 2).clamp_min(1e-12)
    w = (d2.amin(1, keepdim=True) / d2) ** (1.0 / (m - 1.0))
    return w / w.sum(1, keepdim=True)


def _start(x, C, m):
    """Sorted FCM centres of a sample of x, and the memberships they give x."""
    s = x.reshape(-1)[:: max(1, x.numel() // 50_000)].double()
    c = (torch.arange(C, device="cuda", dtype=torch.float64) + 0.5) / C
    for _ in range(8):
        w = _memberships64(s, c, m) ** m
        c = (w * s[:, None]).sum(0) / w.sum(0)
    c = c.sort().values.float()
    U = torch.cat([_memberships64(t.double(), c.double(), m).float() for t in x.reshape(-1).split(1 << 20)])
    return c.cpu().numpy(), U


def _particles(P, seed):
    v = np.random.default_rng(seed).random((P, 2))
    return (v * (0.95 / np.maximum(0.95, v.sum(1, keepdims=True)))).astype(np.float32)


def _params(case):
    return Params(C=case["C"], m=case["m"], V=case["V"], h=1.0, eps=case["eps"], max_iter=case["iters"],
                  flags=PIFCM_SHELL_SQDIST if case["sq"] else 0)


def _inputs(case, seed):
    """Everything of a state but the library's handle."""
    s = dict(case)
    raws = [_raw(shape, seed * 64 + b) for b, shape in enumerate(_shapes(case))]
    if case["kind"] == "normalize":
        return dict(s, raw=raws[0])
    s["xs"] = [_normalized(r) for r in raws]
    if case["kind"] == "fcm":
        return s
    starts = [_start(x, case["C"], case["m"]) for x in s["xs"]]
    parts = _particles(max(1, case["P"]), seed)
    if case["kind"] == "adjoint":  # where the swarm's refinement starts: inside the region
        parts = parts * np.float32(0.7)
    return dict(s, c0=np.stack([c for c, _ in starts]), U0=[U for _, U in starts], parts=parts)


_handle = []  # one context for the whole program, as a program that segments many volumes keeps it


def prepare(case, seed):
    if not _handle:
        _handle.append(Context(0))
    return dict(_inputs(case, seed), ctx=_handle[0], p=_params(case))


# ------------------------------------------------------------------ the pass


def run(s):
    ctx, p, kind = s["ctx"], s["p"], s["kind"]
    if kind == "normalize":
        return ctx.pifcm_normalize(s["raw"])
    if kind == "fcm":
        c, U, it = ctx.pifcm_fcm_init(s["xs"][0], p)
        return dict(c=c, U=U, iters=it)
    if kind == "swarm":
        r = ctx.swarm_evaluate(s["xs"], p, s["parts"], s["c0"], s["U0"],
                               mode=PIFCM_SWARM_PLAIN if s["plain"] else PIFCM_SWARM_BATCHED)
        # The fitness is a sum of float32 terms (only the sums of tiles are added in 64 bits).
        return dict(r, fitness=r["fitness"].astype(np.float32))
    lam, xi = (float(v) for v in s["parts"][0])
    x, c0, U0 = s["xs"][0], s["c0"][0], s["U0"][0]
    if kind == "solve":
        return ctx.ifcm_solve(x, p, lam, xi, c0, U_in=U0, labels=s["labels"])
    if kind == "slab":
        z = x.shape[0] // 2
        return ctx.ifcm_solve_slab(x, z, z + 1, p, lam, xi, c0, U0, labels=s["labels"])
    r = ctx.ifcm_backward(x, p, lam, xi, c0, U0, s["iters"], min(CKPT, s["iters"]))
    return dict(r, dc=r["dc"].astype(np.float32))  # sums of float32 terms, as above


def _cells(case):
    if case["sq"]:
        return len(_offsets(case["V"], True))
    return (2 * case["V"] + 1) ** 3 - 1


def work(case):
    """Per iteration and particle the whole state is read and written once (the
    centres close an iteration over all voxels); FCM memberships are a function
    of x and the centres, so its iterations need x alone."""
    n, C, T, P = sum(z * y * x for z, y, x in _shapes(case)), case["C"], case["iters"], max(1, case["P"])
    if case["eps"] > 0:
        T = (T + 1) // 2  # where the stop rule usually ends it
    each = _cells(case) * (2 * C - 1) + 34 * C  # attraction sums, then distance, memberships, centres
    kind = case["kind"]
    if kind == "normalize":
        return dict(bytes=8.0 * n, flops=4.0 * n)
    if kind == "fcm":
        return dict(bytes=4.0 * n * T + 4.0 * C * n, flops=14.0 * C * n * T)
    if kind == "slab":
        plane = n // _shapes(case)[0][0]
        return dict(bytes=8.0 * C * n + T * plane * (8.0 * C + 4.0), flops=float(each) * plane * T)
    if kind == "adjoint":
        return dict(bytes=n * T * (20.0 * C + 8.0), flops=3.0 * each * n * T)
    return dict(bytes=n * float(T) * (8.0 * C * P + 4.0), flops=float(each) * n * T * P)


# ------------------------------------------------- the same in 64 bits (torch)


def _offsets(V, sq):
    R = math.isqrt(V) if sq else V
    out = []
    for dz in range(-R, R + 1):
        for dy in range(-R, R + 1):
            for dx in range(-R, R + 1):
                r = dx * dx + dy * dy + dz * dz if sq else max(abs(dx), abs(dy), abs(dz))
                if 1 <= r <= V:
                    out.append((dz, dy, dx, r, float(dx * dx + dy * dy + dz * dz) ** 2))
    return out


class _Exact:
    """One volume's IFCM iteration; U is (C, Z, Y, X), planes [za, zb) iterated."""

    def __init__(self, x, case, za=0, zb=None):
        self.C, self.m, self.V, self.sq = case["C"], case["m"], case["V"], case["sq"]
        self.za, self.zb = za, x.shape[0] if zb is None else zb
        self.off = _offsets(self.V, self.sq)
        self.R = max(max(abs(v) for v in o[:3]) for o in self.off)
        self.x = x.double()[self.za:self.zb]
        self.xp = torch.nn.functional.pad(x.double(), [self.R] * 6)
        self.one = torch.nn.functional.pad(torch.ones_like(x, dtype=torch.float64), [self.R] * 6)
        w = [math.exp(-(r - 1) / 1.0) for r in range(1, self.V + 1)]
        self.W = [v / sum(w) for v in w]
        z = torch.zeros_like(self.x)
        self.gs, self.qs, self.n = ([z.clone() for _ in w] for _ in range(3))
        for dz, dy, dx, r, q in self.off:
            ok = self._at(self.one, dz, dy, dx)
            self.gs[r - 1] += (self.x - self._at(self.xp, dz, dy, dx)).abs() * ok
            self.qs[r - 1] += q * ok
            self.n[r - 1] += ok
        self.flat = any(bool((g == 0).any()) for g in self.gs)

    def _at(self, a, dz, dy, dx):
        R, (Z, Y, X) = self.R, self.x.shape
        z = R + self.za + dz
        return a[..., z:z + Z, R + dy:R + dy + Y, R + dx:R + dx + X]

    def attraction(self, U, lam, xi):
        Up = torch.nn.functional.pad(U, [self.R] * 6)
        a = torch.ones((self.C, *self.x.shape), dtype=torch.float64, device=U.device)
        for r in range(1, self.V + 1):
            if not any(o[3] == r for o in self.off):
                continue
            h = torch.zeros_like(a)
            f = torch.zeros_like(a)
            mean = torch.zeros_like(a) if self.flat else None
            for dz, dy, dx, ring, q in self.off:
                if ring != r:
                    continue
                u = self._at(Up, dz, dy, dx)
                g = (self.x - self._at(self.xp, dz, dy, dx)).abs()
                h = h + g * u if U.requires_grad else h.addcmul_(u, g)
                f = f + q * (u * u) if U.requires_grad else f.addcmul_(u, u, value=q)
                if self.flat:
                    mean = mean + u
            gs, qs, n = self.gs[r - 1], self.qs[r - 1], self.n[r - 1]
            h = h / torch.where(gs > 0, gs, 1.0)
            if self.flat:
                h = torch.where(gs > 0, h, mean / n.clamp_min(1.0))
            a = a - lam * self.W[r - 1] * h - xi * self.W[r - 1] * f / qs.clamp_min(1.0)
        return a

    def _own(self, U):
        return U[:, self.za:self.zb]

    def distances(self, U, c, lam, xi):
        e = (self.x - c[:, None, None, None]) ** 2 * self.attraction(U, lam, xi)
        return e.clamp_min(1e-12)

    def objective(self, U, c, lam, xi):
        return (self._own(U) ** self.m * self.distances(U, c, lam, xi)).sum()

    def step(self, U, c, lam, xi):
        """(U', c', J of the input)"""
        d = self.distances(U, c, lam, xi)
        J = (self._own(U) ** self.m * d).sum()
        w = (d.amin(0, keepdim=True).detach() / d) ** (1.0 / (self.m - 1.0))
        u = w / w.sum(0, keepdim=True)
        um = u ** self.m
        c2 = (um * self.x).sum((1, 2, 3)) / um.sum((1, 2, 3))
        if self.zb - self.za < U.shape[1]:
            u = torch.cat([U[:, :self.za], u, U[:, self.zb:]], 1)
        return u, c2, J

    def solve(self, U, c, lam, xi, iters, eps):
        before, t = None, 0
        while t < iters:
            U, c, J = self.step(U, c, lam, xi)
            J, t = float(J), t + 1
            if t >= 2 and eps > 0 and abs(J - before) <= eps * abs(before):
                break
            before = J
        return U, c, float(self.objective(U, c, lam, xi)), t


def _planes(U, x, C):
    return U.double().reshape(*x.shape, C).permute(3, 0, 1, 2).contiguous()


def _rows(U):
    return U.permute(1, 2, 3, 0).reshape(-1, U.shape[0])


def _exact_fcm(x, case, eps):
    C, m = case["C"], case["m"]
    v = x.reshape(-1).double()
    c = torch.tensor([np.float32((j + 0.5) / C) for j in range(C)], dtype=torch.float64, device=v.device)
    U, before, t = _memberships64(v, c, m), None, 0
    while t < case["iters"]:
        d2 = ((v[:, None] - c) ** 2).clamp_min(1e-12)
        J, t = float((U ** m * d2).sum()), t + 1
        U = _memberships64(v, c, m)
        w = U ** m
        c = (w * v[:, None]).sum(0) / w.sum(0)
        if t >= 2 and eps > 0 and abs(J - before) <= eps * abs(before):
            break
        before = J
    at = torch.argsort(c, stable=True)
    return dict(c=c[at], U=U[:, at], iters=t)


def _exact_adjoint(x, case, lam, xi, c0, U0):
    from torch.utils.checkpoint import checkpoint
    E = _Exact(x, case)
    lam, xi = (torch.tensor(float(v), dtype=torch.float64, device="cuda", requires_grad=True) for v in (lam, xi))
    c0 = c0.clone().requires_grad_()
    U, c = U0.clone().requires_grad_(), c0
    for _ in range(case["iters"]):
        U, c, _ = checkpoint(E.step, U, c, lam, xi, use_reentrant=False)
    J = checkpoint(E.objective, U, c, lam, xi, use_reentrant=False)
    gl, gx, gc = torch.autograd.grad(J, (lam, xi, c0))
    return dict(J=J.detach(), dlam=gl, dxi=gx, dc=gc)


def exact(case, seed):
    s = _inputs(case, seed)
    if case["kind"] == "normalize":
        lo, hi = s["raw"].min().double(), s["raw"].max().double()
        return (s["raw"].double() - lo) / (hi - lo)
    eps, C, x = float(np.float32(case["eps"])), case["C"], s["xs"][0]
    if case["kind"] == "fcm":
        return _exact_fcm(x, case, eps)
    if case["kind"] == "swarm":
        B, P = len(s["xs"]), case["P"]
        out = dict(fitness=np.empty((B, P)), centres=np.empty((B, P, C)), iters=np.empty((B, P), np.int32))
        for b, x in enumerate(s["xs"]):
            E, U0 = _Exact(x, case), _planes(s["U0"][b], x, C)
            c0 = torch.from_numpy(s["c0"][b]).double().cuda()
            for k, (lam, xi) in enumerate(s["parts"].tolist()):
                _, c, out["fitness"][b, k], out["iters"][b, k] = E.solve(U0, c0, lam, xi, case["iters"], eps)
                out["centres"][b, k] = c.cpu().numpy()
        return out
    lam, xi = s["parts"][0].tolist()
    U0, c0 = _planes(s["U0"][0], x, C), torch.from_numpy(s["c0"][0]).double().cuda()
    if case["kind"] == "adjoint":
        return _exact_adjoint(x, case, lam, xi, c0, U0)
    E = _Exact(x, case)
    if case["kind"] == "slab":
        z = x.shape[0] // 2
        E = _Exact(x, case, z, z + 1)
    U, c, J, t = E.solve(U0, c0, lam, xi, case["iters"], eps)
    return dict(U=_rows(U), c=c, J=np.array(J), iters=t, labels=None)
