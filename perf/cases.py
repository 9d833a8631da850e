"""The work a user of libmdwf has it do, as cases that can be timed.

A case is a dict of plain values; ``kind`` says which entry points it takes:

* ``solve``  one ``Context.solve``: the propagators of ``nrhs`` sources,
* ``batch``  continuous batching: three jobs of different quark mass begun,
  stepped together 25 iterations at a time until all are done, and ended,
* ``op``     one ``Context.dslash`` (``noalloc``: ``dslash_noalloc``),
* ``source`` the sources of a sequential propagator: read the 4D propagator
  off the walls, apply a current, form the physical 5D source.

Links are exp(i eps H) with H a Gaussian traceless Hermitian matrix, sources
are complex Z2 noise or spin-colour points on the walls, operator inputs are
Gaussian: the distributions of the benchmark and of the tests.  Every solve
is carried to 3e-13 on the normal equations.
"""
from __future__ import annotations

import math

import torch

from paper_1810_01609_amd import mdwf as M

B5, C5, M5 = 1.5, 0.5, 1.3
TOL = 3e-13
STEP_ITERS = 25

_ctx = None


def _context():
    """One context per process, as a user's program has."""
    global _ctx
    if _ctx is None:
        _ctx = M.Context(0)
    return _ctx


def _case(name, kind, L, L5, mq, eps, prec, nrhs, **more):
    c = dict(kind=kind, Lx=L[0], Ly=L[1], Lz=L[2], Lt=L[3], L5=L5, mq=mq, eps=eps, prec=prec, nrhs=nrhs,
             source="z2", op="", noalloc=False, mask=0, tap=True)
    if name:
        c["name"] = name
    c.update(more)
    return c


def listed():
    return [
        # one point source on the smallest lattice: latency of some 700 launches
        _case("solve 4x4x4x8 L8 f32", "solve", (4, 4, 4, 8), 8, 0.05, 0.3, "f32", 1, source="point"),
        # the serving loop's smallest lane: requests of different mass and size stepped together
        _case("batch 8x8x8x16 L8 f32 11rhs", "batch", (8, 8, 8, 16), 8, 0.02, 0.2, "f32", 11),
        # one stochastic propagator on a small production lattice, fields about as large as the caches
        _case("solve 16x16x16x32 L12 f32", "solve", (16, 16, 16, 32), 12, 0.02, 0.2, "f32", 1),
        # the twelve spin-colour point sources of a propagator fused, 16-bit storage
        _case("solve 16x16x16x32 L12 f16 12rhs", "solve", (16, 16, 16, 32), 12, 0.02, 0.2, "f16", 12, source="point"),
        # a medium lattice with a longer fifth dimension
        _case("solve 24x24x24x64 L16 f16", "solve", (24, 24, 24, 64), 16, 0.01, 0.15, "f16", 1),
        # the largest lattice at a light mass
        _case("solve 32x32x32x64 L12 f16", "solve", (32, 32, 32, 64), 12, 0.005, 0.15, "f16", 1),
        # the paper's fixed-point storage, on a ragged lattice (sites per parity no multiple of 16)
        _case("solve 10x6x14x18 L10 i16 2rhs", "solve", (10, 6, 14, 18), 10, 0.03, 0.25, "i16", 2),
        # the Dirac operator in full precision, as a user's residual check applies it
        _case("op D 16x16x16x32 L12 f64", "op", (16, 16, 16, 32), 12, 0.02, 0.2, "f64", 1, op="D"),
        # the normal operator on the largest lattice in the arithmetic type of the solver
        _case("op NORMAL 32x32x32x64 L12 f32", "op", (32, 32, 32, 64), 12, 0.005, 0.15, "f32", 1, op="NORMAL"),
        # a preconditioner-style application in 16-bit storage, several fields
        _case("op MHAT 24x24x24x64 L16 f16 2rhs", "op", (24, 24, 24, 64), 16, 0.01, 0.15, "f16", 2, op="MHAT"),
        # the allocation-free call in a tight loop on a small ragged lattice
        _case("op M+ noalloc 6x10x4x14 L5 f64", "op", (6, 10, 4, 14), 5, 0.05, 0.3, "f64", 1, op="MHATDAG",
              noalloc=True, tap=False),
        # sequential sources of the twelve spin-colours with an axial current
        _case("source 16x16x16x32 L12 12rhs", "source", (16, 16, 16, 32), 12, 0.02, 0.2, "f64", 12, mask=11),
    ]


_OPS = ["D", "DDAG", "MHAT", "MHATDAG", "NORMAL", "HOP_EO", "HOP_OE", "HOP", "HOPDAG", "M5", "M5INV", "MPHI", "PREP"]


def _even_log(rng, lo, hi):
    return 2 * max(1, round(math.exp(rng.uniform(math.log(lo / 2), math.log(hi / 2)))))


def draw(rng):
    while True:
        kind = rng.choice(["solve", "solve", "solve", "batch", "op", "op", "op", "source"])
        big = 32 if kind != "batch" else 14
        L = [_even_log(rng, 4, big) for _ in range(3)] + [_even_log(rng, 4, 64 if kind != "batch" else 24)]
        L5 = rng.choice([8, 12, 16, rng.randint(1, 24)])
        mq = round(rng.uniform(0.005, 0.05), 4)
        eps = round(rng.uniform(0.15, 0.3), 3)
        nrhs = rng.choice([1, 1, 2, rng.randint(3, 12)])
        prec = rng.choice(["f64", "f32", "f32", "f16", "f16", "bf16", "i16"])
        sites = L[0] * L[1] * L[2] * L[3] * L5
        more = {}
        if kind == "batch":
            nrhs = rng.randint(3, 12)
            prec = rng.choice(["f32", "f16"])
        if kind == "op":
            more["op"] = rng.choice(_OPS)
            more["tap"] = rng.random() < 0.8
            more["noalloc"] = 5 * nrhs * sites / 2 * 192 < 200e6 and rng.random() < 0.5
        if kind == "source":
            prec = "f64"
            more["mask"] = rng.randint(0, 15)
        if kind == "solve":
            more["source"] = rng.choice(["z2", "point"])
        most = {"solve": 6e6, "batch": 2e6, "op": 25e6, "source": 25e6}[kind]
        if sites * nrhs <= most:
            return _case(None, kind, L, L5, mq, eps, prec, nrhs, **more)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed, k):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 16 + k)
    return g


def _links(case, seed):
    """SU(3) links exp(i eps H), complex128 [t][z][y][x][mu][3][3], on the GPU."""
    V = case["Lx"] * case["Ly"] * case["Lz"] * case["Lt"]
    out = torch.empty((V, 4, 3, 3), dtype=torch.complex128, device="cuda")
    g = _gen(seed, 1)
    for mu in range(4):
        a = torch.randn((V, 3, 3, 2), dtype=torch.float64, device="cuda", generator=g)
        a = torch.view_as_complex(a)
        h = 0.5 * (a + a.transpose(1, 2).conj())
        tr = (h[:, 0, 0] + h[:, 1, 1] + h[:, 2, 2]) / 3
        for k in range(3):
            h[:, k, k] -= tr
        x = (1j * case["eps"]) * h
        # (1 + x/n (1 + ...)) and a Gram-Schmidt of the rows
        eye = torch.eye(3, dtype=torch.complex128, device="cuda")
        u = eye.expand(V, 3, 3)
        for n in (6, 5, 4, 3, 2, 1):
            u = eye + (x[:, :, :, None] * u[:, None, :, :]).sum(2) / n
        r0 = u[:, 0] / u[:, 0].norm(dim=1, keepdim=True)
        r1 = u[:, 1] - (r0.conj() * u[:, 1]).sum(1, keepdim=True) * r0
        r1 = r1 / r1.norm(dim=1, keepdim=True)
        out[:, mu, 0], out[:, mu, 1] = r0, r1
        out[:, mu, 2] = torch.linalg.cross(r0, r1, dim=1).conj()
    return out.view(case["Lt"], case["Lz"], case["Ly"], case["Lx"], 4, 3, 3)


def _lat(case):
    return (case["Lt"], case["Lz"], case["Ly"], case["Lx"])


def _wall(case, xi):
    """5D source of a 4D one: spins 0,1 on the last slice, spins 2,3 on the first."""
    eta = torch.zeros((case["L5"],) + xi.shape, dtype=torch.complex128, device="cuda")
    eta[case["L5"] - 1, ..., :2, :] = xi[..., :2, :]
    eta[0, ..., 2:, :] += xi[..., 2:, :]
    return eta


def _sources(case, seed):
    g = _gen(seed, 2)
    lat = _lat(case)
    n = case["nrhs"]
    eta = torch.empty((n, case["L5"]) + lat + (4, 3), dtype=torch.complex128, device="cuda")
    place = [int(torch.randint(0, e, (1,), device="cuda", generator=g)) for e in lat]
    for r in range(n):
        if case["source"] == "point":
            xi = torch.zeros(lat + (4, 3), dtype=torch.complex128, device="cuda")
            xi[place[0], place[1], place[2], place[3], (r // 3) % 4, r % 3] = 1
        else:
            b = torch.randint(0, 2, lat + (4, 3, 2), device="cuda", generator=g)
            xi = torch.view_as_complex((1 - 2 * b).to(torch.float64) / math.sqrt(2.0))
        eta[r] = _wall(case, xi)
    return eta


def _gauss(case, seed, shape):
    a = torch.randn(shape + (2,), dtype=torch.float64, device="cuda", generator=_gen(seed, 3))
    return torch.view_as_complex(a)


class _State:
    def __init__(self, **kw):
        self.__dict__.update(kw)

    def __del__(self):
        try:
            self.gauge.free()
        except Exception:
            pass


def _batch_sizes(n):
    """Sources of the three jobs of a batch."""
    a = max(1, n // 2)
    b = max(1, (n - a) // 2)
    return [a, b, max(1, n - a - b)]


def _batch_masses(case):
    return [case["mq"], case["mq"] * 1.5, case["mq"] * 2.0]


def prepare(case, seed):
    ctx = _context()
    L = (case["Lx"], case["Ly"], case["Lz"], case["Lt"])
    act = M.Action.make(L, case["L5"], B5, C5, M5, case["mq"], 1 if case["tap"] else 0)
    links = _links(case, seed)
    gauge = ctx.gauge_load(L, links, precs=tuple(dict.fromkeys(("f64", case["prec"]))))
    del links
    n, lat = case["nrhs"], _lat(case)
    s = _State(case=case, ctx=ctx, act=act, gauge=gauge)
    if case["kind"] == "solve":
        s.eta = _sources(case, seed)
        s.opts = M.CGOpts.make(tol=TOL, inner=case["prec"])
    elif case["kind"] == "batch":
        sizes = _batch_sizes(n)
        s.opts = M.CGOpts.make(tol=TOL, inner=case["prec"])
        s.etas = [_sources(dict(case, nrhs=k), seed + 7 * i) for i, k in enumerate(sizes)]
        s.acts = [M.Action.make(L, case["L5"], B5, C5, M5, m, 1) for m in _batch_masses(case)]
    elif case["kind"] == "op":
        s.x = _gauss(case, seed, (n, case["L5"]) + lat + (4, 3))
    else:
        s.psi = _gauss(case, seed, (n, case["L5"]) + lat + (4, 3))
    return s


# the type in which a user keeps a result of each storage precision
_KEPT = {"f64": torch.complex128, "f32": torch.complex64, "f16": torch.complex32, "bf16": torch.complex32,
         "i16": torch.complex32}


def run(s):
    c, n = s.case, s.case["nrhs"]
    if c["kind"] == "solve":
        psi = torch.empty_like(s.eta)
        s.ctx.solve(s.gauge, s.act, s.opts, s.eta, psi, nrhs=n)
        return list(psi)
    if c["kind"] == "batch":
        psis = [torch.empty_like(e) for e in s.etas]
        jobs = [s.ctx.job_begin(s.gauge, a, s.opts, e, p, nrhs=e.shape[0]) for a, e, p in zip(s.acts, s.etas, psis)]
        live = list(jobs)
        while live:
            st = s.ctx.job_step(live, STEP_ITERS)
            if st != M.OK:
                raise M.MDWFError(st, "mdwf_job_step")
            live = [j for j in live if not j.poll()[0]]
        for j in jobs:
            j.end()
        return psis
    if c["kind"] == "op":
        out = torch.empty_like(s.x)
        call = s.ctx.dslash_noalloc if c["noalloc"] else s.ctx.dslash
        call(s.gauge, s.act, getattr(M, "OP_" + c["op"]), c["prec"], s.x, out, nrhs=n)
        return out.to(_KEPT[c["prec"]])
    q = torch.empty((n,) + _lat(c) + (4, 3), dtype=torch.complex128, device="cuda")
    s.ctx.propagator_4d(s.act, s.psi, q, nrhs=n)
    eta = torch.empty_like(s.psi)
    s.ctx.source_physical(s.gauge, s.act, q, eta, gamma_mask=c["mask"], nrhs=n)
    return {"q": q, "eta": eta}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
_SPINOR = {"f64": 192, "f32": 96, "f16": 52, "bf16": 52, "i16": 52}
_REAL = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2, "i16": 2}


def _iterations(mq):
    """CG iterations to 3e-13 as they go with the quark mass on links of this roughness."""
    return 125.0 * (0.05 / mq) ** 0.45


def work(case):
    v4 = case["Lx"] * case["Ly"] * case["Lz"] * case["Lt"]
    full = float(v4 * case["L5"])  # 5D sites, both parities
    half = full / 2
    n = case["nrhs"]
    sp, links = _SPINOR[case["prec"]], float(v4) * 4 * 12 * _REAL[case["prec"]]
    if case["kind"] in ("solve", "batch"):
        it = _iterations(case["mq"])
        # user fields in and out; per iteration four hop sweeps, each one field in and one out,
        # and x, r, p read and written
        nbytes = 2 * n * full * 192 + it * (n * half * sp * 14 + 4 * links)
        return {"bytes": nbytes, "flops": it * n * half * 6300.0}
    if case["kind"] == "op":
        hops = {"D": 2, "DDAG": 2, "HOP": 2, "HOPDAG": 2, "NORMAL": 4, "MHAT": 2, "MHATDAG": 2, "HOP_EO": 1,
                "HOP_OE": 1, "PREP": 1, "M5": 0, "M5INV": 0, "MPHI": 0}[case["op"]]
        read = full if hops in (0, 2) and case["op"] not in ("MHAT", "MHATDAG") or case["op"] == "PREP" else half
        return {"bytes": n * (read + full) * 192 + (links if hops else 0), "flops": n * half * (1320.0 * hops + 200)}
    # two walls of psi read once, q and eta written
    return {"bytes": n * (2 * v4 * 192.0 + full * 192) + links, "flops": n * v4 * 1500.0}


# ---------------------------------------------------------------------------
# the same in 64 bits with plain torch
# ---------------------------------------------------------------------------
def _gammas():
    i = 1j
    return torch.tensor([
        [[0, 0, 0, i], [0, 0, i, 0], [0, -i, 0, 0], [-i, 0, 0, 0]],
        [[0, 0, 0, -1], [0, 0, 1, 0], [0, 1, 0, 0], [-1, 0, 0, 0]],
        [[0, 0, i, 0], [0, 0, 0, -i], [-i, 0, 0, 0], [0, i, 0, 0]],
        [[0, 0, 1, 0], [0, 0, 0, 1], [1, 0, 0, 0], [0, 1, 0, 0]]], dtype=torch.complex128)


class _Plain:
    """The Moebius operator on [s][t][z][y][x][spin][colour], from its definition."""

    def __init__(self, case, seed, mq=None):
        self.c = case
        self.mq = case["mq"] if mq is None else mq
        self.U = _links(case, seed)
        if case["tap"]:
            self.U = self.U.clone()
            self.U[-1, :, :, :, 3] *= -1  # antiperiodic time
        self.g = _gammas().tolist()

    def _spin(self, mu, sg, x):
        """(1 + sg gamma_mu) x: gamma_mu has one entry per row."""
        y = x.clone()
        for a in range(4):
            for b in range(4):
                if self.g[mu][a][b] != 0:
                    y[..., a, :] += (sg * self.g[mu][a][b]) * x[..., b, :]
        return y

    @staticmethod
    def _mul(u, x):
        """u (lattice, 3, 3) on the colour of x (s, lattice, 4, 3)."""
        y = torch.empty_like(x)
        for a in range(3):
            t = u[..., a, 0, None] * x[..., 0]
            t += u[..., a, 1, None] * x[..., 1]
            t += u[..., a, 2, None] * x[..., 2]
            y[..., a] = t
        return y

    def hop(self, x, dag=False):
        out = torch.zeros_like(x)
        sf = 1 if dag else -1
        for mu in range(4):
            ax = 4 - mu  # t is axis 1 of x and mu = 3
            u = self.U[..., mu, :, :]
            out += self._spin(mu, sf, self._mul(u, torch.roll(x, -1, ax)))
            ud = torch.roll(u, 1, ax - 1).transpose(-1, -2).conj()
            out += self._spin(mu, -sf, self._mul(ud, torch.roll(x, 1, ax)))
        return out

    def p5(self, x, dag=False):
        up = torch.roll(x, -1 if dag else 1, 0)
        dn = torch.roll(x, 1 if dag else -1, 0)
        y = torch.cat([up[..., :2, :], dn[..., 2:, :]], -2)
        first, last = (self.c["L5"] - 1, 0) if dag else (0, self.c["L5"] - 1)
        y[first, ..., :2, :] *= -self.mq
        y[last, ..., 2:, :] *= -self.mq
        return y

    def fifth(self, a, b, x, dag=False):
        return a * x + b * self.p5(x, dag)

    def mphi(self, x, dag=False):
        return self.fifth(B5, C5, x, dag)

    def m5(self, x, dag=False):
        return self.fifth(B5 * (4 - M5) + 1, C5 * (4 - M5) - 1, x, dag)

    def m5inv(self, x, dag=False):
        n = self.c["L5"]
        e = torch.zeros((n, n, 1, 1, 1, 1, 4, 1), dtype=torch.complex128, device="cuda")
        e[range(n), range(n)] = 1
        m = torch.stack([self.m5(e[k], dag) for k in range(n)], 1)[:, :, 0, 0, 0, 0, :, 0]  # [row][column][spin]
        y = torch.empty_like(x)
        for w in (0, 1):
            inv = torch.linalg.inv(m[:, :, 2 * w].cpu()).to(x.device)
            for s in range(n):
                t = torch.zeros_like(x[0, ..., :2, :])
                for k in range(n):
                    t += inv[s, k] * x[k, ..., 2 * w:2 * w + 2, :]
                y[s, ..., 2 * w:2 * w + 2, :] = t
        return y

    def parity(self, p):
        Lt, Lz, Ly, Lx = _lat(self.c)
        r = [torch.arange(k, device="cuda") for k in (Lt, Lz, Ly, Lx)]
        s = r[0][:, None, None, None] + r[1][:, None, None] + r[2][:, None] + r[3]
        return ((s & 1) == p).to(torch.float64)[None, ..., None, None]

    def D(self, x):
        return self.m5(x) - 0.5 * self.hop(self.mphi(x))

    def Ddag(self, x):
        return self.m5(x, True) - 0.5 * self.mphi(self.hop(x, True), True)

    def mhat(self, x):
        """On a field of the even sites: the two hops change parity by themselves."""
        return x - 0.25 * self.m5inv(self.hop(self.mphi(self.m5inv(self.hop(self.mphi(x))))))

    def mhat_dag(self, x):
        y = self.hop(self.m5inv(x, True), True)
        y = self.hop(self.m5inv(self.mphi(y, True), True), True)
        return x - 0.25 * self.mphi(y, True)

    def op(self, name, x):
        even, odd = self.parity(0), self.parity(1)
        if name in ("D", "DDAG"):
            return self.D(x) if name == "D" else self.Ddag(x)
        if name in ("HOP", "HOPDAG"):
            return self.hop(x, name == "HOPDAG")
        if name == "HOP_EO":
            return self.hop(odd * x)
        if name == "HOP_OE":
            return self.hop(even * x)
        if name == "M5":
            return self.m5(x)
        if name == "M5INV":
            return self.m5inv(x)
        if name == "MPHI":
            return self.mphi(x)
        if name == "PREP":
            return self.m5inv(even * x + 0.5 * self.hop(self.mphi(self.m5inv(odd * x))))
        x = even * x
        if name == "MHAT":
            return self.mhat(x)
        if name == "MHATDAG":
            return self.mhat_dag(x)
        return self.mhat_dag(self.mhat(x))

    def solve(self, eta):
        """CG on D^+ D x = D^+ eta, restarted from the true residual."""
        x = torch.zeros_like(eta)
        b = self.Ddag(eta)
        bb = float((b.abs() ** 2).sum())
        for tol in (1e-7, 1e-13):
            r = self.Ddag(eta - self.D(x))
            p = r.clone()
            rr = (r.abs() ** 2).sum()
            for k in range(3000):
                q = self.D(p)
                a = rr / (q.abs() ** 2).sum()
                x += a * p
                r -= a * self.Ddag(q)
                new = (r.abs() ** 2).sum()
                p = r + (new / rr) * p
                rr = new
                if k % 10 == 9 and float(rr) <= tol * tol * bb:
                    break
        return x


def exact(case, seed):
    sites = case["Lx"] * case["Ly"] * case["Lz"] * case["Lt"] * case["L5"]
    n = case["nrhs"]
    if case["kind"] == "solve":
        if sites > 1.7e6:
            return None
        p = _Plain(case, seed)
        eta = _sources(case, seed)
        return [p.solve(eta[r]) if r < 2 and (r == 0 or sites < 4e5) else None for r in range(n)]
    if case["kind"] == "batch":
        if sites > 1.7e6:
            return None
        sizes = _batch_sizes(n)
        first = _Plain(case, seed).solve(_sources(dict(case, nrhs=sizes[0]), seed)[0]) if sizes[0] == 1 else None
        last = None
        if sizes[2] <= 3:
            p = _Plain(case, seed, _batch_masses(case)[2])
            last = torch.stack([p.solve(e) for e in _sources(dict(case, nrhs=sizes[2]), seed + 14)])
        return [None if first is None else first[None], None, last]
    if case["kind"] == "op":
        p = _Plain(case, seed)
        x = _gauss(case, seed, (n, case["L5"]) + _lat(case) + (4, 3))
        return torch.stack([p.op(case["op"], x[r]) for r in range(n)])
    p = _Plain(case, seed)
    psi = _gauss(case, seed, (n, case["L5"]) + _lat(case) + (4, 3))
    last = case["L5"] - 1
    q = torch.cat([psi[:, last, ..., :2, :], psi[:, 0, ..., 2:, :]], -2)
    gam = torch.eye(4, dtype=torch.complex128)
    for mu in range(4):
        if (case["mask"] >> mu) & 1:
            gam = gam @ _gammas()[mu]
    out = torch.zeros_like(psi)
    for r in range(n):
        xi = torch.zeros_like(q[r])
        for a in range(4):
            for b in range(4):
                if gam[a, b] != 0:
                    xi[..., a, :] += complex(gam[a, b]) * q[r][..., b, :]
        w = torch.zeros_like(psi[r])
        w[0, ..., :2, :] = xi[..., :2, :]
        w[last, ..., 2:, :] += xi[..., 2:, :]
        out[r] = (1 - C5 * (4 - M5)) * w + 0.5 * C5 * p.hop(w)
    return {"q": q, "eta": out}
