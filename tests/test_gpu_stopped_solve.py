"""psi of a solve that stops before it converges holds every complete iteration.

x takes two directions at a time, so a stop can find one of them not entered
yet.  Three ways to stop: the iteration limit (odd and even), and a number
beyond the FP64 range at each of the two places of an iteration that look for
one, <p, A p> and |r|^2, in each of the two phases.  The even half of psi is
compared with a CG in numpy stopped at the same iteration; FP64 at 1e-10 (a few
iterations of a well conditioned system at 1.1e-16), FP32 at 1e-4.

For the overflow the source is built from eigenvectors of M^+M^ whose weights
make that number the largest so far, by the margins asserted, and is scaled
until it alone is above the range.
"""
import numpy as np
import pytest

import mdwf_synth as S
import oracle as O
from gpu_util import empty_like_dev, log, to_dev, to_host

pytestmark = pytest.mark.gpu

ENAN, ENOCONV = -6, -4
LAT, L5, MQ = (2, 2, 2, 2), 4, 0.02
SHAPE = (L5,) + LAT[::-1] + (4, 3)


def _dense():
    """Links, the oracle's action, M^ on the even sites and their indices."""
    U = S.gauge_field(LAT, 0.6, 3)
    a = O.Action(LAT, L5, 1.5, 0.5, 1.3, MQ)
    even = np.broadcast_to(O.parity_mask(a, 0), SHAPE).reshape(-1) != 0
    idx = np.nonzero(even)[0]
    Mh = np.empty((len(idx), len(idx)), dtype=np.complex128)
    for k, i in enumerate(idx):
        e = np.zeros(even.size, dtype=np.complex128)
        e[i] = 1
        Mh[:, k] = O.mhat(U, e.reshape(SHAPE), a).reshape(-1)[idx]
    return U, a, Mh, idx


def _cg(Mh, b, n):
    """x, <p, A p> and |r|^2 of n iterations on M^+M^ x = b."""
    x, r, p = np.zeros_like(b), b.copy(), b.copy()
    rr = np.vdot(r, r).real
    xs, pqs, rrs = [x], [], [rr]
    for _ in range(n):
        q = Mh @ p
        pq = np.vdot(q, q).real
        x = x + (rr / pq) * p
        r = r - (rr / pq) * (Mh.conj().T @ q)
        new = np.vdot(r, r).real
        p = r + (new / rr) * p
        rr = new
        xs.append(x)
        pqs.append(pq)
        rrs.append(rr)
    return xs, pqs, rrs


def _solve(U, a, Mh, idx, b, inner, **opts):
    """The source whose normal equations have the right-hand side b."""
    from paper_1810_01609_amd import mdwf as M

    hat = np.zeros(int(np.prod(SHAPE)), dtype=np.complex128)
    hat[idx] = np.linalg.solve(Mh.conj().T, b)
    eta = O.m5(hat.reshape(SHAPE), a)
    act = M.Action.make(LAT, L5, 1.5, 0.5, 1.3, MQ)
    with M.Context(0) as ctx:
        g = ctx.gauge_load(LAT, U, precs=("f64", inner))
        psi = empty_like_dev(SHAPE)
        st = ctx.solve(g, act, M.CGOpts.make(tol=1e-14, inner=inner, **opts), to_dev(eta), psi, raise_on_fail=False)[0]
        got = to_host(psi).reshape(-1)[idx]
        g.free()
    return st, got


# what overflows: (weights on the eigenvectors of these eigenvalues, iteration, phase, "pq" or "rr")
STOPS = {
    "rr_phase0": ([(2.70, 0.2016), (0.129, 0.9786), (0.401, 0.0417)], 0, "rr"),
    "pq_phase1": ([(2.70, 0.1116), (0.222, 0.9936), (0.331, 0.0187)], 1, "pq"),
    "rr_phase1": ([(0.129, 0.7551), (0.967, 0.6376), (2.518, 0.1526)], 1, "rr"),
    "pq_phase0": ([(2.469, 0.0398), (0.129, 0.8426), (0.976, 0.4904), (1.913, 0.0469), (1.0001, 0.0762),
                   (0.712, 0.1998)], 2, "pq"),
}


@pytest.mark.parametrize("name", list(STOPS))
def test_overflow_keeps_complete_iterations(name):
    weights, it, what = STOPS[name]
    U, a, Mh, idx = _dense()
    lam, V = np.linalg.eigh(Mh.conj().T @ Mh)
    b = sum(w * V[:, np.argmin(np.abs(lam - l))] for l, w in weights)
    xs, pqs, rrs = _cg(Mh, b, it + 1)
    before = pqs[:it] + rrs[:it + 1] + ([pqs[it]] if what == "rr" else [])
    top = pqs[it] if what == "pq" else rrs[it + 1]
    assert top > 1.25 * max(before), (top, before)
    scale = np.sqrt(np.finfo(np.float64).max) * np.sqrt(1.0 / (top * max(before))) ** 0.5
    st, got = _solve(U, a, Mh, idx, scale * b, "f64")
    want = scale * xs[it if what == "pq" else it + 1]
    err = np.abs(got - want).max() / np.abs(want).max()
    log(f"[stop] {name}: status {st['status']} iterations {st['iters']} error {err:.1e}")
    assert st["status"] == ENAN and st["iters"] == (it if what == "pq" else it + 1)
    assert err < 1e-10


@pytest.mark.parametrize("inner,tol", [("f64", 1e-10), ("f32", 1e-4)])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 7, 8])
def test_iteration_limit(inner, tol, n):
    U, a, Mh, idx = _dense()
    rng = np.random.default_rng(5)
    b = rng.standard_normal(len(idx)) + 1j * rng.standard_normal(len(idx))
    st, got = _solve(U, a, Mh, idx, b, inner, max_iter=n, **({} if inner == "f64" else {"delta": 0.0}))
    want = _cg(Mh, b, n)[0][n]
    err = np.abs(got - want).max() / np.abs(want).max()
    log(f"[stop] {inner} max_iter {n}: status {st['status']} iterations {st['iters']} error {err:.1e}")
    assert st["status"] == ENOCONV and st["iters"] == n
    assert err < tol
