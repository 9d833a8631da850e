"""The physical source rounds each complex product of the colour multiplication
once before it joins the sum, and each term of the hop once as it joins the
source: the arithmetic repeated here in numpy.

Multiply-adds are formed in long double (64-bit mantissa) and rounded to FP64:
one in 2^10 comes out one unit off, so with some 50 of them behind a value about
5 % of the values may differ.  A chain of multiply-adds over the whole colour
sum, 1 to 3 % further from the exact source, agrees in less than half of them.
The bar is 90 %.
"""
import numpy as np
import pytest

import mdwf_synth as S
import oracle as O
from gpu_util import empty_like_dev, log, to_dev, to_host

pytestmark = pytest.mark.gpu


def _fma(a, b, c):
    return (a.astype(np.longdouble) * b + c).astype(np.float64)


def _cmul(a, b):
    """a b as the links' third row is rebuilt from the first two."""
    return _fma(a.real, b.real, -(a.imag * b.imag)) + 1j * _fma(a.real, b.imag, a.imag * b.real)


def _expected(U, xi, b5, c5, m5, mask, L5):
    U = U.copy()
    for j in range(3):
        k, l = (j + 1) % 3, (j + 2) % 3
        U[..., 2, j] = (_cmul(U[..., 0, k], U[..., 1, l]) - _cmul(U[..., 0, l], U[..., 1, k])).conj()
    beta, hc = np.full((), 1.0 - c5 * (4.0 - m5)), 0.5 * c5
    chi = np.einsum("ab,...bc->...ac", O.gamma_product(mask), xi)
    out = np.zeros((L5,) + xi.shape, dtype=np.complex128)
    for w in (0, 1):
        v = np.zeros_like(chi)
        v[..., 2 * w:2 * w + 2, :] = chi[..., 2 * w:2 * w + 2, :]
        re, im = beta * v.real, beta * v.imag
        for mu in range(4):
            ax = 3 - mu
            for fb in (0, 1):
                u = U[..., mu, :, :] if fb == 0 else np.roll(U[..., mu, :, :], 1, ax).swapaxes(-1, -2).conj()
                n = np.roll(v, 1 if fb else -1, ax)
                y = np.zeros_like(v)
                for a in range(3):
                    for b in range(3):
                        p, q = u[..., a, b, None], n[..., b]
                        y[..., a] += _fma(p.real, q.real, -(p.imag * q.imag)) + 1j * _fma(p.imag, q.real, p.real * q.imag)
                z = y + (1 if fb else -1) * np.einsum("ab,...bc->...ac", O.GAMMA[mu], y)
                c = np.full(xi.shape, hc)
                if mu == 3:
                    c[-1 if fb == 0 else 0] = -hc
                re, im = _fma(c, z.real, re), _fma(c, z.imag, im)
        out[0 if w == 0 else L5 - 1] += re + 1j * im
    return out


@pytest.mark.parametrize("b5,c5,m5", [(1.5, 0.5, 1.3), (1.7, 0.7, 1.1)])
def test_source_arithmetic(b5, c5, m5):
    from paper_1810_01609_amd import mdwf as M

    L, L5, mask = (6, 4, 4, 6), 3, 11
    U = S.gauge_field(L, 0.3, 12)
    xi = S.random_spinor(L, 1, 13)[0]
    act = M.Action.make(L, L5, b5, c5, m5, 0.05)
    with M.Context(0) as ctx:
        g = ctx.gauge_load(L, U)
        eta = empty_like_dev((L5,) + xi.shape)
        ctx.source_physical(g, act, to_dev(xi), eta, gamma_mask=mask)
        got = to_host(eta)
        g.free()
    want = _expected(U, xi, b5, c5, m5, mask, L5)
    same = np.mean([(got.real == want.real)[[0, -1]].mean(), (got.imag == want.imag)[[0, -1]].mean()])
    log(f"[source] b5 {b5} c5 {c5}: {100 * same:.1f} % of the values equal")
    assert np.abs(got - want).max() < 1e-14
    assert same > 0.9
