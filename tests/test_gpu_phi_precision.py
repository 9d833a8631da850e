"""The operators on 16-bit user fields form M_phi psi in FP32 and round only the
projected half-spinors: what two nearly equal spins differ by survives.

One site holds spin 0 on slices s - 1 and s and spin 2 on slice s, with b5 = 1
and c5 far below the storage roundoff of 1: (M_phi psi)_0 = 1 + c5 and
(M_phi psi)_2 = 1 on slice s, and the neighbour below in t receives their
difference c5 (1 - gamma_t).  A field of M_phi psi in 16-bit storage holds
1 + c5 as 1 and gives nothing there.

Tolerances, relative to that neighbour's own magnitude.  FP16, BF16 (c5 =
2^-13): psi, the sum, the difference and the product with unit links are exact
in FP32 and the difference is exact in 16 bits, so the output's storage and M5's
FP32 sums remain: the bars of the operator tests (16 u).  int16 (c5 = 1.4 units
of the storage grid): four FP32 roundoffs of values near 1 against c5,
4 * 2^-24 / 4.3e-5 = 5.6e-3, and the storage's 1e-3: 1e-2.
"""
import numpy as np
import pytest

import mdwf_synth as S
import oracle as O
from gpu_util import empty_like_dev, log, to_dev, to_host

pytestmark = pytest.mark.gpu

C5 = {"f16": 2.0 ** -13, "bf16": 2.0 ** -13, "i16": 1.4 / 32767}
TOL = {"f16": 8e-3, "bf16": 6e-2, "i16": 1e-2}


@pytest.mark.parametrize("prec", list(C5))
@pytest.mark.parametrize("L5", [5, 8])
@pytest.mark.parametrize("site", [(2, 1, 0, 2), (2, 1, 0, 3)], ids=["odd", "even"])
def test_difference_of_near_equal_spins(prec, L5, site):
    from paper_1810_01609_amd import mdwf as M

    L = (4, 2, 2, 4)
    U = S.unit_gauge(L)
    act = M.Action.make(L, L5, 1.0, C5[prec], 1.3, 0.05, 0)
    oact = O.Action(L, L5, 1.0, C5[prec], 1.3, 0.05, t_antiperiodic=False)
    X, Y, Z, T = site
    s = 2
    x = np.zeros((L5,) + L[::-1] + (4, 3), dtype=np.complex128)
    x[s - 1, T, Z, Y, X, 0, 1] = 1
    x[s, T, Z, Y, X, 0, 1] = 1
    x[s, T, Z, Y, X, 2, 1] = 1
    want = O.dirac(U, x, oact)[s, T - 1, Z, Y, X]
    assert 0 < np.abs(want).max() < 2 * C5[prec]
    with M.Context(0) as ctx:
        g = ctx.gauge_load(L, U, precs=("f64", prec))
        out = empty_like_dev(x.shape)
        ctx.dslash(g, act, M.OP_D, prec, to_dev(x), out)
        got = to_host(out)[s, T - 1, Z, Y, X]
        g.free()
    err = np.abs(got - want).max() / np.abs(want).max()
    log(f"[phi] {prec} L5={L5} {site}: {err:.2e} (bar {TOL[prec]:.0e})")
    assert err <= TOL[prec]
