"""The quad stencil's FP32 results are as close to FP64 as the general kernel's
(which MDWF_STAGE=0 selects) on the same inputs.

The errors are norms over at least 4e5 independent roundings, whose own spread
is 1 / sqrt(2 * 4e5) = 0.1 %: the quad stencil may be 1 % further off.
"""
import numpy as np
import pytest

import mdwf_synth as S
from gpu_util import empty_like_dev, log, rel, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L5,b5,c5,m5,mq", [(4, 1.5, 0.5, 1.3, 0.05), (12, 1.5, 0.5, 1.3, 0.02), (24, 1.25, 0.25, 1.3, 0.2),
                                            (8, 1.0, 0.0, 1.8, 0.01)])
def test_fp32_error_against_general_kernel(L5, b5, c5, m5, mq, monkeypatch):
    from paper_1810_01609_amd import mdwf as M

    L = (8, 8, 8, 8)
    U = S.gauge_field(L, 0.2, 4)
    act = M.Action.make(L, L5, b5, c5, m5, mq)
    x = to_dev(S.random_spinor(L, L5, 6))
    with M.Context(0) as ctx:
        g = ctx.gauge_load(L, U, precs=("f64", "f32"))

        def run(op, prec, stage):
            monkeypatch.setenv("MDWF_STAGE", stage)
            out = empty_like_dev(x.shape)
            ctx.dslash(g, act, getattr(M, "OP_" + op), prec, x, out)
            return to_host(out)

        for op in ("D", "DDAG", "MHAT", "MHATDAG", "NORMAL", "PREP"):
            want = run(op, "f64", "1")
            general, quad = (rel(run(op, "f32", s), want) for s in ("0", "1"))
            log(f"[error] {op} L5={L5}: general {general:.3e} quad {quad:.3e} ({quad / general:.3f})")
            assert quad <= 1.01 * general
        g.free()


# |error| of the source preparation on these inputs with M_phi M5^-1 formed in
# FP32 registers on every neighbour, measured with that kernel
PREP = [(5, 1.5, 0.5, 1.3, 0.05, 7.549e-8), (10, 1.5, 0.5, 1.3, 0.02, 7.191e-8), (12, 1.5, 0.5, 1.3, 0.02, 7.177e-8),
        (7, 1.25, 0.25, 1.3, 0.2, 7.126e-8), (8, 1.7, 0.7, 1.1, 0.05, 9.126e-8)]


@pytest.mark.parametrize("L5,b5,c5,m5,mq,was", PREP)
def test_fp32_source_preparation(L5, b5, c5, m5, mq, was):
    """Storing M_phi M5^-1 eta_o in FP32 costs one rounding, which M5^-1 gives
    back: no further off than `was`, by three spreads of 0.1 %."""
    from paper_1810_01609_amd import mdwf as M

    L = (8, 8, 8, 8)
    act = M.Action.make(L, L5, b5, c5, m5, mq)
    x = to_dev(S.random_spinor(L, L5, 6))
    got = {}
    with M.Context(0) as ctx:
        g = ctx.gauge_load(L, S.gauge_field(L, 0.2, 4), precs=("f64", "f32"))
        for prec in ("f64", "f32"):
            out = empty_like_dev(x.shape)
            ctx.dslash(g, act, M.OP_PREP, prec, x, out)
            got[prec] = to_host(out)
        g.free()
    err = rel(got["f32"], got["f64"])
    log(f"[error] PREP L5={L5}: {err:.3e} (was {was:.3e})")
    assert err <= 1.003 * was
