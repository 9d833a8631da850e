"""A slice that is not finite makes the same outputs not finite in FP32 as in
FP64: the operators couple neighbouring slices and sites only, whichever kernel
applies them.  No tolerance: the two sets of finite outputs are equal."""
import numpy as np
import pytest

import mdwf_synth as S
from gpu_util import empty_like_dev, log, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L5", [4, 5, 8, 12])
@pytest.mark.parametrize("op", ["D", "DDAG", "HOP"])
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_reach_of_a_nonfinite_slice(op, L5, value):
    from paper_1810_01609_amd import mdwf as M

    L = (6, 2, 4, 2)
    U = S.gauge_field(L, 0.3, 8)
    act = M.Action.make(L, L5, 1.5, 0.5, 1.3, 0.05)
    with M.Context(0) as ctx:
        g = ctx.gauge_load(L, U, precs=("f64", "f32"))
        for s in {0, 1, 3, L5 - 1}:
            x = S.random_spinor(L, L5, 3 + s)
            x[s, 1, 2, 0, 3, :, 1] = value
            finite = {}
            for prec in ("f64", "f32"):
                out = empty_like_dev(x.shape)
                ctx.dslash(g, act, getattr(M, "OP_" + op), prec, to_dev(x), out)
                got = to_host(out)
                finite[prec] = np.isfinite(got.real) & np.isfinite(got.imag)
            log(f"[nonfinite] {op} L5={L5} slice {s} {value}: {(~finite['f64']).sum()} / {(~finite['f32']).sum()}")
            assert (~finite["f64"]).any()
            assert np.array_equal(finite["f64"], finite["f32"])
        g.free()
