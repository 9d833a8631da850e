"""The quad stencil over workgroups of several 16-site tiles and several
wavefronts per tile (MDWF_CB_LOG2, as the autotuner may choose them): operators
and a solve give bitwise what 16-site workgroups give.  The second lattice leaves
the last workgroup with tiles beyond the lattice and a ragged one.  The FP64
oracle holds the 16-site results to the operator tests' bars; D and PREP run at
the fifth dimensions where the quad kernel's split can go wrong."""
import numpy as np
import pytest

import mdwf_synth as S
import oracle as O
from gpu_util import check, empty_like_dev, log, to_dev, to_host

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-6, "f16": 8e-3, "bf16": 6e-2, "i16": 1e-3}
LATS = [(8, 8, 4, 4), (6, 4, 2, 4)]


@pytest.mark.parametrize("prec", list(TOL))
@pytest.mark.parametrize("L5", [8, 12, 16, 28])
@pytest.mark.parametrize("L", LATS, ids=lambda l: "x".join(map(str, l)))
def test_wide_workgroups_bitwise(prec, L5, L, monkeypatch):
    from paper_1810_01609_amd import mdwf as M

    act = M.Action.make(L, L5, 1.5, 0.5, 1.3, 0.05)
    x = S.random_spinor(L, L5, 3, nrhs=2)
    eta = to_dev(x)
    with M.Context(0) as ctx:
        g = ctx.gauge_load(L, S.gauge_field(L, 0.3, 7), precs=("f64", prec))

        def results(lg):
            monkeypatch.setenv("MDWF_CB_LOG2", str(lg))
            outs = []
            for op in ("D", "DDAG", "HOP", "HOPDAG", "MHATDAG", "NORMAL", "PREP"):
                out = empty_like_dev(x.shape)
                ctx.dslash(g, act, getattr(M, "OP_" + op), prec, eta, out, nrhs=2)
                outs.append(to_host(out))
            psi = empty_like_dev(x.shape)
            st = ctx.solve(g, act, M.CGOpts.make(tol=1e-9, inner=prec, max_iter=24), eta, psi, nrhs=2, raise_on_fail=False)
            return outs + [to_host(psi)], [s["iters"] for s in st]

        want, iters = results(4)
        for lg in range(5, 8):
            if (L5 << lg) > 1024:
                break
            log(f"[wide] {L} L5={L5} {prec}: {1 << lg} sites")
            got, its = results(lg)
            assert its == iters
            for a, b in zip(got, want):
                assert np.array_equal(a, b)
        g.free()


@pytest.mark.parametrize("prec", list(TOL))
@pytest.mark.parametrize("L,L5,b5,c5,m5,tap", [((2, 2, 2, 2), 4, 1.5, 0.5, 1.3, 1), ((4, 4, 2, 6), 20, 1.0, 0.0, 1.8, 0),
                                               ((6, 4, 2, 4), 12, 1.5, 0.5, 2.0, 1), ((4, 2, 2, 4), 28, 1.5, 0.5, 1.3, 1),
                                               ((4, 2, 2, 6), 32, 1.25, 0.25, 1.3, 1)])
def test_d_and_prep_at_the_edges(prec, L, L5, b5, c5, m5, tap):
    from paper_1810_01609_amd import mdwf as M

    U = S.gauge_field(L, 0.3, 31)
    act = M.Action.make(L, L5, b5, c5, m5, 0.05, tap)
    oact = O.Action(L, L5, b5, c5, m5, 0.05, t_antiperiodic=bool(tap))
    x = S.random_spinor(L, L5, 41, nrhs=2)
    even = O.parity_mask(oact, 0)
    with M.Context(0) as ctx:
        g = ctx.gauge_load(L, U, precs=("f64", prec))
        for op, ref in (("D", lambda y: O.dirac(U, y, oact)), ("PREP", lambda y: even * O.prep_source(U, y, oact))):
            out = empty_like_dev(x.shape)
            ctx.dslash(g, act, getattr(M, "OP_" + op), prec, to_dev(x), out, nrhs=2)
            got = to_host(out)
            for r in range(2):
                check(got[r], ref(x[r]), TOL[prec], f"{L} L5={L5} {prec} {op} rhs {r}")
        g.free()
