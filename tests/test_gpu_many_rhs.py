"""Calls with so many right-hand sides that their tables fill the 1 MB region
they are uploaded through: they give what one right-hand side at a time gives,
bitwise, or are refused and leave the context usable."""
import numpy as np
import pytest

import mdwf_synth as S
from gpu_util import empty_like_dev, log, to_dev, to_host

pytestmark = pytest.mark.gpu

LAT, L5 = (2, 2, 2, 2), 1


def _context():
    from paper_1810_01609_amd import mdwf as M

    ctx = M.Context(0)
    g = ctx.gauge_load(LAT, S.gauge_field(LAT, 0.3, 2), precs=("f64", "f32"))
    return M, ctx, g, M.Action.make(LAT, L5, 1.5, 0.5, 1.3, 0.1)


def _fields(n):
    rng = np.random.default_rng(n)
    shape = (n, L5) + LAT[::-1] + (4, 3)
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


def test_solve_fills_the_table_region():
    """9361 right-hand sides: the tables of the iteration leave less room than
    one of the final step's would need, were it uploaded too."""
    M, ctx, g, act = _context()
    n = 9361
    x = _fields(n)
    eta, psi = to_dev(x), empty_like_dev(x.shape)
    opts = M.CGOpts.make(tol=1e-9, inner="f32")
    st = ctx.solve(g, act, opts, eta, psi, nrhs=n)
    got = to_host(psi)
    log(f"[many] {n} solves, iterations {min(s['iters'] for s in st)} to {max(s['iters'] for s in st)}")
    assert all(s["converged"] == 1 and s["rel_res_full"] < 1e-7 for s in st)
    for r in (0, 1, 4680, n - 1):
        one = empty_like_dev(x.shape[1:])
        s1 = ctx.solve(g, act, opts, to_dev(x[r]), one)[0]
        assert np.array_equal(to_host(one), got[r])
        assert (s1["iters"], s1["rel_res_full"]) == (st[r]["iters"], st[r]["rel_res_full"])
    with pytest.raises(M.MDWFError) as e:
        ctx.solve(g, act, opts, to_dev(_fields(9400)), empty_like_dev((9400,) + x.shape[1:]), nrhs=9400)
    assert e.value.status == M.EHIP
    ctx.solve(g, act, opts, to_dev(x[0]), one)
    assert np.array_equal(to_host(one), got[0])
    g.free()
    ctx.close()


@pytest.mark.parametrize("call", ["dslash", "hop_split"])
def test_operators_fill_the_table_region(call):
    M, ctx, g, act = _context()

    def run(x, n):
        out = empty_like_dev(x.shape)
        if call == "dslash":
            ctx.dslash(g, act, M.OP_NORMAL, "f64", to_dev(x), out, nrhs=n)
        else:
            ctx.hop_split(g, act, "f64", 12, to_dev(x), out, nrhs=n)
        return to_host(out)

    n = 12000
    x = _fields(n)
    got = run(x, n)
    for r in (0, 5999, n - 1):
        assert np.array_equal(run(x[r], 1), got[r])
    with pytest.raises(M.MDWFError) as e:
        run(_fields(23000), 23000)
    assert e.value.status == M.EHIP
    assert np.array_equal(run(x[0], 1), got[0])
    g.free()
    ctx.close()
