"""The autotuner's table names the kernel an entry was measured on, and an entry
the launch does not admit is not taken: the call gives what an untuned one gives,
bitwise."""
import numpy as np
import pytest

import mdwf_synth as S
from gpu_util import empty_like_dev, log, to_dev, to_host

pytestmark = pytest.mark.gpu

LAT = (8, 4, 4, 4)


def _normal(M, ctx, L5, prec, x):
    g = ctx.gauge_load(LAT, S.gauge_field(LAT, 0.3, 5), precs=("f64", prec))
    out = empty_like_dev(x.shape)
    ctx.dslash(g, M.Action.make(LAT, L5, 1.5, 0.5, 1.3, 0.05), M.OP_NORMAL, prec, to_dev(x), out)
    got = to_host(out)
    g.free()
    return got


@pytest.mark.parametrize("L5,prec,kernel", [(8, "f64", "general-quads"), (5, "f32", "general"), (8, "f32", "quad")])
def test_entries_beyond_the_limits_are_ignored(tmp_path, L5, prec, kernel):
    from paper_1810_01609_amd import mdwf as M

    x = S.random_spinor(LAT, L5, 9)
    path = tmp_path / "tune.txt"
    with M.Context(0) as ctx:
        want = _normal(M, ctx, L5, prec, x)
        ctx.tune_mode(1)
        assert np.array_equal(_normal(M, ctx, L5, prec, x), want)
        ctx.tune_save(path)
    lines = open(path).read().splitlines()
    hops = [l for l in lines if " h1 " in l]
    assert len(hops) >= 4 and all(l.split()[0] == kernel for l in hops)
    # 128 sites x 8 slices are more threads than FP64 admits; 8 time slices a
    # block and 200 bands divide nothing
    code = 7 | 1 << 8 | 9 << 12 | 200 << 16 if prec != "f64" else 7 | 1 << 8
    with open(path, "w") as f:
        for l in lines:
            f.write(f"{l.split(' | ')[0]} | {code} 0.001\n")
    with M.Context(0) as ctx:
        ctx.tune_load(path)
        assert ctx.tune_entries() == len(lines)
        log(f"[tune] {kernel} {prec}: {ctx.tune_entries()} entries with code {code}")
        got = _normal(M, ctx, L5, prec, x)
    assert np.array_equal(got, want)
