"""Sampled timing of Jacobi-CG in its two forms: on a small grid one launch is a whole iteration, so
there is no update launch to time and its time is 0; with tile_planes given both launches are timed.
pb_time_stencil times the kernel of the form that the problem's solve runs, and a solve after it is
the same as before."""
from dataclasses import replace

import numpy as np
import pytest

from paper_2502_09323_amd import binding as B
from paper_2502_09323_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [I.FP64, I.MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("planes", [0, 32])
def test_profile_of_small_grids(planes, prec):
    mol, grid = I.kirkwood_c1(rtol=1e-9)
    grid = replace(grid, tile_planes=planes, precision=prec, inner_rtol=1e-2)
    B.load()
    ctx = B.Context(0)
    ctx.set_profiling(True)
    pb = B.Problem(ctx, mol, grid)
    first, x = pb.solve(), pb.potential()
    p = pb.profile()
    print(f"tile_planes {planes}: {p}, {first['iters']} iterations", flush=True)
    assert 0 < p["samples"] <= first["iters"] // 8 + 2 and p["stencil_ms"] > 0.0
    assert p["update_ms"] == 0.0 if planes == 0 else p["update_ms"] > 0.0
    for fp32 in (False, True):
        assert pb.time_stencil(5, fp32) > 0.0
    again = pb.solve()
    assert again["iters"] == first["iters"] and np.array_equal(x, pb.potential())
    pb.close()
    ctx.close()
