"""Jacobi-CG on grids whose vectors stay in cache (one launch per iteration) against the marching
form, which a given tile_planes selects: the same recurrences with the sums in another order, so
FP64 potentials agree to 1e-8 of the largest at rtol 1e-12 (error of the solves: condition number of
the scaled system, about n^2, times rtol), mixed ones to 1e-5 at rtol 1e-9.  Grids at the edges of
the tiles: one node in the last row, column or plane of tiles; fewer rows than a tile; one, two and
four nodes per thread; a cap on the iterations inside, at the end of and just after a chunk of 16; a
mixed solve whose FP32 residual drifts, so that an update ends inside a chunk and the iteration goes
on at any parity."""
from dataclasses import replace

import numpy as np
import pytest

from paper_2502_09323_amd import binding as B
from paper_2502_09323_amd import inputs as I

pytestmark = pytest.mark.gpu

GRIDS = [(33, 33, 33), (35, 35, 35), (17, 9, 71), (12, 41, 34), (67, 67, 37), (70, 131, 67), (99, 99, 99)]


@pytest.fixture(scope="module")
def ctx():
    B.load()
    c = B.Context(0)
    yield c
    c.close()


def problem(n, prec, **kw):
    h = 0.6
    half = 0.5 * (min(n) - 1) * h
    mol = I.random_molecule(10, max(half - 2.2, 0.5), 5, min_dist=0.3, r_lo=0.8, r_hi=1.2)
    origin = tuple(-0.5 * (v - 1) * h for v in n)
    kw = {"rtol": 1e-12 if prec == I.FP64 else 1e-9, "inner_rtol": 1e-2, **kw}
    return mol, I.GridSpec(n=n, h=h, origin=origin, precision=prec, **kw)


def both(ctx, mol, grid):
    out = []
    for planes in (0, 32):
        pb = B.Problem(ctx, mol, replace(grid, tile_planes=planes))
        st = pb.solve()
        out.append((st, pb.potential()))
        again = pb.solve()
        assert again["iters"] == st["iters"] and np.array_equal(out[-1][1], pb.potential())
        pb.close()
    return out


def close(a, b, tol):
    err = np.abs(a - b).max() / np.abs(b).max()
    print(f"difference {err:.1e} of the largest", flush=True)
    assert err < tol


@pytest.mark.parametrize("prec", [I.FP64, I.MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("n", GRIDS, ids=["x".join(map(str, n)) for n in GRIDS])
def test_small_grids(ctx, n, prec):
    mol, grid = problem(n, prec)
    (s0, x0), (s1, x1) = both(ctx, mol, grid)
    assert s0["status"] == s1["status"] == B.PB_OK
    assert abs(s0["iters"] - s1["iters"]) <= (1 if prec == I.FP64 else 16)
    close(x0, x1, 1e-8 if prec == I.FP64 else 1e-5)


@pytest.mark.parametrize("cap", [1, 15, 16, 17, 40])
def test_iteration_cap(ctx, cap):
    """The same number of steps in both forms: 1e-10 of the largest value after at most 40."""
    mol, grid = problem((35, 21, 37), I.FP64, max_iter=cap)
    (s0, x0), (s1, x1) = both(ctx, mol, grid)
    assert s0["status"] == s1["status"] == B.PB_ENOCONV and s0["iters"] == s1["iters"]
    close(x0, x1, 1e-10)


@pytest.mark.parametrize("rtol", [1e-7, 1e-8, 1e-9, 1e-10, 1e-11])
def test_update_inside_a_chunk(ctx, rtol):
    mol, grid = problem((33, 37, 35), I.MIXED, rtol=rtol, inner_rtol=1e-9)
    (s0, x0), (s1, x1) = both(ctx, mol, grid)
    # so few updates may stall the iteration (ENOCONV); then both forms do
    assert s0["status"] == s1["status"]
    assert s0["status"] == B.PB_ENOCONV or s0["relres"] <= rtol
    assert s0["iters"] <= s1["iters"] + 48
    close(x0, x1, 1e4 * rtol + 1e-6)
