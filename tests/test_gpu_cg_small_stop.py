"""Jacobi-CG on grids whose vectors stay in cache: what a solve leaves when it stops inside a chunk of
launches.  The launches after the stopping one must leave the solution alone, so a solve that converges
after k iterations holds, bit for bit, what a solve with an unreachable tolerance capped at k + 1
iterations holds (the launch that finds the residual of iterate k small has applied steps 0 to k - 1,
as the capped solve has).  Grids of one block, of fewer blocks than the device takes at once and of
several rounds of them, and tolerances that put the stop at many places in a chunk, its first and last
launches among them.  Mixed solves stop once per update: two runs give the same bits."""
from dataclasses import replace

import numpy as np
import pytest

from paper_2502_09323_amd import binding as B
from paper_2502_09323_amd import inputs as I

pytestmark = pytest.mark.gpu

GRIDS = [(9, 5, 19), (33, 33, 33), (67, 41, 70), (145, 131, 129)]


@pytest.fixture(scope="module")
def ctx():
    B.load()
    c = B.Context(0)
    yield c
    c.close()


def problem(n, prec, **kw):
    h = 0.6
    half = 0.5 * (min(n) - 1) * h
    r = min(1.2, 0.5 * half)
    mol = I.Molecule(np.zeros((1, 3)), np.array([0.6 * r]), np.array([1.0])) if half < 3.0 else \
        I.random_molecule(10, half - 2.2, 5, min_dist=0.3, r_lo=0.8, r_hi=1.2)
    return mol, I.GridSpec(n=n, h=h, origin=tuple(-0.5 * (v - 1) * h for v in n), precision=prec, **kw)


def solved(ctx, mol, grid):
    pb = B.Problem(ctx, mol, grid)
    st = pb.solve()
    x = pb.potential()
    pb.close()
    return st, x


@pytest.mark.parametrize("n", GRIDS, ids=["x".join(map(str, n)) for n in GRIDS])
def test_stop_leaves_the_solution(ctx, n):
    places = set()
    for k in range(24):
        mol, grid = problem(n, I.FP64, rtol=10.0 ** (-1.0 - 0.4 * k))
        st, x = solved(ctx, mol, grid)
        assert st["status"] == B.PB_OK and st["relres"] <= grid.rtol
        capped, y = solved(ctx, mol, replace(grid, rtol=1e-200, max_iter=st["iters"] + 1))
        assert capped["status"] == B.PB_ENOCONV
        assert np.array_equal(x, y), (n, grid.rtol, st["iters"])
        places.add(st["iters"] % 16)
    print(n, "stops at", sorted(places), flush=True)
    assert len(places) >= 4


@pytest.mark.parametrize("n", GRIDS[1:], ids=["x".join(map(str, n)) for n in GRIDS[1:]])
def test_mixed_runs_agree(ctx, n):
    mol, grid = problem(n, I.MIXED, rtol=1e-9, inner_rtol=3e-2)
    runs = [solved(ctx, mol, grid) for _ in range(3)]
    assert runs[0][0]["status"] == B.PB_OK
    for st, x in runs[1:]:
        assert st["iters"] == runs[0][0]["iters"] and np.array_equal(x, runs[0][1])
