"""The multigrid's small levels in one block, held in LDS: one V-cycle against the oracle's on
hierarchies at the edges of that form -- its largest first level, a first level that is also the
coarsest, anisotropic levels, several smoothing steps -- element by element, with the tolerances of
the other V-cycle tests (FP64 1e-12, FP32 1e-5 of the largest value)."""
import numpy as np
import pytest

from oracle import mg as M
from paper_2502_09323_amd import binding as B
from paper_2502_09323_amd import inputs as I

pytestmark = pytest.mark.gpu

# nodes per axis, smoothing steps, coarsest sweeps, level cap
CASES = [
    ((41, 41, 41), 1, 4, 0),     # first small level 21^3: the most nodes per thread in FP32
    ((33, 33, 33), 2, 3, 0),     # 17^3: the most per thread in FP64
    ((33, 33, 33), 1, 5, 2),     # the first small level is the coarsest
    ((65, 17, 33), 1, 4, 0),     # anisotropic: 33 x 9 x 17 and below
    ((97, 13, 21), 3, 2, 0),     # ends at 25 x 4 x 6
]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n,nu,cs,levels", CASES, ids=["x".join(map(str, c[0])) + f"-{c[3]}" for c in CASES])
def test_small_levels_vcycle(n, nu, cs, levels, prec):
    h = 0.5
    half = 0.5 * (min(n) - 1) * h
    mol = I.random_molecule(12, max(half - 2.6, 0.6), 31, min_dist=0.3, r_lo=0.8, r_hi=1.2)
    origin = tuple(-0.5 * (v - 1) * h for v in n)
    grid = I.GridSpec(n=n, h=h, origin=origin, precision=I.MIXED if prec == "mixed" else I.FP64, precond=I.MG,
                      mg_smooth=nu, mg_coarse_sweeps=cs, mg_levels=levels, inner_rtol=1e-4)
    r = np.zeros(n)
    r[1:-1, 1:-1, 1:-1] = np.random.default_rng(3).normal(size=tuple(v - 2 for v in n))
    if prec == "mixed":
        r = r.astype(np.float32).astype(np.float64)
    B.load()
    ctx = B.Context(0)
    pb = B.Problem(ctx, mol, grid)
    z, nlev = pb.mg_vcycle(r)
    pb.close()
    ctx.close()
    hier = M.hierarchy(M.fine_level(grid, mol), levels)
    assert len(hier) == nlev
    ref = M.vcycle(hier, r, nu=nu, coarse_sweeps=cs)
    err = np.abs(z - ref).max() / np.abs(ref).max()
    print(f"{n} {prec}: {nlev} levels, difference {err:.1e} of the largest value", flush=True)
    assert err < (1e-12 if prec == "fp64" else 1e-5)
