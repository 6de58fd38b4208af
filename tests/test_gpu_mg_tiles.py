"""Level-0 multigrid passes on grids whose tiles just fill, overfill and underfill the rounds of tile
runs dealt to the XCDs (512 tiles a round), with and without salt (the diagonal of an uncut node is
formed, not loaded): one V-cycle against the oracle's, element by element, with the tolerances of the
other V-cycle tests (FP64 1e-12, FP32 1e-5 of the largest value)."""
import numpy as np
import pytest

from oracle import mg as M
from paper_2502_09323_amd import binding as B
from paper_2502_09323_amd import inputs as I

pytestmark = pytest.mark.gpu

CASES = [   # nodes per axis, ionic strength; tiles
    ((129, 65, 65), 0.145),   # 512
    ((131, 65, 65), 0.0),     # 520
    ((67, 65, 131), 0.5),     # 660
    ((65, 65, 65), 0.0),      # 256
]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n,salt", CASES, ids=["x".join(map(str, c[0])) for c in CASES])
def test_level0_tiles_vcycle(n, salt, prec):
    h = 0.4
    mol = I.random_molecule(60, 0.5 * (min(n) - 1) * h - 3.0, 17, min_dist=0.6, r_lo=1.0, r_hi=1.6)
    origin = tuple(-0.5 * (v - 1) * h for v in n)
    grid = I.GridSpec(n=n, h=h, origin=origin, precision=I.MIXED if prec == "mixed" else I.FP64, precond=I.MG,
                      ionic_M=salt, inner_rtol=1e-4)
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
    hier = M.hierarchy(M.fine_level(grid, mol), 0)
    assert len(hier) == nlev
    ref = M.vcycle(hier, r, nu=grid.mg_smooth, coarse_sweeps=grid.mg_coarse_sweeps)
    err = np.abs(z - ref).max() / np.abs(ref).max()
    print(f"{n} {prec}: {nlev} levels, difference {err:.1e} of the largest value", flush=True)
    assert err < (1e-12 if prec == "fp64" else 1e-5)
