"""The refined solve's passes over both grids (operator with its sums, residual, restriction,
prolongation) where the fine sub-lattice starts at odd and even coarse cells and reaches close to the
box, with bricks of one to five cells and a solute out of the centre: two-level and Jacobi solves of
the composite system, FP64 and mixed, against the oracle's refined run.  Tolerances as for the other
refined cases: energies 1e-10 in FP64 (rtol 1e-12), 1e-6 in mixed precision (rtol 1e-8); in FP64 with
the two-level form the oracle's own iteration count, one step more or less."""
from dataclasses import replace

import numpy as np
import pytest

from oracle import refined as R
from paper_2502_09323_amd import binding as B
from paper_2502_09323_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    B.load()
    c = B.Context(0)
    yield c
    c.close()


CASES = [   # nodes, displacement of the solute, refine, shell, brick
    ((25, 21, 27), (0.0, 0.0, 0.0), 1, 0.6, 1),
    ((25, 27, 23), (1.3, -0.9, 0.7), 1, 1.0, 1),
    ((23, 25, 33), (-0.2, 0.8, -2.2), 1, 1.0, 3),
    ((27, 25, 25), (0.9, 0.4, -0.6), 1, 2.4, 2),     # refined cells next to the box's layer
    ((27, 26, 32), (0.3, -0.4, 2.3), 2, 0.7, 5),
]


@pytest.mark.parametrize("prec", [I.FP64, I.MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("n,shift,mode,shell,brick", CASES)
def test_refined_odd_offsets(ctx, n, shift, mode, shell, brick, prec):
    mol = I.random_molecule(12, 2.0, 21, min_dist=0.4, r_lo=0.8, r_hi=1.3)
    mol = replace(mol, xyz=mol.xyz + np.array(shift))
    h = 0.6
    grid = I.GridSpec(n=n, h=h, origin=tuple(-0.5 * (v - 1) * h for v in n), refine=mode, refine_shell=shell,
                      refine_brick=brick, precision=prec, rtol=1e-12 if prec == I.FP64 else 1e-8, inner_rtol=1e-2)
    ref = R.refined_run(mol, replace(grid, precision=I.FP64), delta=shell, brick=brick, rtol=1e-12,
                        mode="box" if mode == 2 else "surface", solver="mg")
    for pre in (I.MG, I.JACOBI):
        pb = B.Problem(ctx, mol, replace(grid, precond=pre))
        st = pb.solve()
        en = pb.energy()
        assert st["status"] == B.PB_OK
        np.testing.assert_array_equal(pb.refined_cells().astype(bool), ref.refined)
        pb.close()
        if pre == I.MG and prec == I.FP64:
            assert abs(st["iters"] - ref.iters) <= 1, (st["iters"], ref.iters)
        tol = 1e-10 if prec == I.FP64 else 1e-6
        print(n, pre, st["iters"], abs(en["e_pol"] / ref.energy["e_pol"] - 1), flush=True)
        for k in ("e_pol", "e_coul"):
            assert abs(en[k] - ref.energy[k]) <= tol * abs(ref.energy[k]), k
