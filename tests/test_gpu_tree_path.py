"""Which way the energy read-back's sums over cut points go, and the box expansions where a box's points
fill little of it.

With profiling on, a read-back by box expansions reports no pairs of the direct kernel, and one by the
direct sum all of them; the direct sum also takes the shapes for which the boxes would be too large to
gain anything (an atom far from the rest, a sheet across the lattice).  Thin sheets and hollow shells put the cut points of a box into planes and
corners, the patterns for which a box's expansion is least exact.  Tolerance, relative to the sums of
absolute values, as for the other shapes: 1e-13 (terms left out: at most 3e-13 of a box's own sum for
plane patches, a fraction of the whole; a pair's squared distance is rounded to 2e-13 at the worst, for a
few pairs)."""
import math

import numpy as np
import pytest

import test_gpu_tree as T
from paper_2502_09323_amd import binding as B
from paper_2502_09323_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    B.load()
    c = B.Context(0)
    c.set_profiling(True)
    yield c
    c.close()


def with_atoms(mol, xyz, radius=1.5):
    m = len(xyz)
    return I.Molecule(np.ascontiguousarray(np.concatenate([mol.xyz, xyz])),
                      np.concatenate([mol.radius, np.full(m, radius)]),
                      np.concatenate([mol.charge, np.where(np.arange(m) % 2, -0.3, 0.3)]))


def box_grid(mol, h, pad=3.0, **kw):
    """Grid around the balls, not centred at the origin."""
    lo, hi = mol.xyz.min(0) - 2.0 - pad, mol.xyz.max(0) + 2.0 + pad
    n = tuple(16 * math.ceil((hi[d] - lo[d]) / h / 16) + 1 for d in range(3))
    return I.GridSpec(n=n, h=h, origin=tuple(lo), precision=I.MIXED, rtol=1e-3, inner_rtol=1e-2, bc=I.BC_ZERO,
                      precond=I.MG, **kw)


def case_sheet():
    mol = T.lattice_molecule(lambda p: np.abs(p[:, 2]) < 1.0, (110.0, 110.0, 3.0), 7)
    return mol, box_grid(mol, 0.4)


def case_tilted_sheet():
    mol = T.lattice_molecule(lambda p: np.abs(p @ np.array([0.8, 0.36, 0.48])) < 1.6, (80.0, 80.0, 80.0), 8)
    return mol, box_grid(mol, 0.45)


def case_hollow():
    mol = T.lattice_molecule(lambda p: np.abs(np.linalg.norm(p, axis=1) - 60.0) < 2.0, (64.0, 64.0, 64.0), 9)
    return mol, box_grid(mol, 0.45)


def case_crowded():
    """A thousand atoms within 0.05 A: one bin, and one cell, of the curve that orders the atoms."""
    mol = T.globule(30.0, 1)
    x = np.random.default_rng(3).uniform(-0.025, 0.025, (1000, 3)) + np.array([3.0, -2.0, 1.0])
    return with_atoms(mol, x), box_grid(mol, 0.5)


def case_outlier():
    mol = with_atoms(T.globule(46.0, 1), np.array([[400.0, 10.0, -5.0]]))
    return mol, box_grid(mol, 1.0)


def check_sums(pb, mol, grid, got):
    rng = np.random.default_rng(0)
    atoms = np.unique(np.concatenate([[0, mol.n - 1], rng.integers(0, mol.n, 60)]))
    phi, scale = T.direct(pb, mol, grid, atoms)
    err = np.abs(got["phi_reac"][atoms] - phi) / scale
    print(f"largest error of the absolute-value scale {err.max():.1e}", flush=True)
    assert err.max() < 1e-13


EXPANSIONS = [T.case_globule, T.case_rod, T.case_far_from_origin, T.case_two_clusters, T.case_refined, case_sheet,
              case_hollow, case_crowded, case_outlier]


@pytest.mark.parametrize("case", EXPANSIONS)
def test_expansions_run(ctx, case):
    mol, grid = case()
    print(f"box expansions: {case.__name__}, {mol.n} atoms, grid {grid.n}", flush=True)
    pb = B.Problem(ctx, mol, grid)
    assert pb.solve()["status"] == 0
    got = pb.energy(per_atom=True)
    assert pb.energy_profile() == {"nbody_ms": 0.0, "nbody_pairs": 0.0}
    assert np.array_equal(got["phi_reac"], pb.energy(per_atom=True)["phi_reac"])
    check_sums(pb, mol, grid, got)
    if got["n_cut"] < 1.2e6:            # within the scratch of the read-back without allocation
        free = pb.energy_noalloc(per_atom=True)
        assert np.max(np.abs(free["phi_reac"] - got["phi_reac"])) <= 1e-12 * np.max(np.abs(got["phi_reac"]))
    pb.close()


def case_few_pairs():
    mol = T.globule(24.0, 1)
    return mol, box_grid(mol, 0.75)


def case_far_outlier():
    mol = with_atoms(T.globule(46.0, 1), np.array([[2400.0, 10.0, -5.0]]))
    return mol, box_grid(mol, 1.0)


def case_outlier_of_a_small_globule():
    mol = with_atoms(T.globule(28.5, 1), np.array([[800.0, 0.0, 0.0]]))
    return mol, box_grid(mol, 0.5)


@pytest.mark.parametrize("case", [case_few_pairs, case_far_outlier, case_outlier_of_a_small_globule, case_tilted_sheet])
def test_direct_sum_runs(ctx, case):
    mol, grid = case()
    print(f"direct sum: {case.__name__}, {mol.n} atoms, grid {grid.n}", flush=True)
    pb = B.Problem(ctx, mol, grid)
    assert pb.solve()["status"] == 0
    pb.energy()
    got = pb.energy(per_atom=True)
    assert pb.energy_profile()["nbody_pairs"] == float(mol.n) * got["n_cut"]
    assert got["t_energy_s"] < 0.1      # a few milliseconds
    pb.close()


def test_little_work_space(ctx):
    """A read-back without allocation of a problem that nearly fills its scratch: larger boxes or the
    direct sum, the same potentials."""
    mol = T.globule(32.0, 3)
    grid = box_grid(mol, 0.36)
    pb = B.Problem(ctx, mol, grid)
    assert pb.solve()["status"] == 0
    got = pb.energy(per_atom=True)
    assert 1.0e6 < got["n_cut"] < 1.3e6
    free = pb.energy_noalloc(per_atom=True)
    assert np.max(np.abs(free["phi_reac"] - got["phi_reac"])) <= 1e-12 * np.max(np.abs(got["phi_reac"]))
    pb.close()
