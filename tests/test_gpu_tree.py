"""The energy read-back's sums over cut points by box expansions (large problems) against the
direct sum over the problem's cut points, formed here in FP64 torch.

Tolerance, relative to the sums of absolute values: the expansions are truncated below 3e-14 and
a pair's terms carry the rounding of the squared distance, under 2e-13 for the closest pairs of
these molecules and far less for the others; 1e-13 bounds both."""
import math

import numpy as np
import pytest

from paper_2502_09323_amd import binding as B
from paper_2502_09323_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    B.load()
    c = B.Context(0)
    yield c
    c.close()


def lattice_molecule(inside, half, seed):
    """Jittered lattice points (at least 1 A apart) of the box of half-extents `half` that `inside`
    keeps, with the package's radii and charges."""
    rng = np.random.default_rng(seed)
    ax = [np.arange(-h, h + 1e-9, 2.56) for h in half]
    p = np.stack(np.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 3)
    p = p[inside(p)] + 0.0
    p += rng.uniform(-0.75, 0.75, p.shape)
    q = rng.normal(0.0, 0.4, len(p))
    return I.Molecule(np.ascontiguousarray(p), rng.uniform(1.2, 2.0, len(p)), q - (q.sum() - 1.0) / len(p))


def globule(R, seed):
    return lattice_molecule(lambda p: (p * p).sum(1) < R * R, (R, R, R), seed)


def grid_for(mol, h, pad, center=(0.0, 0.0, 0.0), **kw):
    ext = np.abs(mol.xyz - np.asarray(center)).max(0) + 2.0 + pad
    n = [2 * int(math.ceil(e / h)) + 1 for e in ext]
    org = tuple(float(c) - 0.5 * (k - 1) * h for c, k in zip(center, n))
    return I.GridSpec(n=tuple(n), h=h, origin=org, precision=I.MIXED, rtol=1e-3, inner_rtol=1e-2, bc=I.BC_ZERO, **kw)


def case_globule():
    mol = globule(30.0, 1)                      # 6700 atoms, not a multiple of 64
    return mol, grid_for(mol, 0.5, 2.0)


def case_rod():
    mol = lattice_molecule(lambda p: p[:, 1] ** 2 + p[:, 2] ** 2 < 144.0, (290.0, 12.0, 12.0), 2)
    return mol, grid_for(mol, 0.75, 2.0)


def case_far_from_origin():
    mol = globule(32.0, 3)
    c = (3000.0, -1500.0, 800.0)
    mol = I.shifted(mol, c)
    return mol, grid_for(mol, 0.55, 2.0, center=c)


def case_two_clusters():
    a, b = globule(27.0, 4), globule(27.0, 5)
    d = np.array([0.0, 0.0, 60.0])
    mol = I.Molecule(np.concatenate([a.xyz - d, b.xyz + d]), np.concatenate([a.radius, b.radius]),
                     np.concatenate([a.charge, b.charge]))
    return mol, grid_for(mol, 0.6, 2.0)


def case_refined():
    mol = globule(33.0, 6)
    return mol, grid_for(mol, 1.0, 8.0, refine=1, refine_shell=2.0)


def direct(pb, mol, grid, atoms):
    """phi_reac of the given atoms by direct sums, and the sums of absolute values."""
    import torch

    c = pb.cut(fields=True)
    up = {k: torch.tensor(v, device="cuda") for k, v in c.items()}
    u = up["np"] * (up["wp"] * up["phip"])[:, None]
    e, kb, eps0 = 1.602176634e-19, 1.380649e-23, 8.8541878128e-12
    lb = e * e / (4.0 * math.pi * eps0 * kb * grid.temp_K) * 1e10
    f4 = 1.0 / (4.0 * math.pi)
    phi, scale = [], []
    for a in atoms:
        v = up["rp"] - torch.tensor(mol.xyz[a], device="cuda")
        r = v.square().sum(1).sqrt()
        pol = (1.0 / grid.eps_out - 1.0 / grid.eps_in) * f4
        ion = f4 / grid.eps_out
        sd = (v * u).sum(1) / r ** 3
        phi.append(lb * float(((pol - ion) * up["F"] / r + f4 * sd).sum()))
        scale.append(lb * float(((abs(pol) + ion) * up["F"].abs() / r + f4 * u.norm(dim=1) / r ** 2).sum()))
    return np.array(phi), np.array(scale)


@pytest.mark.parametrize("case", [case_globule, case_rod, case_far_from_origin, case_two_clusters, case_refined])
def test_box_expansions_equal_direct_sum(ctx, case):
    mol, grid = case()
    print(f"box expansions: {case.__name__}, {mol.n} atoms, grid {grid.n}", flush=True)
    pb = B.Problem(ctx, mol, grid)
    assert pb.solve()["status"] == 0
    got = pb.energy(per_atom=True)
    assert mol.n >= 1024 and mol.n * got["n_cut"] >= 2e9      # else the direct sum runs
    again = pb.energy(per_atom=True)
    assert np.array_equal(got["phi_reac"], again["phi_reac"])
    rng = np.random.default_rng(0)
    atoms = np.unique(np.concatenate([[0, mol.n - 1], rng.integers(0, mol.n, 60)]))
    phi, scale = direct(pb, mol, grid, atoms)
    err = np.abs(got["phi_reac"][atoms] - phi) / scale
    print(f"largest error of the absolute-value scale {err.max():.1e}", flush=True)
    assert err.max() < 1e-13
    free = pb.energy_noalloc(per_atom=True)
    assert np.max(np.abs(free["phi_reac"] - got["phi_reac"])) <= 1e-12 * np.max(np.abs(got["phi_reac"]))
    pb.close()
