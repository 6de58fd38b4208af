"""Mixed-precision Debye-Hueckel box values of solutes that are long against a Debye length, where an
atom's share of the value falls by many orders of magnitude along a face, and of boxes for which the
interpolation from samples on the faces declines, against FP64 sums over the atoms.

Tolerance, relative to each node's sum of absolute values.  Interpolated: 1e-8, the least that the FP32
sums it replaces are off by (the plan aims at 1e-7 as a bound on the worst arrangement of atoms).  FP32
sums: the exponent kD r and the distance each carry a few roundings of 2^-24, so a term is off by at
most 2^-22 (4 + kD r), r the distance at which the nearest atoms lie, up to sqrt(3) times the margin
and a solute's radius; and by more than 1e-9, which tells them from interpolated values."""
import math

import numpy as np
import pytest

from paper_2502_09323_amd import binding as B
from paper_2502_09323_amd import inputs as I

pytestmark = pytest.mark.gpu


def ball(n, R, rng):
    v = rng.normal(size=(n, 3))
    return v * (R * rng.random(n) ** (1.0 / 3.0) / np.linalg.norm(v, axis=1))[:, None]


def rod(n, half, r, axis, rng):
    d = np.asarray(axis, float) / np.linalg.norm(axis)
    b = ball(n, r, rng)
    return b - np.outer(b @ d, d) + np.outer(rng.uniform(-half, half, n), d)


def pair(n, apart, rng):
    d = 0.5 * np.asarray(apart, float)
    return np.concatenate([ball(n // 2, 27.0, rng) - d, ball(n // 2, 10.0, rng) + d])


# label, atoms, margin to each face, spacing, ionic strength, whether the interpolation runs (None: either)
CASES = [
    ("rod 580 A, 60 A margin", lambda g: rod(12000, 290.0, 12.0, (1, 0, 0), g), 60.0, 1.0, 0.145, True),
    ("rod 580 A, 40 A margin", lambda g: rod(12000, 290.0, 12.0, (0, 1, 0), g), 40.0, 0.8, 0.145, True),
    ("rod 580 A, 60 A margin, 1 M", lambda g: rod(12000, 290.0, 12.0, (1, 0, 0), g), 60.0, 1.0, 1.0, None),
    ("rod 580 A, 30 A margin, 1 M", lambda g: rod(12000, 290.0, 12.0, (0, 0, 1), g), 30.0, 0.8, 1.0, None),
    ("rod across the box, 1 M", lambda g: rod(9000, 120.0, 8.0, (1, 1, 1), g), 25.0, 0.9, 1.0, None),
    ("two clusters", lambda g: pair(10000, (300.0, 0.0, 120.0), g), 30.0, 0.7, 0.145, True),
    ("two clusters, 1 M", lambda g: pair(10000, (300.0, 0.0, 120.0), g), 30.0, 1.0, 1.0, None),
    ("globule", lambda g: ball(20000, 30.0, g), 20.0, 0.6, 1.0, True),
    ("atoms next to the faces", lambda g: ball(20000, 14.0, g), 2.6, 0.5, 0.145, False),
    ("margin of 33 Debye lengths", lambda g: ball(3000, 14.0, g), 100.0, 0.9, 1.0, False),
]


@pytest.mark.parametrize("label,atoms,margin,h,ionic,interp", CASES, ids=[c[0] for c in CASES])
def test_long_solutes_box_values(label, atoms, margin, h, ionic, interp):
    import torch

    rng = np.random.default_rng(11)
    x = np.ascontiguousarray(atoms(rng))
    q = rng.normal(0.0, 0.4, len(x))
    lo, hi = x.min(0), x.max(0)
    origin = lo - margin
    n = tuple(int(math.ceil((hi[d] - lo[d] + 2.0 * margin) / h)) + 1 for d in range(3))
    grid = I.GridSpec(n=n, h=h, origin=tuple(origin), ionic_M=ionic, precision=I.MIXED)
    e, kb, eps0, na = 1.602176634e-19, 1.380649e-23, 8.8541878128e-12, 6.02214076e23
    lb = e * e / (4.0 * math.pi * eps0 * kb * grid.temp_K)
    kd = math.sqrt(8.0 * math.pi * lb * ionic * na * 1e3 / grid.eps_out * 1e-20)
    print(f"box values: {label}, grid {n}, kD {kd:.3f}", flush=True)
    B.load()
    ctx = B.Context(0)
    pb = B.Problem(ctx, I.Molecule(x, np.full(len(x), 1.5), q), grid)
    phi = pb.potential()
    pb.close()
    ctx.close()
    # nodes of the faces, edges among them
    idx = np.stack([rng.integers(0, k, 60000) for k in n], 1)
    ax = rng.integers(0, 3, len(idx))
    idx[np.arange(len(idx)), ax] = rng.integers(0, 2, len(idx)) * (np.array(n)[ax] - 1)
    got = phi[idx[:, 0], idx[:, 1], idx[:, 2]] / (lb * 1e10)
    y = torch.tensor(origin + h * idx, device="cuda")
    X, Q = torch.tensor(x, device="cuda"), torch.tensor(q, device="cuda")
    err = []
    for s in range(0, len(y), 4096):
        r = (y[s:s + 4096, None, :] - X[None]).square().sum(-1).sqrt()
        # relative to the nearest atom's exp(-kD r), so that no sum underflows
        near = r.amin(1, keepdim=True)
        t = torch.exp(-kd * (r - near)) / (grid.eps_out * r)
        v = torch.tensor(got[s:s + 4096], device="cuda") * torch.exp(kd * near[:, 0])
        err.append(((v - t @ Q).abs() / (t @ Q.abs())).cpu().numpy())
    err = np.concatenate(err)
    print(f"largest error of the absolute-value scale {err.max():.1e}", flush=True)
    sums = 2.0 ** -22 * (4.0 + kd * (math.sqrt(3.0) * margin + 30.0))
    assert np.all(np.isfinite(err))
    assert err.max() < (1e-8 if interp else sums)
    if interp is False:
        assert err.max() > 1e-9
