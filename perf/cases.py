"""The work that a user has this framework do, as cases whose time and results can be measured.

A case is one call pattern of ``paper_2502_09323_amd.binding``:

- ``solve``: one molecule at a time through ``binding.solve`` (coefficient build, CG solve and
  energy read-back), in the forms the package offers: FP64 (the default) or FP32 with FP64
  reliable updates, Jacobi or multigrid preconditioning, Debye-Hueckel or zero box values,
  uniform or locally refined grids;
- ``readback``: energies and per-atom reaction potentials of a problem that stays resident;
- ``salt``: the salt contribution to the energy from two runs of one geometry, at the actual
  and at zero ionic strength, through the grid energy;
- ``stream``: a burst of requests of mixed sizes through the continuous-batching server.

``listed`` gives the named cases, ``draw`` more of the same ranges, ``prepare`` and ``run`` the
call itself, ``work`` what a pass cannot do without, and ``exact`` the results in plain FP64
torch where they can be had that way.
"""
from __future__ import annotations

import math
from dataclasses import replace

import numpy as np
import torch

from paper_2502_09323_amd import binding as B
from paper_2502_09323_amd import inputs as I

ENERGIES = ("e_coul", "e_pol", "e_ion", "e_solv", "e_total", "q_pol_total", "area_total")


def _case(name, op, atoms, n, h, precision="mixed", precond="mg", rtol=1e-8, smooth=1, bc="dh", ionic=0.145,
          refine=0, shell=3.0):
    nx, ny, nz = (n, n, n) if isinstance(n, int) else n
    c = dict(op=op, atoms=atoms, nx=nx, ny=ny, nz=nz, h=h, precision=precision, precond=precond, rtol=rtol,
             smooth=smooth, bc=bc, ionic=ionic, refine=refine, shell=shell)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the package's smallest use: one charged ball with every option at its default
        _case("sphere_65_fp64", "solve", 1, 65, 0.25, "fp64", "jacobi", 1e-10),
        # a small molecule on a grid that fits no tile, without salt and with zero box values
        _case("ragged_fp64", "solve", 40, (45, 38, 51), 0.6, "fp64", "jacobi", 1e-10, bc="zero", ionic=0.0),
        # requests of the serving stream's smallest, middle and largest grids, one at a time
        _case("request_65_mixed", "solve", 400, 65, 0.75),
        _case("request_129_mixed", "solve", 3000, 129, 0.75),
        _case("request_257_mixed", "solve", 18000, 257, 0.5),
        # the 2000-atom molecule with default options, and the reference-quality multigrid solve
        _case("molecule_161_fp64", "solve", 2000, 161, 0.5, "fp64", "jacobi", 1e-10),
        # the salt contribution of the same molecule from two runs
        _case("salt_161_mixed", "salt", 2000, 161, 0.5),
        # energies and reaction potentials of a resident problem, after a tight FP64 solve
        _case("readback_161_fp64", "readback", 2000, 161, 0.5, "fp64", "mg", 1e-10),
        # the largest single problem, with multigrid and as the Jacobi-CG comparison solve
        _case("large_385_mixed", "solve", 60000, 385, 0.5, smooth=2),
        _case("large_385_jacobi", "solve", 60000, 385, 0.5, precond="jacobi"),
        # one level of refinement near the surface, two-level preconditioner
        _case("refined_193_mixed", "solve", 20000, 193, 1.0, refine=1),
        # a burst of requests of mixed sizes served together
        dict(name="stream_16", op="stream", requests=16, most_atoms=20000, precision="mixed", precond="mg", rtol=1e-8),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _reach(atoms):
    """Half the extent that _molecule may fill, Angstrom."""
    return 20.0 * (atoms / 2000.0) ** (1.0 / 3.0) + 5.0


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "jacobi", "readback", "salt", "refined", "stream"])
    if kind == "stream":
        return dict(op="stream", requests=rng.randint(3, 16), most_atoms=int(_log(rng, 2000, 20000)), precision="mixed",
                    precond="mg", rtol=1e-8)
    # a read-back follows a tight solve, so that its results do not show the solve's tolerance
    precision = "fp64" if kind == "readback" else rng.choice(["mixed", "mixed", "fp64"])
    rtol = 1e-8 if precision == "mixed" else 1e-10
    bc = rng.choice(["dh", "dh", "dh", "zero"])
    ionic = rng.choice([0.145, 0.145, 0.05] if kind == "salt" else [0.145, 0.145, 0.05, 0.0])
    if kind == "refined":
        # 2:1 refinement near the surface, or around the whole solute on a box far from it
        atoms, refine = int(_log(rng, 200, 6000)), rng.choice([1, 2])
        n = 2 * int(_reach(atoms) * (1.2 if refine == 1 else 2.0) / 8 + 1) * 8 + 1
        return _case(None, "solve", atoms, n, 1.0, precision, "mg", rtol, bc="dh" if refine == 1 else "zero",
                     refine=refine, shell=rng.choice([2.0, 3.0]))
    atoms = int(_log(rng, 1, 20000)) if kind != "salt" else int(_log(rng, 50, 4000))
    h = rng.choice([0.5, 0.75, 1.0])
    sides = []
    for _ in range(3):
        least = 2.0 * _reach(atoms) / h
        cells = max(24.0, least * rng.uniform(1.15, 1.8))
        # multigrid coarsens while the cell counts are even; Jacobi takes any count
        cells = 16 * math.ceil(cells / 16) if kind != "jacobi" else int(cells)
        sides.append(min(cells, 288) + 1)
    return _case(None, "solve" if kind == "jacobi" else kind, atoms, tuple(sides), h, precision,
                 "jacobi" if kind == "jacobi" else "mg", rtol, rng.choice([1, 1, 2]), bc, ionic)


def _molecule(atoms, seed):
    """A porous globule of the density of the package's synthetic molecules (2000 atoms in a
    ball of 20 A), centres at least 1 A apart, radii 1.2 to 2 A, partial charges with a net
    charge that is a non-zero integer."""
    rng = np.random.default_rng(seed)
    step, jitter = 2.56, 0.75
    m = int(math.ceil(20.0 * (atoms / 2000.0) ** (1.0 / 3.0) / step)) + 2
    ax = np.arange(-m, m + 1) * step
    p = np.stack(np.meshgrid(ax, ax, ax, indexing="ij"), axis=-1).reshape(-1, 3) + rng.uniform(-0.5, 0.5, 3) * step
    p = p[np.argsort((p * p).sum(1), kind="stable")[:atoms]]
    xyz = p - p.mean(0) + rng.uniform(-jitter, jitter, p.shape)
    charge = rng.normal(0.0, 0.4, atoms)
    net = float(rng.choice([-3.0, -2.0, -1.0, 1.0, 2.0, 3.0]))
    charge += (net - charge.sum()) / atoms
    return I.Molecule(np.ascontiguousarray(xyz), rng.uniform(1.2, 2.0, atoms), charge)


def _problem(case, seed):
    n = (case["nx"], case["ny"], case["nz"])
    h = case["h"]
    grid = I.GridSpec(n=n, h=h, origin=tuple(-0.5 * (v - 1) * h for v in n), ionic_M=case["ionic"],
                      bc={"dh": B.PB_BC_DH, "zero": B.PB_BC_ZERO}[case["bc"]], rtol=case["rtol"],
                      precision={"fp64": B.PB_FP64, "mixed": B.PB_MIXED}[case["precision"]],
                      inner_rtol=1e-2 if case["precond"] == "jacobi" else 1e-4,
                      precond={"jacobi": B.PB_PRECOND_JACOBI, "mg": B.PB_PRECOND_MG}[case["precond"]],
                      mg_smooth=case["smooth"], refine=case["refine"], refine_shell=case["shell"])
    return _molecule(case["atoms"], seed), grid


def _requests(case, seed):
    """Requests with the serving stream's rule: atom counts log-uniform, spacings 0.5 to 1 A,
    grids of 65^3 to 257^3. Sizes come from the case, molecules from the seed."""
    rng = np.random.default_rng(case["requests"] + case["most_atoms"])
    out = []
    for k in range(case["requests"]):
        atoms = int(round(math.exp(rng.uniform(math.log(200.0), math.log(case["most_atoms"])))))
        h = float(rng.choice([0.5, 0.75, 1.0]))
        n = I.serving_sizes(atoms, h)[1]
        grid = I.cubic_grid(n, h, precision=B.PB_MIXED, rtol=case["rtol"], inner_rtol=1e-4, precond=B.PB_PRECOND_MG)
        out.append((_molecule(atoms, 1000 * seed + k), grid))
    return out


class _State:
    """The context (and server or resident problem) that a program keeps, and the inputs."""

    def __init__(self, case, seed):
        self.case = case
        self.ctx = B.Context(0)
        self.server = self.problem = None
        if case["op"] == "stream":
            self.requests = _requests(case, seed)
            self.side = B.Context(0, stream=torch.cuda.Stream(0))
            self.server = B.Server(self.ctx, self.side, max_resident=64)
            return
        self.mol, self.grid = _problem(case, seed)
        if case["op"] == "readback":
            self.problem = B.Problem(self.ctx, self.mol, self.grid)
            self.problem.solve()


def prepare(case, seed):
    return _State(case, seed)


def _energies(r):
    return {k: r[k] for k in ENERGIES} | {"n_cut": r["n_cut"]}


def _grid_energy(state, ionic):
    pb = B.Problem(state.ctx, state.mol, replace(state.grid, ionic_M=ionic))
    status = pb.solve()["status"]
    e = pb.grid_energy()
    pb.close()
    return e, status


def run(state):
    op = state.case["op"]
    if op == "solve":
        r = B.solve(state.mol, state.grid, state.ctx)
        return _energies(r) | {"status": r["status"]}
    if op == "readback":
        r = state.problem.energy(per_atom=True)
        return _energies(r) | {"phi_reac": r["phi_reac"]}
    if op == "salt":
        (g, s), (g0, s0) = _grid_energy(state, state.case["ionic"]), _grid_energy(state, 0.0)
        return {"with_salt": g, "without": g0, "salt": g - g0, "status": s, "status0": s0}
    for k, (mol, grid) in enumerate(state.requests):
        state.server.submit(mol, grid, k)
    done = {}
    while len(done) < len(state.requests):
        state.server.step()
        for r in state.server.poll():
            done[r["id"]] = r
    return [{k: done[i][k] for k in ("e_coul", "e_pol", "e_ion", "n_cut")} for i in range(len(done))]


def work(case):
    """Bytes and operations of a pass: the coefficient map, load and solution of every node once,
    each array element of every CG iteration once (the iteration count from the tolerance and
    the preconditioner's usual rate), atoms and cut points once. The read-back's sums over
    atoms and cut points are counted per atom and per point, not per pair: a pair sum of 1/r
    can be had without visiting every pair."""
    if case["op"] == "stream":
        w = {"bytes": 0.0, "flops": 0.0}
        for mol, grid in _requests(case, 0):
            one = _case(None, "solve", mol.n, grid.n, grid.h)
            for k, v in work(one).items():
                w[k] += v
        return w
    nodes = case["nx"] * case["ny"] * case["nz"]
    e = 8.0 if case["precision"] == "fp64" else 4.0
    digits = math.log(1.0 / case["rtol"])
    if case["precond"] == "mg":
        iters = digits / math.log(2.7 if case["smooth"] == 1 else 4.1)
        per_bytes, per_flops = (24.0 if case["smooth"] == 1 else 38.0) * e + 20.0, 90.0 * case["smooth"] + 30.0
    else:
        iters = 0.06 * digits * max(case["nx"], case["ny"], case["nz"])
        per_bytes, per_flops = 8.0 * e + 4.0, 30.0
    if case["refine"]:
        nodes *= 1.6
    points = 17.8 * case["atoms"] / (case["h"] * (0.5 if case["refine"] else 1.0)) ** 2
    readback = {"bytes": 96.0 * points + 48.0 * case["atoms"], "flops": 40.0 * points + 40.0 * case["atoms"]}
    if case["op"] == "readback":
        return readback
    runs = 2.0 if case["op"] == "salt" else 1.0
    return {"bytes": runs * (20.0 * nodes + iters * per_bytes * nodes) + readback["bytes"],
            "flops": runs * iters * per_flops * nodes + readback["flops"]}


# ---- results in plain FP64 torch ---------------------------------------------------------

def _constants(grid, ionic):
    """Bjerrum length (A) in vacuum units and the squared screening constant (1/A^2)."""
    e, kb, na, eps0 = 1.602176634e-19, 1.380649e-23, 6.02214076e23, 8.8541878128e-12
    lb = e * e / (4.0 * math.pi * eps0 * kb * grid.temp_K)
    return lb * 1e10, 8.0 * math.pi * lb * ionic * na * 1e3 / grid.eps_out * 1e-20


def _distances(y, x):
    """Distances of every point of y to every point of x."""
    r2 = (y[:, None, 0] - x[None, :, 0]).square_()
    for d in (1, 2):
        r2 += (y[:, None, d] - x[None, :, d]).square_()
    return r2.sqrt_()


def _coulomb(mol, grid):
    x = torch.tensor(mol.xyz, device="cuda")
    q = torch.tensor(mol.charge, device="cuda")
    s = 0.0
    for c in range(0, mol.n, 2048):
        d = _distances(x[c:c + 2048], x)
        s += float((q[c:c + 2048, None] * q[None, :] / d).masked_fill_(d == 0, 0.0).sum())
    return 0.5 * _constants(grid, 0.0)[0] * s / grid.eps_in


class _Plain:
    """The discrete problem on a uniform grid, node by node: media, edge weights with the
    harmonic average at the first exit from the union of balls, charges, box values."""

    def __init__(self, mol, grid, ionic):
        self.mol, self.grid = mol, grid
        self.lb, kd2 = _constants(grid, ionic)
        self.kd2 = kd2
        dev = dict(device="cuda", dtype=torch.float64)
        self.x, self.r = torch.tensor(mol.xyz, **dev), torch.tensor(mol.radius, **dev)
        self.q = torch.tensor(mol.charge, **dev)
        n, h = grid.n, grid.h
        self.axes = [grid.origin[d] + h * torch.arange(n[d], **dev) for d in range(3)]
        org = torch.tensor(grid.origin, **dev)
        self.base = torch.floor((self.x - org) / h).long()
        reach = int(math.ceil(float(self.r.max()) / h))
        self.offsets = [(a, b, c) for a in range(-reach, reach + 2) for b in range(-reach, reach + 2)
                        for c in range(-reach, reach + 2)]
        self.solute = torch.zeros(n, dtype=torch.bool, device="cuda")
        flat = self.solute.view(-1)
        for o in self.offsets:
            idx, d, ok = self._around(o)
            flat[idx[ok & ((d * d).sum(1) < self.r * self.r)]] = True
        self._edges()
        self._load()

    def _around(self, o):
        """Node base + o of every atom: flat index, offset from the atom, inside the grid."""
        n = self.grid.n
        ijk = self.base + torch.tensor(o, device="cuda")
        ok = ((ijk >= 0) & (ijk < torch.tensor(n, device="cuda"))).all(1)
        ijk = torch.where(ok[:, None], ijk, torch.zeros_like(ijk))
        d = torch.stack([self.axes[k][ijk[:, k]] for k in range(3)], 1) - self.x
        return (ijk[:, 0] * n[1] + ijk[:, 1]) * n[2] + ijk[:, 2], d, ok

    def _edges(self):
        g, n = self.grid, self.grid.n
        strides = (n[1] * n[2], n[2], 1)
        self.k, self.cut = [], []
        for ax in range(3):
            lo = self.solute.narrow(ax, 0, n[ax] - 1)
            hi = self.solute.narrow(ax, 1, n[ax] - 1)
            k = torch.where(lo, g.eps_in, g.eps_out).double() * g.h
            ijk = torch.nonzero(lo != hi)
            e = (ijk[:, 0] * n[1] + ijk[:, 1]) * n[2] + ijk[:, 2]
            low = self.solute.view(-1)[e]
            s = torch.where(low, e, e + strides[ax])
            dirn = torch.where(low, 1.0, -1.0).double()
            # edges by their solute node: one towards each side along the axis
            at = torch.full((2, self.solute.numel()), -1, dtype=torch.int32, device="cuda")
            at[(~low).long(), s] = torch.arange(len(e), dtype=torch.int32, device="cuda")
            pe, plo, phi = [], [], []
            for o in self.offsets:
                idx, d, ok = self._around(o)
                perp2 = (d * d).sum(1) - d[:, ax] ** 2
                ok = ok & (perp2 < self.r * self.r)
                for side in (0, 1):
                    ed = at[side, idx]
                    sel = ok & (ed >= 0)
                    ed = ed[sel].long()
                    half = torch.sqrt(self.r[sel] ** 2 - perp2[sel])
                    tc = -d[sel, ax] * dirn[ed]
                    pe.append(ed)
                    plo.append(tc - half)
                    phi.append(tc + half)
            pe, plo, phi = torch.cat(pe), torch.cat(plo), torch.cat(phi)
            t = torch.zeros(len(e), device="cuda", dtype=torch.float64)
            while True:
                te = t[pe]
                inside = (plo <= te) & (te < phi)
                tn = t.scatter_reduce(0, pe[inside], phi[inside], "amax")
                if torch.equal(tn, t):
                    break
                t = tn
            t = t.clamp(max=g.h)
            al = t / g.h
            ke = g.h / (al / g.eps_in + (1.0 - al) / g.eps_out)
            k[ijk[:, 0], ijk[:, 1], ijk[:, 2]] = ke
            kijk = torch.stack([s // strides[0], (s // n[2]) % n[1], s % n[2]], 1)
            rp = torch.stack([self.axes[d][kijk[:, d]] for d in range(3)], 1)
            rp[:, ax] += dirn * t
            self.k.append(k)
            self.cut.append((s, torch.where(low, e + strides[ax], e), ke, rp))

    def _load(self):
        g, n = self.grid, self.grid.n
        f = (self.x - torch.tensor(g.origin, device="cuda", dtype=torch.float64)) / g.h
        c = torch.minimum(torch.floor(f).clamp(min=0), torch.tensor(n, device="cuda").double() - 2)
        t, c = f - c, c.long()
        self.corner = []
        b = torch.zeros(self.solute.numel(), device="cuda", dtype=torch.float64)
        for o in range(8):
            bit = torch.tensor([(o >> 2) & 1, (o >> 1) & 1, o & 1], device="cuda")
            w = torch.where(bit.bool(), t, 1.0 - t).prod(1)
            ijk = c + bit
            idx = (ijk[:, 0] * n[1] + ijk[:, 1]) * n[2] + ijk[:, 2]
            self.corner.append((idx, w))
            b.index_add_(0, idx, 4.0 * math.pi * self.q * w)
        self.b = b.view(n)
        self.ionic = torch.where(self.solute, 0.0, g.h ** 3 * g.eps_out * self.kd2).double()
        inner = torch.zeros(n, dtype=torch.bool, device="cuda")
        inner[1:-1, 1:-1, 1:-1] = True
        self.inner = inner
        self.box = torch.zeros(n, device="cuda", dtype=torch.float64)
        if g.bc == B.PB_BC_DH:
            nodes = torch.nonzero(~inner)
            kd = math.sqrt(self.kd2)
            for s in range(0, len(nodes), 1 << 14):
                p = nodes[s:s + (1 << 14)]
                y = torch.stack([self.axes[d][p[:, d]] for d in range(3)], 1)
                v = torch.zeros(len(p), device="cuda", dtype=torch.float64)
                for a in range(0, self.mol.n, 4096):
                    r = _distances(y, self.x[a:a + 4096])
                    v += torch.exp(-kd * r).div_(r) @ self.q[a:a + 4096]
                self.box[p[:, 0], p[:, 1], p[:, 2]] = v / g.eps_out

    def apply(self, p):
        """A p on the inner nodes, p given on all of them."""
        out = self.ionic * p
        for ax in range(3):
            m = p.shape[ax] - 1
            f = self.k[ax] * (p.narrow(ax, 1, m) - p.narrow(ax, 0, m))
            out.narrow(ax, 0, m).sub_(f)
            out.narrow(ax, 1, m).add_(f)
        return out.mul_(self.inner)

    def solve(self, rtol=1e-12):
        diag = self.ionic.clone()
        for ax in range(3):
            m = diag.shape[ax] - 1
            diag.narrow(ax, 0, m).add_(self.k[ax])
            diag.narrow(ax, 1, m).add_(self.k[ax])
        dinv = torch.where(self.inner, 1.0 / diag, 0.0)
        b = self.b * self.inner - self.apply(self.box)
        x, r = torch.zeros_like(b), b.clone()
        z = dinv * r
        p, rz = z.clone(), torch.sum(r * z)
        stop = rtol * rtol * float(torch.sum(b * b))
        for it in range(20000):
            q = self.apply(p)
            al = rz / torch.sum(p * q)
            x.addcmul_(p, al)
            r.addcmul_(q, -al)
            if it % 16 == 15 and float(torch.sum(r * r)) <= stop:
                break
            z = dinv * r
            new = torch.sum(r * z)
            p = torch.addcmul(z, p, new / rz)
            rz = new
        return x + self.box

    def grid_energy(self, phi):
        v = (phi * self.inner).view(-1)
        return 0.5 * self.lb * float(sum(torch.sum(self.q * w * v[idx]) for idx, w in self.corner))

    def polarization(self, phi):
        g, phi = self.grid, phi.view(-1)
        eps = 1.0 / g.eps_out - 1.0 / g.eps_in
        rp = torch.cat([c[3] for c in self.cut])
        f = torch.cat([c[2] * (phi[c[0]] - phi[c[1]]) for c in self.cut])
        pot = torch.zeros(self.mol.n, device="cuda", dtype=torch.float64)
        mid = self.x.mean(0)
        x, y = self.x - mid, rp - mid
        xx, yy = (x * x).sum(1), (y * y).sum(1)
        for a in range(0, len(x), 8192):
            for s in range(0, len(y), 1 << 16):
                r2 = xx[a:a + 8192, None] + yy[None, s:s + (1 << 16)]
                r2 = r2.addmm_(x[a:a + 8192], y[s:s + (1 << 16)].T, alpha=-2.0)
                pot[a:a + 8192] += r2.rsqrt_() @ f[s:s + (1 << 16)]
        return {"e_pol": 0.5 * self.lb * eps / (4.0 * math.pi) * float(torch.sum(self.q * pot)),
                "q_pol_total": eps / (4.0 * math.pi) * float(f.sum()), "n_cut": len(f)}


def exact(case, seed):
    """Coulomb and polarization energies, polarization charge and grid energies in FP64 torch
    from the problem's definition; None where a value needs the marching-cubes areas, a refined
    grid, or too long."""
    if case["op"] == "stream":
        return [{"e_coul": _coulomb(mol, grid), "e_pol": None, "e_ion": None, "n_cut": None}
                for mol, grid in _requests(case, seed)]
    mol, grid = _problem(case, seed)
    if case["op"] == "salt":
        g = [p.grid_energy(p.solve()) for p in (_Plain(mol, grid, c) for c in (case["ionic"], 0.0))]
        return {"with_salt": g[0], "without": g[1], "salt": g[0] - g[1], "status": None, "status0": None}
    out = dict.fromkeys(ENERGIES) | {"n_cut": None, "status" if case["op"] == "solve" else "phi_reac": None}
    out["e_coul"] = _coulomb(mol, grid)
    if not case["refine"]:
        plain = _Plain(mol, grid, case["ionic"])
        out |= plain.polarization(plain.solve())
    return out
