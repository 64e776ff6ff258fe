"""Performance cases: what programs that use the solver have it do.

A program assembles an operator and its preconditioner once per mesh,
velocity model and frequency, keeps that context, and then applies it or
solves with it for many right-hand sides.  The cases follow that: the kept
context is the plan (`prepare` builds it once per process and shares it
between states), the right-hand sides come from the seed.  The setup itself is
a case too, since a frequency sweep or a model update pays for it each time.

Operators are the repository's own (the 4,913-unknown P1 cube, the 8 x 8 x 2 km
thrust model in P2 at 100 m cells and at the serving size) plus boxes of other
sizes, with odd cell counts, other partitions and overlaps among them.

Work: the bytes and floating-point operations a pass cannot do without: every
stored factor entry once per sweep, every matrix entry once (12 bytes: a real
value and a column index), every vector read and written once.
"""
from __future__ import annotations

import itertools
import math
from collections import OrderedDict

import numpy as np
import torch

from paper_2004_06309_amd import helm
from paper_2004_06309_amd import workloads as wl

DEV = "cuda:0"


# ---- the cases ---------------------------------------------------------------

def _op(mesh, nx, ny, nz, order, freq, parts, overlap, two_level, c64):
    return {"mesh": mesh, "nx": nx, "ny": ny, "nz": nz, "order": order, "freq": freq, "px": parts[0],
            "py": parts[1], "pz": parts[2], "overlap": overlap, "two_level": two_level, "c64": c64}


P1_5K = _op("cube", 16, 16, 16, 1, 4.0, (2, 2, 2), 1, False, 0)
MID = _op("thrust", 80, 80, 20, 2, 5.0, (8, 8, 1), 2, True, 0)
MID_C64 = dict(MID, c64=1)
SERVED = _op("thrust", 56, 56, 14, 2, 3.0, (8, 8, 1), 2, True, 1)
ODD = _op("thrust", 41, 37, 13, 2, 2.5, (5, 3, 2), 1, True, 2)
SETUP = _op("thrust", 40, 40, 10, 2, 2.5, (4, 4, 1), 2, True, 0)


def listed():
    return [
        # the smallest call: one local-solve application inside a caller's own Krylov loop; latency of a
        # dozen dependent levels
        {"name": "oras_p1_5k", "kind": "oras", "nrhs": 1, **P1_5K},
        # a whole solve of a small problem: launches, synchronisation and the host's part of every step
        {"name": "solve_p1_5k", "kind": "solve", "nrhs": 1, **P1_5K},
        # the product with A at one million P2 unknowns (residuals, a caller's own Krylov method)
        {"name": "apply_a_p2_1m", "kind": "apply_a", "nrhs": 1, **MID},
        # the coarse correction alone: a chain of short levels between two sparse products
        {"name": "coarse_p2_1m", "kind": "coarse", "nrhs": 1, **MID},
        # the two-level preconditioner, the bulk of every iteration, in complex128
        {"name": "precond_p2_1m", "kind": "precond", "nrhs": 1, **MID},
        # a whole solve for one source: the paper's experiment at the benchmark's size
        {"name": "solve_p2_1m", "kind": "solve", "nrhs": 1, **MID},
        # the preconditioner with complex64 factors (mixed-precision solves)
        {"name": "precond_p2_1m_c64", "kind": "precond", "nrhs": 1, **MID_C64},
        # many sources per operator: 16 in one block Krylov space, complex64 factors
        {"name": "block16_p2_1m_c64", "kind": "block_gmres", "nrhs": 16, **MID_C64},
        # serving: more requests than slots on the 3 Hz serving operator, continuous batching
        {"name": "serve20_p2_370k_c64", "kind": "serve", "nrhs": 20, **SERVED},
        # a few sources advanced together on a box of odd sizes: a block of 5, padded columns, rounded factors
        {"name": "pseudo5_p2_odd", "kind": "pseudo_block", "nrhs": 5, **ODD},
        # the local solves of that box: overlap 1, 30 uneven subdomains
        {"name": "oras_p2_odd", "kind": "oras", "nrhs": 1, **ODD},
        # a new frequency or model: assembly, decomposition, factorisation, and the first application
        {"name": "setup_p2_140k", "kind": "setup", "nrhs": 1, **SETUP},
    ]


def draw(rng):
    kind = rng.choice(["apply_a", "oras", "oras", "coarse", "precond", "precond", "solve", "block_gmres",
                       "pseudo_block", "serve", "setup"])
    order = rng.choice([1, 2, 2, 2])
    # horizontal cells over their logarithm; whole solves and setups stay below the largest listed ones
    top = {"setup": 40, "block_gmres": 64, "pseudo_block": 56, "serve": 48}.get(kind, 80)
    nx = round(math.exp(rng.uniform(math.log(9), math.log(top))))
    ny = max(8, min(top, round(nx * rng.uniform(0.7, 1.3))))
    nz = max(4, round(nx * rng.uniform(0.2, 0.35)))
    if order == 1:  # P1 takes twice the cells per wavelength
        nx, ny, nz = min(2 * nx, 96), min(2 * ny, 96), min(2 * nz, 32)
    cells = 8 if order == 2 else 10
    parts = (max(1, min(8, round(nx / rng.uniform(cells, 2 * cells)))), max(1, min(8, round(ny / rng.uniform(cells, 2 * cells)))),
             2 if nz >= 16 and rng.random() < 0.4 else 1)
    # at least seven nodes per slowest wavelength; cells are 100 m in P2, 50 m in P1
    freq = round(rng.uniform(1.5, 5.0), 2)
    overlap = rng.choice([1, 2, 2, 3])
    two_level = kind == "coarse" or rng.random() < 0.75
    nrhs = 1
    if kind == "block_gmres":
        nrhs = rng.randint(3, 16)
    elif kind == "pseudo_block":
        nrhs = rng.randint(2, 16)
    elif kind == "serve":
        nrhs = rng.randint(5, 24)
    return {"kind": kind, "nrhs": nrhs, **_op("thrust", nx, ny, nz, order, freq, parts, overlap, two_level,
                                              rng.choice([0, 0, 1, 2]))}


# ---- operators (kept by the program) ------------------------------------------

_OP_KEYS = ("mesh", "nx", "ny", "nz", "order", "freq", "px", "py", "pz", "overlap", "two_level", "c64")
_CACHE_BYTES = 150e9  # device memory of the kept operators and their solver work spaces
_meshes: OrderedDict = OrderedDict()
_operators: OrderedDict = OrderedDict()


def _key(case):
    return tuple(case[k] for k in _OP_KEYS)


def _workload(case):
    """Mesh, velocity, partition and coarse mesh of a case (host arrays)."""
    key = _key(case)[:-1]
    if key in _meshes:
        _meshes.move_to_end(key)
        return _meshes[key]
    n = (case["nx"], case["ny"], case["nz"])
    parts = (case["px"], case["py"], case["pz"])
    if case["mesh"] == "cube":
        w = wl.tiny(nx=n[0], n_parts=parts, overlap=case["overlap"], freq=case["freq"])
    else:
        cell = 100.0 if case["order"] == 2 else 50.0
        size = tuple(cell * v for v in n)
        xyz, tets = wl.kuhn_mesh(*n, *size)
        model = wl.ThrustModel.draw(*size, 12, 0)
        c = model.velocity(wl.tet_centroids(xyz, tets)).astype(np.complex128)
        part = wl.box_partition(xyz, tets, parts)
        cx = ct = None
        if case["two_level"]:
            cx, ct = wl.kuhn_mesh(*((v + 1) // 2 for v in n), *size)
        w = wl.Workload("thrust", xyz, tets, case["order"], c, 2 * np.pi * case["freq"], part, int(np.prod(parts)),
                        case["overlap"], cx, ct, None, None)
    _meshes[key] = w
    while len(_meshes) > 6:
        _meshes.popitem(last=False)
    return w


def _operator(case):
    """The assembled and factored context of a case, kept while memory allows."""
    key = _key(case)
    if key not in _operators:
        w = _workload(case)
        h = helm.from_workload(w, device=0, c64=case["c64"])
        st = h.stats()
        size = st["factor_entries"] * (8 if case["c64"] else 16) + 16 * 104 * 16 * h.n
        _operators[key] = (h, st, size)
    _operators.move_to_end(key)
    while len(_operators) > 1 and sum(o[2] for o in _operators.values()) > _CACHE_BYTES:
        _operators.popitem(last=False)  # closed once no state holds it
    return _operators[key][:2]


# ---- inputs, one pass, work ----------------------------------------------------

def _vectors(n, seed, count=1):
    g = torch.Generator(device=DEV).manual_seed(seed)
    shape = (n,) if count == 1 else (count, n)
    return torch.complex(torch.randn(shape, dtype=torch.float64, device=DEV, generator=g),
                         torch.randn(shape, dtype=torch.float64, device=DEV, generator=g))


def _source_points(case, seed, count):
    """Random points at 10 m depth over the middle nine tenths of the top face."""
    w = _workload(case)
    rng = np.random.default_rng(seed)
    ext = w.xyz.max(axis=0)
    xy = rng.uniform(0.05, 0.95, (count, 2)) * ext[:2]
    return np.concatenate([xy, np.full((count, 1), 10.0)], axis=1)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "setup":
        # a perturbed model (a model update): another velocity per seed on the kept mesh
        w = _workload(case)
        rng = np.random.default_rng(seed)
        c = w.c_tet * rng.uniform(0.98, 1.02, w.c_tet.shape)
        h = helm.Helm(0)
        n = h.assemble(w.xyz, w.tets, w.order, w.c_tet, w.omega)
        r = _vectors(n, seed)
        return {"case": case, "h": h, "w": w, "c": c, "r": r, "z": torch.empty_like(r)}
    h, _ = _operator(case)
    state = {"case": case, "h": h, "w": _workload(case)}
    if kind in ("apply_a", "oras", "coarse", "precond"):
        state["r"] = _vectors(h.n, seed)
        state["z"] = torch.empty_like(state["r"])
    else:
        pts = _source_points(case, seed, case["nrhs"])
        b = np.stack([h.point_source(p) for p in pts])
        state["b"] = torch.from_numpy(b[0] if case["nrhs"] == 1 else b).to(DEV)
        state["u"] = torch.zeros_like(state["b"])
    return state


def run(state):
    case, h, w = state["case"], state["h"], state["w"]
    kind = case["kind"]
    if kind in ("apply_a", "oras", "coarse", "precond"):
        r, z = state["r"], state["z"]
        {"apply_a": h.apply_A, "oras": h.apply_oras, "coarse": h.apply_coarse, "precond": h.apply_precond}[kind](r, z)
        return z
    if kind == "setup":
        h.assemble(w.xyz, w.tets, w.order, state["c"], w.omega)
        h.precond_setup(w.part, w.n_sub, w.overlap, w.coarse_xyz, w.coarse_tets, c64=case["c64"])
        h.apply_precond(state["r"], state["z"])
        return state["z"]
    b, u = state["b"], state["u"]
    if kind == "serve":
        srv = helm.Server(h, slots=16, restart=w.restart, tol=w.tol)
        for i in range(case["nrhs"]):
            srv.submit(b[i], u[i], i)
        left = case["nrhs"]
        while left:
            srv.launch()
            left -= len(srv.finish())
        srv.close()
        return u
    kw = {"solve": {}, "block_gmres": {"block": 16, "block_gmres": True}, "pseudo_block": {"block": 16}}[kind]
    h.solve(b, u, tol=w.tol, restart=w.restart, **kw)
    return u


# Arnoldi steps counted for the work of a whole solve: 92 at the benchmark's
# size, fewer on smaller boxes (they grow with the box in wavelengths); block
# steps about two thirds of that.
def _steps(case):
    if case["mesh"] == "cube":
        return 13
    waves = case["freq"] * max(case["nx"], case["ny"]) * (100.0 if case["order"] == 2 else 50.0) / 2000.0
    its = 8 + 4.2 * waves
    return its * (0.65 if case["kind"] == "block_gmres" else 1.0)


def work(case):
    kind = case["kind"]
    if kind == "setup":
        # symbolic sizes only: a host-only context factors nothing
        w = _workload(case)
        h = helm.Helm(-1)
        n = h.assemble(w.xyz, w.tets, w.order, w.c_tet, w.omega)
        nnz = h.matrix_csr()[0][-1]
        h.precond_setup(w.part, w.n_sub, w.overlap, w.coarse_xyz, w.coarse_tets, c64=case["c64"])
        st = h.stats()
        h.close()
        entries = 16 if case["c64"] == 0 else 8
        return {"bytes": float(12 * nnz + 32 * n + 2 * entries * st["factor_entries"]),
                "flops": float(st["factor_flops"] + 8 * st["factor_entries"])}
    h, st = _operator(case)
    n = h.n
    nnz = float(h.matrix_csr()[0][-1]) if kind in ("apply_a", "solve", "block_gmres", "pseudo_block", "serve") else 0.0
    entry = 8 if case["c64"] else 16
    vec = 16.0 * n
    a_bytes, a_flops = 12.0 * nnz, 4.0 * nnz
    local_bytes, local_flops = float(entry * st["factor_entries"]), 8.0 * st["factor_entries"]
    coarse_bytes, coarse_flops = 16.0 * st["coarse_entries"], 8.0 * st["coarse_entries"]
    if st["n_coarse"]:
        coarse_bytes += 2 * 12.0 * 3.4 * n  # Z^T and Z
        coarse_flops += 2 * 4.0 * 3.4 * n
    if kind == "apply_a":
        return {"bytes": a_bytes + 2 * vec, "flops": a_flops}
    if kind == "coarse":
        return {"bytes": coarse_bytes + 2 * vec, "flops": coarse_flops}
    if kind == "oras":
        return {"bytes": local_bytes + 2 * vec, "flops": local_flops}
    pre_bytes, pre_flops = local_bytes + coarse_bytes, local_flops + coarse_flops
    if kind == "precond":
        return {"bytes": pre_bytes + 2 * vec, "flops": pre_flops}
    s = case["nrhs"]
    steps = _steps(case)
    passes = math.ceil(s / 16)
    # one step: operator and factors once per group of 16, two passes over each Krylov basis (mean length
    # min(steps, 50) / 2), the vectors of the step
    basis = min(steps, 50.0) / 2
    step_bytes = passes * (pre_bytes + a_bytes) + s * vec * (2 * basis + 6)
    dots = 16.0 * n * basis * s * (16 if kind == "block_gmres" else 1)
    step_flops = s * (pre_flops + a_flops) + 2 * dots
    return {"bytes": steps * step_bytes, "flops": steps * step_flops}


# ---- the same in 64 bits, from the equations ------------------------------------
#
# Plain finite elements on the case's mesh: (Delta + k^2) u = b with the weak
# form -K + M_{k^2} + i B_k, identity rows and columns at the free surface.

def _poly_tables(order):
    """Lagrange basis of a simplex as polynomials in barycentric coordinates:
    {exponents: coefficient} per function, for `d` + 1 vertices."""
    def tables(nv):
        unit = [tuple(int(i == a) for i in range(nv)) for a in range(nv)]
        if order == 1:
            return [{unit[a]: 1.0} for a in range(nv)]
        out = [{tuple(2 * e for e in unit[a]): 2.0, unit[a]: -1.0} for a in range(nv)]
        for a, b in itertools.combinations(range(nv), 2):
            out.append({tuple(x + y for x, y in zip(unit[a], unit[b])): 4.0})
        return out
    return tables


def _integral(p, q, nv):
    """Integral of p q over a simplex of unit measure."""
    total = 0.0
    for (e, c), (f, d) in itertools.product(p.items(), q.items()):
        m = [x + y for x, y in zip(e, f)]
        total += c * d * math.factorial(nv - 1) * math.prod(math.factorial(x) for x in m) / math.factorial(sum(m) + nv - 1)
    return total


def _derivative(p, i):
    out = {}
    for e, c in p.items():
        if e[i]:
            f = tuple(x - (j == i) for j, x in enumerate(e))
            out[f] = out.get(f, 0.0) + c * e[i]
    return out


class _Elements:
    """Element matrices and connectivity of a workload, on the GPU."""

    def __init__(self, w):
        order = w.order
        tables = _poly_tables(order)
        vol, tri = tables(4), tables(3)
        M = torch.tensor([[_integral(p, q, 4) for q in vol] for p in vol], dtype=torch.float64, device=DEV)
        D = [[_derivative(p, i) for i in range(4)] for p in vol]
        self.K_ref = torch.tensor([[[[_integral(D[a][i], D[b][j], 4) for j in range(4)] for i in range(4)]
                                    for b in range(len(vol))] for a in range(len(vol))],
                                  dtype=torch.float64, device=DEV)
        self.M_ref = M
        self.B_ref = torch.tensor([[_integral(p, q, 3) for q in tri] for p in tri], dtype=torch.float64, device=DEV)
        self.nv = w.xyz.shape[0]
        tets = np.asarray(w.tets)
        pairs = list(itertools.combinations(range(4), 2))
        self.n = self.nv
        dofs = tets
        self.edge_keys = None
        if order == 2:
            lo = np.stack([np.minimum(tets[:, a], tets[:, b]) for a, b in pairs], axis=1)
            hi = np.stack([np.maximum(tets[:, a], tets[:, b]) for a, b in pairs], axis=1)
            self.edge_keys, inv = np.unique((lo * self.nv + hi).ravel(), return_inverse=True)
            dofs = np.concatenate([tets, self.nv + inv.reshape(lo.shape)], axis=1)
            self.n += self.edge_keys.size
        self.tets, self.order, self.w = tets, order, w
        self.dofs = torch.from_numpy(np.ascontiguousarray(dofs)).to(DEV)
        x = torch.from_numpy(w.xyz).to(DEV)[torch.from_numpy(tets).to(DEV)]
        e = (x[:, 1:] - x[:, :1]).transpose(1, 2)  # columns: edges from vertex 0
        self.vol = torch.linalg.det(e).abs() / 6
        g = torch.linalg.inv(e)  # rows: gradients of barycentric 1..3
        self.grad = torch.cat([-g.sum(dim=1, keepdim=True), g], dim=1)
        self.k = w.omega / torch.from_numpy(np.asarray(w.c_tet)).to(DEV)
        f = np.concatenate([np.sort(np.delete(tets, i, axis=1), axis=1) for i in range(4)])
        self.faces, self.face_owner = f, np.tile(np.arange(tets.shape[0]), 4)
        self.face_key = (f[:, 0] * self.nv + f[:, 1]) * self.nv + f[:, 2]
        _, first, count = np.unique(self.face_key, return_index=True, return_counts=True)
        bnd = first[count == 1]
        top = (w.xyz[f[bnd], 2] == w.xyz[:, 2].min()).all(axis=1)
        self.absorbing = bnd[~top]
        self.fixed = torch.zeros(self.n, dtype=torch.bool, device=DEV)
        self.fixed[self.face_dofs(f[bnd[top]]).ravel()] = True

    def face_dofs(self, f):
        cols = [f]
        if self.order == 2:
            key = np.stack([f[:, a] * self.nv + f[:, b] for a, b in itertools.combinations(range(3), 2)], axis=1)
            cols.append(self.nv + np.searchsorted(self.edge_keys, key))
        return torch.from_numpy(np.concatenate(cols, axis=1)).to(DEV)

    def blocks(self, lo, hi):
        """Element matrices -K + k^2 M of tets lo..hi."""
        g = torch.matmul(self.grad[lo:hi], self.grad[lo:hi].transpose(1, 2).contiguous())
        m = self.K_ref.shape[0]
        K = torch.matmul(g.reshape(-1, 16), self.K_ref.reshape(m * m, 16).t().contiguous()).reshape(-1, m, m)
        v = self.vol[lo:hi, None, None]
        return (self.k[lo:hi, None, None] ** 2) * (v * self.M_ref) - v * K

    def face_blocks(self, idx):
        f = self.faces[idx]
        x = self.w.xyz[f]
        area = np.linalg.norm(np.cross(x[:, 1] - x[:, 0], x[:, 2] - x[:, 0]), axis=1) / 2
        k = self.k[torch.from_numpy(self.face_owner[idx]).to(DEV)]
        return self.face_dofs(f), 1j * (k * torch.from_numpy(area).to(DEV))[:, None, None] * self.B_ref

    def product(self, x):
        """A x, element by element."""
        x0 = torch.where(self.fixed, 0, x)
        y = torch.zeros_like(x)
        for lo in range(0, self.dofs.shape[0], 1 << 17):
            hi = min(lo + (1 << 17), self.dofs.shape[0])
            d = self.dofs[lo:hi]
            y.index_add_(0, d.reshape(-1), (self.blocks(lo, hi) * x0[d][:, None, :]).sum(dim=2).reshape(-1))
        d, B = self.face_blocks(self.absorbing)
        y.index_add_(0, d.reshape(-1), (B * x0[d][:, None, :]).sum(dim=2).reshape(-1))
        return torch.where(self.fixed, x, y)

    def dense(self, tet_ids=None, extra_faces=None):
        """The matrix over all tets, or of a set of tets with impedance on
        its artificial faces; (matrix, its dofs)."""
        if tet_ids is None:
            tet_ids, faces = np.arange(self.tets.shape[0]), self.absorbing
        else:
            faces = extra_faces
        t = torch.from_numpy(tet_ids).to(DEV)
        dofs = torch.unique(self.dofs[t])
        where = torch.full((self.n,), -1, dtype=torch.int64, device=DEV)
        where[dofs] = torch.arange(dofs.numel(), device=DEV)
        m = dofs.numel()
        A = torch.zeros(m * m, dtype=torch.complex128, device=DEV)

        def add(d, blk):
            d = where[d]
            A.index_add_(0, (d[:, :, None] * m + d[:, None, :]).reshape(-1), blk.reshape(-1))

        for part in torch.split(t, 1 << 14):
            lo = int(part[0])
            if int(part[-1]) - lo + 1 == part.numel():
                add(self.dofs[part], self.blocks(lo, lo + part.numel()))
            else:
                add(self.dofs[part], self.blocks(0, self.dofs.shape[0])[part])
        add(*self.face_blocks(faces))
        A = A.reshape(m, m)
        fixed = self.fixed[dofs]
        A[fixed, :] = 0
        A[:, fixed] = 0
        A[fixed, fixed] = 1
        return A, dofs

    def oras(self, r, overlap):
        """sum_i R_i^T D_i A_i^{-1} R_i r with dense local matrices."""
        w = self.w
        _, inv, count = np.unique(self.face_key, return_inverse=True, return_counts=True)
        bnd = count[inv.ravel()] == 1
        absorbing = np.zeros(self.faces.shape[0], dtype=bool)
        absorbing[self.absorbing] = True
        locals_, weight = [], torch.zeros(self.n, dtype=torch.float64, device=DEV)
        dofs_np = self.dofs.cpu().numpy()
        for i in range(w.n_sub):
            inside = np.asarray(w.part) == i
            layer = np.full(self.n, overlap + 1)
            layer[dofs_np[inside].ravel()] = 0
            for step in range(1, overlap + 1):
                touched = np.zeros(self.nv, dtype=bool)
                touched[self.tets[inside].ravel()] = True
                inside = touched[self.tets].any(axis=1)
                ids = np.unique(dofs_np[inside])
                layer[ids] = np.minimum(layer[ids], step)
            own = inside[self.face_owner]
            _, finv, fcount = np.unique(self.face_key[own], return_inverse=True, return_counts=True)
            idx = np.nonzero(own)[0]
            single = idx[fcount[finv.ravel()] == 1]
            faces = single[absorbing[single] | ~bnd[single]]
            A, dofs = self.dense(np.nonzero(inside)[0], faces)
            chi = torch.clamp(1 - torch.from_numpy(layer).to(DEV)[dofs].double() / overlap, min=0)
            weight[dofs] += chi
            locals_.append((A, dofs, chi))
        z = torch.zeros_like(r)
        for A, dofs, chi in locals_:
            z[dofs] += (chi / weight[dofs]) * torch.linalg.solve(A, r[dofs])
        return z


def exact(case, seed):
    kind = case["kind"]
    points = case["nx"] * case["ny"] * case["nz"] * (8 if case["order"] == 2 else 1)
    if kind == "apply_a":
        w = _workload(case)
        state = prepare(case, seed)
        return _Elements(w).product(state["r"])
    if points > 8000:
        return None  # dense matrices would not fit the time
    if kind == "oras":
        state = prepare(case, seed)
        return _Elements(state["w"]).oras(state["r"], case["overlap"])
    if kind in ("solve", "block_gmres", "pseudo_block", "serve"):
        state = prepare(case, seed)
        A, _ = _Elements(state["w"]).dense()
        b = state["b"]
        u = torch.linalg.solve(A, b.reshape(case["nrhs"], -1).t().contiguous())
        return u.t().contiguous().reshape(b.shape)
    return None
