"""Performance cases: the work that programs using this solver have it do, through
the Python binding's entry points (Solver, PackedSolver).

Four kinds of case:
  solve    one right-hand side on device tensors with a handle the program keeps
           (a load-step or design loop: setup once, many solves);
  block    several load cases at once (option block_rhs);
  packed   many small independent problems solved as one (a batch of requests);
  request  a new mesh from host arrays: setup on the device, solve, free (what one
           request of the serving stream costs its user).

Meshes are structured and jittered (or graded towards a corner), triangles in 2D
and six Kuhn tetrahedra per cube in 3D, with the material ranges of the repository's
workloads: E = 1 or {1, 100} on a checkerboard, nu 0.3 to 0.49. Loads are smooth
nodal forces. Everything random comes from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2505_09064_amd import vasmg as V


def listed():
    return [
        # a small plane-strain model in FP64 with every option at its default:
        # one solve is launch latency and the host round trips of its iterations
        dict(name="small2d_fp64", kind="solve", nx=33, ny=33, nz=1, graded=False, mix=False,
             nu=0.3, fix="boundary", precision="fp64", autotune=0, rtol=1e-6),
        # a small 3D part of the serving stream, FP32 V-cycle, ragged sizes
        dict(name="small3d_mixed", kind="solve", nx=12, ny=9, nz=11, graded=False, mix=True,
             nu=0.35, fix="x0", precision="mixed", autotune=0, rtol=1e-6),
        # a mid-size 2D model with two materials
        dict(name="mid2d_mixed", kind="solve", nx=247, ny=230, nz=1, graded=False, mix=True,
             nu=0.4, fix="boundary", precision="mixed", autotune=0, rtol=1e-6),
        # a mid-size 3D part on symmetry planes (rollers), tighter tolerance
        dict(name="mid3d_mixed", kind="solve", nx=31, ny=27, nz=34, graded=False, mix=True,
             nu=0.3, fix="symmetry", precision="mixed", autotune=0, rtol=1e-8),
        # the benchmark's 65^3 workload as the benchmark runs it (lanes autotuned)
        dict(name="bench3d_mixed", kind="solve", nx=65, ny=65, nz=65, graded=False, mix=False,
             nu=0.3, fix="x0", precision="mixed", autotune=1, rtol=1e-6),
        # the same in FP64 throughout, as a program gets it without asking for more
        dict(name="bench3d_fp64", kind="solve", nx=65, ny=65, nz=65, graded=False, mix=False,
             nu=0.3, fix="x0", precision="fp64", autotune=0, rtol=1e-6),
        # the largest single-column solve here: 2.7 million DOFs, sizes off the powers of two
        dict(name="large3d_mixed", kind="solve", nx=97, ny=92, nz=99, graded=False, mix=False,
             nu=0.3, fix="x0", precision="mixed", autotune=0, rtol=1e-6),
        # nearly incompressible graded 2D model with 1:100 materials: many levels, many iterations
        dict(name="graded2d_mixed", kind="solve", nx=513, ny=513, nz=1, graded=True, mix=True,
             nu=0.49, fix="boundary", precision="mixed", autotune=0, rtol=1e-6),
        # sixteen load cases on the 65^3 mesh, all columns in one block
        dict(name="block16_mixed", kind="block", nx=65, ny=65, nz=65, K=16, n_rhs=16, mix=False,
             nu=0.3, fix="x0", precision="mixed", autotune=0, rtol=1e-6),
        # a few load cases on a small part in FP64; the last block is not full
        dict(name="block4_fp64", kind="block", nx=23, ny=30, nz=26, K=4, n_rhs=6, mix=True,
             nu=0.3, fix="x0", precision="fp64", autotune=0, rtol=1e-6),
        # a batch of small 3D requests packed into one solve (ten, as the server packs them)
        dict(name="packed3d_mixed", kind="packed", lo=5, hi=14, parts=10, dim=3, mix=True, nu=0.35,
             precision="mixed", rtol=1e-6),
        # one request of the serving stream: a new 3D mesh, set up, solved and freed
        dict(name="request3d_mixed", kind="request", nx=41, ny=44, nz=38, graded=False, mix=True,
             nu=0.35, fix="x0", precision="mixed", autotune=0, rtol=1e-6),
    ]


def _box(rng, dim, lo_dofs, hi_dofs):
    """Ragged box sizes whose DOFs are log-uniform in [lo_dofs, hi_dofs]."""
    n = (math.exp(rng.uniform(math.log(lo_dofs), math.log(hi_dofs))) / dim) ** (1.0 / dim)
    s = [max(5, int(round(n * rng.uniform(0.85, 1.15)))) for _ in range(dim)]
    return dict(nx=s[0], ny=s[1], nz=s[2] if dim == 3 else 1)


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "solve", "block", "block", "packed", "request"])
    mat = dict(mix=rng.random() < 0.5, nu=round(rng.uniform(0.25, 0.45), 3))
    prec = dict(precision=rng.choice(["mixed", "mixed", "fp64"]))
    if kind == "packed":
        dim = rng.choice([2, 3])
        lo = rng.randint(5, 9) if dim == 3 else rng.randint(8, 20)
        return dict(kind=kind, lo=lo, hi=lo + rng.randint(3, 8), parts=rng.randint(3, 10), dim=dim,
                    rtol=1e-6, **mat, **prec)
    dim = rng.choice([2, 3, 3])
    fix = dict(fix=rng.choice(["boundary", "x0", "symmetry"] if dim == 2 else ["x0", "x0", "symmetry"]))
    if kind == "block":
        K = rng.choice([4, 8, 16])
        return dict(kind=kind, K=K, n_rhs=rng.randint(2, K + K // 2), autotune=0, rtol=1e-6,
                    **_box(rng, dim, 1e3, 3e5), **mat, **prec, **fix)
    box = _box(rng, dim, 1e3, 1.2e6 if kind == "solve" else 2.5e5)
    graded = kind == "solve" and dim == 2 and rng.random() < 0.4
    if graded:
        box = {k: min(v, 401) for k, v in box.items()}
        fix = dict(fix="boundary")
    return dict(kind=kind, graded=graded, autotune=0, rtol=rng.choice([1e-6, 1e-6, 1e-8]), **box,
                **mat, **prec, **fix)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
_KUHN = [(0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)]


class _Mesh:
    """Host arrays of one mesh and its load vectors, as a program would hand them over."""

    def __init__(self, nx, ny, nz, mix, nu, fix, seed, graded=False, n_rhs=1):
        rng = np.random.default_rng([seed, nx, ny, nz])
        dim = 2 if nz == 1 else 3
        shape = (nx, ny, nz)[:dim]
        h = 1.0 / (max(shape) - 1)
        idx = np.indices(shape[::-1])[::-1].reshape(dim, -1)          # x fastest
        if graded:
            t = idx / (np.array(shape)[:, None] - 1.0)
            coords = np.ascontiguousarray((t * t).T)
        else:
            coords = np.ascontiguousarray((idx * h).T)
        bnd = ((idx == 0) | (idx == np.array(shape)[:, None] - 1)).any(axis=0)
        if not graded:
            J = rng.uniform(-0.2 * h, 0.2 * h, size=coords.shape)
            J[bnd] = 0.0
            coords += J
        stride = np.array([1, nx, nx * ny])[:dim]
        cells = np.indices(tuple(s - 1 for s in shape[::-1]))[::-1].reshape(dim, -1)
        base = (stride[:, None] * cells).sum(axis=0).astype(np.int32)
        if dim == 2:
            tets = [(0, 1, 1 + nx), (0, 1 + nx, nx)]
        else:
            tets = []
            for p in _KUHN:                                           # paths along the axes in order p
                o = [0]
                for a in p:
                    o.append(o[-1] + int(stride[a]))
                if p in ((0, 2, 1), (1, 0, 2), (2, 1, 0)):
                    o[2], o[3] = o[3], o[2]
                tets.append(tuple(o))
        self.dim, self.shape = dim, shape
        self.coords = coords
        self.elems = np.ascontiguousarray(
            np.stack([base[:, None] + np.array(t, dtype=np.int32) for t in tets], axis=1).reshape(-1, dim + 1))
        ne = self.elems.shape[0]
        if mix:
            table = np.where(rng.random((8 if graded else 4,) * dim) < 0.5, 100.0, 1.0)
            g = table.shape[0]
            b = tuple(np.minimum(cells[a] * g // max(shape[a] - 1, 1), g - 1) for a in range(dim))
            self.E = np.repeat(table[b], len(tets))
        else:
            self.E = np.ones(ne)
        self.nu = np.full(ne, nu)
        fixed = np.zeros(coords.shape, dtype=np.uint8)
        if fix == "boundary":
            fixed[bnd] = 1
        elif fix == "x0":
            fixed[idx[0] == 0] = 1
        else:                                                         # rollers on the planes x_a = 0
            for a in range(dim):
                fixed[idx[a] == 0, a] = 1
        self.fixed = fixed
        # smooth nodal forces: a constant body force and three sine modes a component
        t = idx / (np.array(shape)[:, None] - 1.0)
        S = [np.sin(np.pi * np.arange(1, 4)[:, None] * t[a]) for a in range(dim)]
        rhs = np.empty((n_rhs,) + coords.shape)
        for r in range(n_rhs):
            for a in range(dim):
                f = np.full(coords.shape[0], rng.normal())
                for _ in range(3):
                    m = rng.normal() * S[0][rng.integers(3)]
                    for c in range(1, dim):
                        m = m * S[c][rng.integers(3)]
                    f += m
                rhs[r, :, a] = f * h ** dim
        self.rhs = rhs


def _mesh_of(case, seed):
    return _Mesh(case["nx"], case["ny"], case["nz"], case["mix"], case["nu"], case["fix"], seed,
                 case.get("graded", False), case.get("n_rhs", 1))


def _parts_of(case, seed):
    """The packed problems: ragged sizes from the case and the part's number, values from the seed."""
    r = np.random.default_rng([case["lo"], case["hi"], case["parts"], case["dim"]])
    out = []
    for k in range(case["parts"]):
        s = [int(v) for v in r.integers(case["lo"], case["hi"] + 1, size=3)]
        if case["dim"] == 2:
            s[2] = 1
        out.append(_Mesh(*s, case["mix"], case["nu"], "x0" if k % 3 else "symmetry", 1000 * seed + k))
    return out


def _prec(case):
    return V.FP32_PRECOND if case["precision"] == "mixed" else V.FP64


def prepare(case, seed):
    kind = case["kind"]
    if kind == "packed":
        ms = _parts_of(case, seed)
        parts = [V.Solver.from_mesh(m, precision=_prec(case), host_only=1) for m in ms]
        rhs = torch.from_numpy(np.concatenate([m.rhs[0] for m in ms])).cuda()
        return dict(case=case, solver=V.PackedSolver(parts), parts=parts, rhs=rhs,
                    x=torch.zeros_like(rhs))
    m = _mesh_of(case, seed)
    if kind == "request":
        return dict(case=case, mesh=m)
    kw = dict(block_rhs=case["K"]) if kind == "block" else {}
    s = V.Solver.from_mesh(m, precision=_prec(case), autotune=case["autotune"], setup_device=1, **kw)
    rhs = torch.from_numpy(m.rhs if kind == "block" else m.rhs[0]).cuda()
    return dict(case=case, solver=s, rhs=rhs, x=torch.zeros_like(rhs))


def run(state):
    case = state["case"]
    if case["kind"] == "request":
        m = state["mesh"]
        with V.Solver.from_mesh(m, precision=_prec(case), setup_device=1) as s:
            x, info = s.solve(m.rhs[0], case["rtol"])
        return dict(x=x, iterations=info["iterations"])
    if case["kind"] == "packed":
        info = state["solver"].solve_packed_device(state["rhs"], state["x"], case["rtol"])
    else:
        info = state["solver"].solve_device(state["rhs"], state["x"], case["rtol"])
    infos = info if isinstance(info, list) else [info]
    return dict(x=state["x"], iterations=np.array([i["iterations"] for i in infos]))


# ---------------------------------------------------------------------------
# work: what the method cannot do without. Per iteration the fine FP64 operator
# once, and every V-cycle operator twice in the V-cycle's precision (once for the
# forward sweep with its residual, once for the backward sweep); a block solve
# reads them once for all columns. Blocks per vertex of the fine operator and of
# the coarser levels together, and iterations, are those of the meshes above.
# ---------------------------------------------------------------------------
def _solve_work(nv, dim, mixed, iters, cols=1):
    dd = dim * dim
    fine, coarse = (14.6, 110.0) if dim == 3 else (7.0, 34.0)
    t = 4 if mixed else 8
    blocks = nv * (fine + 2 * (fine + coarse))
    nbytes = nv * fine * (8 * dd + 4) + 2 * nv * (fine + coarse) * (t * dd + 4)
    vec = 12 * nv * dim * 8 * cols
    return dict(bytes=float(iters * (nbytes + vec)), flops=float(iters * blocks * 2 * dd * cols))


def work(case):
    mixed = case["precision"] == "mixed"
    if case["kind"] == "packed":
        side = 0.5 * (case["lo"] + case["hi"])
        return _solve_work(case["parts"] * side ** case["dim"], case["dim"], mixed, 9)
    dim = 2 if case["nz"] == 1 else 3
    nv = case["nx"] * case["ny"] * case["nz"]
    iters = 60 if case.get("graded") else 12 if case["rtol"] > 1e-7 else 16
    cols = case.get("n_rhs", 1)
    w = _solve_work(nv, dim, mixed, iters * -(-cols // case.get("K", 1)), min(cols, case.get("K", 1)))
    if case["kind"] == "request":            # the mesh in, the hierarchy's operators written once
        w["bytes"] += nv * (14.6 + 110.0 if dim == 3 else 41.0) * (8 * dim * dim + 4)
    return w


# ---------------------------------------------------------------------------
# exact: the same systems assembled from the lattice stencil and solved by
# Jacobi-preconditioned CG in FP64 to far below the cases' tolerances. Graded
# meshes are too ill-conditioned for that.
# ---------------------------------------------------------------------------
def _assemble(m):
    """CSR of the (unconstrained) stiffness matrix, every lattice neighbour stored."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    dim, nv = m.dim, m.coords.shape[0]
    el = torch.from_numpy(m.elems).to(dev).long()
    X = torch.from_numpy(m.coords).to(dev)[el]                       # [ne, dim+1, dim]
    e = X[:, 1:] - X[:, :1]
    if dim == 3:
        cof = torch.stack([torch.linalg.cross(e[:, 1], e[:, 2]), torch.linalg.cross(e[:, 2], e[:, 0]),
                           torch.linalg.cross(e[:, 0], e[:, 1])], dim=1)
    else:
        cof = torch.stack([torch.stack([e[:, 1, 1], -e[:, 1, 0]], 1),
                           torch.stack([-e[:, 0, 1], e[:, 0, 0]], 1)], dim=1)
    det = (e[:, 0] * cof[:, 0]).sum(1)
    g = cof / det[:, None, None]                                     # gradients of vertices 1..dim
    g = torch.cat([-g.sum(1, keepdim=True), g], dim=1)
    vol = det / (2.0 if dim == 2 else 6.0)
    E, nu = torch.from_numpy(m.E).to(dev), torch.from_numpy(m.nu).to(dev)
    mu, lam = E / (2 * (1 + nu)) * vol, E * nu / ((1 + nu) * (1 - 2 * nu)) * vol
    shape = torch.tensor(m.shape, device=dev)
    strides = torch.cumprod(torch.cat([torch.ones(1, dtype=torch.long, device=dev), shape[:-1]]), 0)
    lat = lambda v: torch.stack([(v // strides[a]) % shape[a] for a in range(dim)], -1)  # noqa: E731
    ns = 3 ** dim
    w = torch.tensor([3 ** a for a in range(dim)], device=dev)
    M = torch.zeros((nv * ns, dim, dim), dtype=torch.float64, device=dev)
    eye = torch.eye(dim, dtype=torch.float64, device=dev)
    for i in range(dim + 1):
        for j in range(dim + 1):
            slot = ((lat(el[:, j]) - lat(el[:, i]) + 1) * w).sum(-1)
            gi, gj = g[:, i], g[:, j]
            dot = (gi * gj).sum(1)
            K = (lam[:, None, None] * gi[:, :, None] * gj[:, None, :]
                 + mu[:, None, None] * gj[:, :, None] * gi[:, None, :]
                 + (mu * dot)[:, None, None] * eye)
            M.index_add_(0, el[:, i] * ns + slot, K)
    M = M.view(nv, ns, dim, dim)
    off = torch.stack([(torch.arange(ns, device=dev) // 3 ** a) % 3 - 1 for a in range(dim)], -1)
    v = torch.arange(nv, device=dev)
    nb = v[:, None] + (off * strides).sum(-1)
    ok = ((lat(v)[:, None] + off >= 0) & (lat(v)[:, None] + off < shape)).all(-1)
    nb = torch.where(ok, nb, v[:, None])                             # absent neighbours: zero blocks
    cols = (nb[:, None, :, None] * dim + torch.arange(dim, device=dev)).expand(nv, dim, ns, dim)
    vals = M.permute(0, 2, 1, 3)
    crow = torch.arange(nv * dim + 1, device=dev) * (ns * dim)
    diag = M[:, ns // 2].diagonal(dim1=1, dim2=2).reshape(-1).clone()
    A = torch.sparse_csr_tensor(crow, cols.reshape(-1), vals.reshape(-1).contiguous(),
                                size=(nv * dim, nv * dim), check_invariants=False)
    return A, diag


def _exact_solve(m):
    A, diag = _assemble(m)
    dev = diag.device
    free = torch.from_numpy(1.0 - m.fixed.reshape(-1)).to(dev)[:, None]
    B = torch.from_numpy(m.rhs.reshape(m.rhs.shape[0], -1).T.copy()).to(dev) * free
    dinv = free / diag[:, None]
    x = torch.zeros_like(B)
    r, z = B.clone(), dinv * B
    p, rho, bn = z.clone(), (B * z).sum(0), B.norm(dim=0)
    for k in range(20000):
        q = free * (A @ (free * p))
        alpha = rho / (p * q).sum(0).clamp_min(1e-300)
        x += alpha * p
        r -= alpha * q
        if k % 50 == 49 and bool((r.norm(dim=0) < 1e-11 * bn).all()):
            break
        z = dinv * r
        new = (r * z).sum(0)
        p = z + (new / rho.clamp_min(1e-300)) * p
        rho = new
    return x.T.reshape(m.rhs.shape).contiguous()


def exact(case, seed):
    if case.get("graded"):
        return None
    if case["kind"] == "packed":
        return dict(x=torch.cat([_exact_solve(m)[0] for m in _parts_of(case, seed)]), iterations=None)
    x = _exact_solve(_mesh_of(case, seed))
    return dict(x=x if case["kind"] == "block" else x[0], iterations=None)
