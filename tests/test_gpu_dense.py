"""The small levels of the cycle as dense tables: the preconditioner application
against the oracle where the tables start at the fused bottom's level, above it,
at their largest part, in the additive form, with unequal sweep counts, on
constrained components, and in a pack whose parts differ in depth; and the same
answers without them, where a server's budget has no room for the tables."""
import numpy as np
import pytest

from oracle import Oracle, OracleOptions
from workloads import small2d, small3d

torch = pytest.importorskip("torch")
from paper_2505_09064_amd import vasmg as V  # noqa: E402

pytestmark = pytest.mark.gpu

MAX_DOFS = 2304


def _first_table_level(s):
    """(first level the tables cover, first level of the fused bottom)."""
    ph = s.profile_iteration(1)
    lo = [p["level"] for p in ph if p["name"] == "bottom"]
    up = [p["level"] for p in ph if p["name"] == "dense_up"]
    down = [p["level"] for p in ph if p["name"] == "dense_down"]
    assert len(lo) == 1 and up == down and len(up) <= 1
    return (up or lo)[0], lo[0]


# name: mesh, options, oracle options
CASES = {
    "bottom only, 2D": (lambda: small2d(9, seed=1), {}, {}),
    "above the bottom, 2D rollers": (lambda: small2d(34, seed=2, fix="symmetry"), {}, {}),
    "above the bottom, 3D": (lambda: small3d(9, seed=3), {}, {}),
    "rollers, 3D": (lambda: small3d(8, seed=4, fix="symmetry"), {}, {}),
    "near the largest, 3D": (lambda: small3d(13, seed=5), {}, {}),
    "past the largest on level 1, 3D": (lambda: small3d(17, seed=6), {}, {}),
    "additive": (lambda: small3d(9, seed=7), dict(cycle=V.CYCLE_ADDITIVE), dict(cycle="additive")),
    "sweeps (2, 1)": (lambda: small3d(9, seed=8), dict(n_pre=2, n_post=1), dict(n_pre=2, n_post=1)),
    "sweeps (1, 0)": (lambda: small2d(21, seed=9), dict(n_pre=1, n_post=0), dict(n_pre=1, n_post=0)),
}


@pytest.mark.parametrize("prec", [V.FP64, V.FP32_PRECOND])
@pytest.mark.parametrize("name", list(CASES))
def test_dense_tables_match_oracle(name, prec):
    """FP64: 1e-11 of the norm, the cycle's own bar. FP32: the operators' float32
    rounding enters as often as in the oracle's FP32 mode, so the distance to the
    FP64 cycle is at most 4 times that mode's (and 16 float32 units)."""
    make, kw, okw = CASES[name]
    m = make()
    o = Oracle(m.coords, m.elems, m.E, m.nu, m.fixed, OracleOptions(**okw))
    s = V.Solver.from_mesh(m, precision=prec, **kw)
    first, lo = _first_table_level(s)
    sizes = [s.level_info(l)["n_vertices"] * m.dim for l in range(s.hierarchy_info()[0])]
    assert sizes[first] <= MAX_DOFS and (first == 1 or sizes[first - 1] > MAX_DOFS), (sizes, first, lo)
    n = o.A[0].shape[0] // m.dim
    r = np.random.default_rng(6).normal(size=(n, m.dim))
    z = torch.zeros((n, m.dim), dtype=torch.float64, device="cuda")
    s.apply_precond_device(torch.from_numpy(r).cuda(), z)
    again = torch.zeros_like(z)
    s.apply_precond_device(torch.from_numpy(r).cuda(), again)
    assert torch.equal(z, again)
    ref = o.apply_precond(r.ravel(), precision="fp64")
    err = np.linalg.norm(z.cpu().numpy().ravel() - ref) / np.linalg.norm(ref)
    if prec == V.FP64:
        assert err < 1e-11
    else:
        ref32 = o.apply_precond(r.ravel(), precision="fp32")
        gap = np.linalg.norm(ref32 - ref) / np.linalg.norm(ref)
        assert err <= max(4 * gap, 16 * 2.0 ** -24), (err, gap)
    s.free()


@pytest.mark.parametrize("prec", [V.FP64, V.FP32_PRECOND])
def test_dense_tables_of_a_pack(prec):
    """Parts of different depth and size, one of them a single small part: every
    part against its own solve alone (the bars of the packed solves)."""
    for ms in ([small3d(5, seed=1), small3d(11, seed=2, fix="symmetry"), small3d(7, seed=3)],
               [small2d(30, seed=4), small2d(8, seed=5), small2d(17, seed=6, fix="symmetry")],
               [small3d(6, seed=7)]):
        parts = [V.Solver.from_mesh(m, precision=prec, host_only=1) for m in ms]
        pk = V.PackedSolver(parts)
        assert any(p["name"] == "bottom" for p in pk.profile_iteration(1))
        xs, infos = pk.solve_packed([m.rhs[0] for m in ms], 1e-8)
        for m, x, i in zip(ms, xs, infos):
            with V.Solver.from_mesh(m, precision=prec) as s:
                xa, ia = s.solve(m.rhs[0], 1e-8)
            assert i["status"] == V.OK and abs(i["iterations"] - ia["iterations"]) <= 1
            assert np.linalg.norm(x - xa) / np.linalg.norm(xa) <= (1e-10 if prec == V.FP64 else 1e-5)
        pk.free()


@pytest.mark.parametrize("K", [4, 8, 16])
@pytest.mark.parametrize("prec", [V.FP64, V.FP32_PRECOND])
def test_dense_tables_of_a_block_solve(prec, K):
    """The products for K columns, with and without tables above the bottom, row
    and vertex counts off the matrix tile: every column of a block solve against
    its single-column solve (the tables are the same, the sums in another order)."""
    for m in (small3d(9, seed=3), small3d(11, seed=5, fix="symmetry"), small2d(9, seed=1),
              small2d(35, seed=2), small3d(17, seed=6)):
        nf = m.n_vertices
        F = np.random.default_rng(K).normal(size=(K + 1, nf, m.dim)) * np.abs(m.rhs[0]).max()
        s = V.Solver.from_mesh(m, precision=prec, block_rhs=K)
        _first_table_level(s)
        x, infos = s.solve(F, 1e-8)
        for k in (0, K - 1, K):
            xa, ia = s.solve(F[k], 1e-8)
            assert infos[k]["status"] == V.OK and abs(infos[k]["iterations"] - ia["iterations"]) <= 1
            assert np.linalg.norm(x[k] - xa) / np.linalg.norm(xa) <= (1e-10 if prec == V.FP64 else 1e-6)
        s.free()


def test_budget_without_room_for_tables():
    """A server's budget that holds the hierarchy but not its tables still serves
    the request (as it did when there were none), to the oracle's bars."""
    m = small3d(11, seed=9)
    s = V.Solver.from_mesh(m, host_only=1)
    b = V.C.c_int64()
    V._check(V.lib().vasmg_device_bytes(s._h, V.C.byref(b)))
    s.free()
    srv = V.Server(slots=1, setup_workers=1, hbm_budget_bytes=b.value - (1 << 20))
    x, res = srv.wait(srv.submit(m, m.rhs[0], 1e-8))
    srv.close()
    assert res["status"] == V.OK and res["device_bytes"] < b.value - (1 << 20), res
    xo, io = Oracle(m.coords, m.elems, m.E, m.nu, m.fixed).solve(m.rhs[0], 1e-8)
    assert abs(res["info"]["iterations"] - io["iterations"]) <= 1
    assert np.linalg.norm(x - xo) / np.linalg.norm(xo) <= 1e-8


def _few_cell_meshes():
    """Meshes whose first coarse levels hold one to eight cells."""
    return [small2d(3, seed=1, fix="x0"), small2d(4, seed=2, fix="x0"), small3d(3, seed=3, fix="x0"),
            small2d(4, seed=4, fix="symmetry"), small3d(3, seed=5, fix="symmetry")]


@pytest.mark.parametrize("prec", [V.FP64, V.FP32_PRECOND])
def test_cells_without_off_cell_blocks(prec):
    """Cells at the ends of the sweep order have no lower or no upper blocks, and a
    level of one cell has none at all: the first step of an empty range is read and
    dropped. Sweeps, residual (through the cycle) and solve against the oracle."""
    for m in _few_cell_meshes():
        o = Oracle(m.coords, m.elems, m.E, m.nu, m.fixed)
        s = V.Solver.from_mesh(m, precision=prec)
        xo, io = o.solve(m.rhs[0], 1e-8)
        x, info = s.solve(m.rhs[0], 1e-8)
        assert info["converged"] == 1 and abs(info["iterations"] - io["iterations"]) <= 1
        assert np.linalg.norm(x - xo) / np.linalg.norm(xo) <= (1e-8 if prec == V.FP64 else 1e-5)
        for l in range(1, s.hierarchy_info()[0] - 1):
            n = s.level_info(l)["n_vertices"]
            b = torch.from_numpy(np.random.default_rng(l).normal(size=(n, m.dim))).cuda()
            y = torch.zeros_like(b)
            for back in (0, 1):
                s.gs_sweep_device(l, prec, back, b, y)
            assert torch.isfinite(y).all()
        s.free()


@pytest.mark.parametrize("make", [lambda: small3d(9, seed=3), lambda: small2d(21, seed=3, fix="x0")])
def test_coarsest_solve_of_the_fp32_cycle_is_fp64(make):
    """The bottom's table, which holds the coarsest solve, has FP64 values in the
    FP32 cycle (its bytes in the profile), and on a slender body (8 : 1, an
    ill-conditioned coarsest operator) the cycle is as near to the FP64 one as the
    oracle's FP32 mode, whose coarsest solve is FP64: 4 times its distance."""
    m = make()
    m.coords[:, 0] *= 8.0
    o = Oracle(m.coords, m.elems, m.E, m.nu, m.fixed)
    s = V.Solver.from_mesh(m, precision=V.FP32_PRECOND)
    bottom = [p for p in s.profile_iteration(1) if p["name"] == "bottom"][0]
    n = s.level_info(bottom["level"])["n_vertices"] * m.dim
    assert bottom["bytes"] == n * ((8 * n + 15) // 16 * 16)
    nf = o.A[0].shape[0] // m.dim
    rng = np.random.default_rng(6)
    for r in (np.ones(nf * m.dim), rng.normal(size=nf * m.dim), o.A[0] @ rng.normal(size=nf * m.dim)):
        z = torch.zeros((nf, m.dim), dtype=torch.float64, device="cuda")
        s.apply_precond_device(torch.from_numpy(r.reshape(nf, m.dim)).cuda(), z)
        ref, ref32 = (o.apply_precond(r, precision=p) for p in ("fp64", "fp32"))
        gap = np.linalg.norm(ref32 - ref)
        assert np.linalg.norm(z.cpu().numpy().ravel() - ref) <= 4 * gap
    s.free()


@pytest.mark.parametrize("prec", [V.FP64, V.FP32_PRECOND])
def test_pack_tables_apply_each_part_s_cycle(prec):
    """One application of a pack's preconditioner through its tables, part by part
    against the part's oracle (the bars of the single tables): a wrong block of one
    part's table would hide behind a converged solve."""
    for ms in ([small3d(5, seed=1), small3d(11, seed=2, fix="symmetry"), small3d(7, seed=3)],
               [small2d(30, seed=4), small2d(8, seed=5), small2d(17, seed=6, fix="symmetry")]):
        dim = ms[0].dim
        pk = V.PackedSolver([V.Solver.from_mesh(m, precision=prec, host_only=1) for m in ms])
        assert any(p["name"] == "dense_up" for p in pk.profile_iteration(1))
        os_ = [Oracle(m.coords, m.elems, m.E, m.nu, m.fixed) for m in ms]
        r = [np.random.default_rng(i).normal(size=o.A[0].shape[0]) for i, o in enumerate(os_)]
        z = torch.zeros((sum(v.size for v in r) // dim, dim), dtype=torch.float64, device="cuda")
        pk.apply_precond_device(torch.from_numpy(np.concatenate(r).reshape(-1, dim)).cuda(), z)
        z = np.split(z.cpu().numpy().ravel(), np.cumsum([v.size for v in r])[:-1])
        for o, ri, zi in zip(os_, r, z):
            ref = o.apply_precond(ri, precision="fp64")
            err = np.linalg.norm(zi - ref) / np.linalg.norm(ref)
            if prec == V.FP64:
                assert err < 1e-11
            else:
                gap = np.linalg.norm(o.apply_precond(ri, precision="fp32") - ref) / np.linalg.norm(ref)
                assert err <= max(4 * gap, 16 * 2.0 ** -24), (err, gap)
        pk.free()
