"""The small levels of the cycle without dense tables: the fused bottom kernel in the
V-cycle, and the level kernels on cells and parts without off-cell blocks. The
profile names the bottom's launch "bottom" whichever kernel it is; its bytes tell a
table (every value once) from the fused kernel (the levels' operators)."""
import numpy as np
import pytest

from oracle import Oracle, OracleOptions
from workloads import small2d, small3d

torch = pytest.importorskip("torch")
from paper_2505_09064_amd import vasmg as V  # noqa: E402

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24


def _handle(m, tables, **kw):
    s = V.Solver.from_mesh(m, host_only=1, **kw)
    s.set_dense_tables(tables)
    V._check(V.lib().vasmg_upload(s.handle, None))
    return s


def _table_bytes(s, level):
    n = s.level_info(level)["n_vertices"] * s.dim
    return n * ((8 * n + 15) // 16 * 16)


def _precond(s, r):
    z = torch.zeros(r.shape, dtype=torch.float64, device="cuda")
    s.apply_precond_device(torch.from_numpy(r).cuda(), z)
    return z.cpu().numpy().ravel()


# name: mesh, options, oracle options
CASES = {
    "2D, 4 levels": (lambda: small2d(17, seed=2, fix="symmetry"), {}, {}),
    "2D, graded": (lambda: small2d(33, seed=None, graded=True, nu=0.49), {}, {}),
    "2D, 3 levels": (lambda: small2d(9, seed=1), {}, {}),
    "3D, 2 levels": (lambda: small3d(9, seed=5), {}, {}),
    "3D, 3 levels, rollers": (lambda: small3d(8, seed=4, fix="symmetry"), {}, {}),
    "sweeps (2, 1)": (lambda: small3d(9, seed=8), dict(n_pre=2, n_post=1), dict(n_pre=2, n_post=1)),
    "sweeps (2, 2), 2D": (lambda: small2d(21, seed=9), dict(n_pre=2, n_post=2), dict(n_pre=2, n_post=2)),
    "sweeps (1, 0)": (lambda: small2d(21, seed=9), dict(n_pre=1, n_post=0), dict(n_pre=1, n_post=0)),
}


@pytest.mark.parametrize("tables", [False, True])
@pytest.mark.parametrize("prec", [V.FP64, V.FP32_PRECOND])
@pytest.mark.parametrize("name", list(CASES))
def test_bottom_with_and_without_tables(name, prec, tables):
    """The same handle either way: which kernel ran, and the preconditioner against
    the oracle (FP64 1e-11; FP32 4 of the oracle's own distances between its FP32 and
    FP64 modes, at least 16 float32 units)."""
    make, kw, okw = CASES[name]
    m = make()
    s = _handle(m, tables, precision=prec, **kw)
    ph = s.profile_iteration(1)
    bottom = [p for p in ph if p["name"] == "bottom"]
    assert len(bottom) == 1
    lo = bottom[0]["level"]
    assert (bottom[0]["bytes"] == _table_bytes(s, lo)) == tables
    launched = [p for p in ph if p["name"] == "gs_bwd" and 1 <= p["level"] < lo]
    dense = [p for p in ph if p["name"].startswith("dense")]
    assert len(dense) == (2 if tables and lo > 1 else 0) and (len(launched) == 0 or not tables)
    o = Oracle(m.coords, m.elems, m.E, m.nu, m.fixed, OracleOptions(**okw))
    r = np.random.default_rng(4).normal(size=(o.A[0].shape[0] // m.dim, m.dim))
    ref = o.apply_precond(r.ravel(), precision="fp64")
    err = np.linalg.norm(_precond(s, r) - ref) / np.linalg.norm(ref)
    if prec == V.FP64:
        assert err < 1e-11
    else:
        ref32 = o.apply_precond(r.ravel(), precision="fp32")
        assert err <= max(4 * np.linalg.norm(ref32 - ref) / np.linalg.norm(ref), 16 * U32)
    s.free()


def _few_cell_meshes():
    """Meshes whose first coarse level holds one to eight cells."""
    return {"2D 3": small2d(3, seed=1, fix="x0"), "2D 4": small2d(4, seed=2, fix="x0"),
            "3D 3": small3d(3, seed=3, fix="x0"), "2D 4 rollers": small2d(4, seed=4, fix="symmetry"),
            "3D 3 rollers": small3d(3, seed=5, fix="symmetry")}


@pytest.mark.parametrize("prec", [V.FP64, V.FP32_PRECOND])
@pytest.mark.parametrize("name", list(_few_cell_meshes()))
def test_sweeps_of_few_cells(name, prec):
    """Levels of one to eight cells, whose first cells have no lower and whose last no
    upper blocks: sweeps from a nonzero start, and the product, against the oracle."""
    m = _few_cell_meshes()[name]
    o = Oracle(m.coords, m.elems, m.E, m.nu, m.fixed)
    s = V.Solver.from_mesh(m, precision=prec)
    rng = np.random.default_rng(1)
    for l in range(o.L):
        n = o.A[l].shape[0] // m.dim
        x, b = rng.normal(size=(n, m.dim)), rng.normal(size=(n, m.dim))
        y = torch.zeros((n, m.dim), dtype=torch.float64, device="cuda")
        s.spmv_device(l, prec, torch.from_numpy(x).cuda(), y)
        ref = o.A[l] @ x.ravel()
        assert np.abs(y.cpu().numpy().ravel() - ref).max() < (1e-13 if prec == V.FP64 else 2e-6) * np.abs(ref).max()
        for back in (0, 1):
            g = torch.from_numpy(x).cuda()
            s.gs_sweep_device(l, prec, back, torch.from_numpy(b).cuda(), g)
            got = g.cpu().numpy().ravel()
            S = o.gs(l)
            ref = (S.backward if back else S.forward)(b.ravel(), x.ravel())
            err = np.abs(got - ref).max() / np.abs(ref).max()
            if prec == V.FP64:
                assert err < 1e-11, (l, back)
            else:
                S32 = o.gs(l, np.float32)
                b32, x32 = b.ravel().astype(np.float32), x.ravel().astype(np.float32)
                ref32 = (S32.backward if back else S32.forward)(b32, x32).astype(np.float64)
                gap = np.abs(ref32 - ref).max() / np.abs(ref).max()
                assert np.abs(got - ref32).max() / np.abs(ref).max() <= max(4 * gap, 16 * U32), (l, back)
    s.free()


@pytest.mark.parametrize("prec", [V.FP64, V.FP32_PRECOND])
@pytest.mark.parametrize("dim,copies", [(2, 14), (3, 6)])
def test_cycle_of_few_cells_launched_level_by_level(dim, copies, prec):
    """A pack whose coarsest levels together exceed 256 DOFs has neither fused bottom
    nor tables: every level is launched, the zero-guess sweep and the residual on
    cells without off-cell blocks among them. Every part's cycle against the oracle's."""
    ms = [m for m in _few_cell_meshes().values() if m.dim == dim] * copies
    os_ = [Oracle(m.coords, m.elems, m.E, m.nu, m.fixed) for m in ms]
    assert sum(o.A[-1].shape[0] for o in os_) > 256
    pk = V.PackedSolver([V.Solver.from_mesh(m, precision=prec, host_only=1) for m in ms])
    ph = pk.profile_iteration(1)
    assert not [p for p in ph if p["name"] == "bottom" or p["name"].startswith("dense")]
    assert [p for p in ph if p["name"] == "gs_fwd_zero" and p["level"] >= 1]
    r = [np.random.default_rng(i).normal(size=o.A[0].shape[0]) for i, o in enumerate(os_)]
    z = _precond(pk, np.concatenate(r).reshape(-1, dim))
    at = 0
    for o, ri in zip(os_, r):
        got = z[at:at + ri.size]
        at += ri.size
        ref = o.apply_precond(ri, precision="fp64")
        err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        if prec == V.FP64:
            assert err < 1e-11
        else:
            ref32 = o.apply_precond(ri, precision="fp32")
            assert err <= max(4 * np.linalg.norm(ref32 - ref) / np.linalg.norm(ref), 16 * U32)
    pk.free()


def test_a_tight_budget_leaves_the_tables_out():
    """A served request under a budget without room for its tables holds less, by
    the tables, than under a large one."""
    m = small3d(11, seed=9)
    with _handle(m, True) as s:
        tables = sum(p["bytes"] for p in s.profile_iteration(1) if p["name"] in ("bottom", "dense_down", "dense_up"))
    held = []
    for budget in (64 << 20, 16 << 30):
        srv = V.Server(slots=1, setup_workers=1, hbm_budget_bytes=budget)
        x, res = srv.wait(srv.submit(m, m.rhs[0], 1e-8))
        srv.close()
        assert res["status"] == V.OK
        held.append(res["device_bytes"])
    assert tables > 30 << 20 and abs(held[1] - held[0] - tables) < 1 << 16, (held, tables)


def test_dense_tables_are_chosen_before_the_upload():
    m = small3d(5, seed=1)
    with V.Solver.from_mesh(m, host_only=1) as s:
        s.set_dense_tables(False)
        with pytest.raises(V.VasmgError):
            V._check(V.lib().vasmg_set_dense_tables(s.handle, 2))
        pk = V.PackedSolver([s])
        assert not [p for p in pk.profile_iteration(1) if p["name"].startswith("dense")]
        with pytest.raises(V.VasmgError):
            pk.set_dense_tables(True)
        pk.free()


def _contrast(m, E=1.0, nu=None):
    """Every second element E times as stiff (or of Poisson ratio nu)."""
    m.E = np.where(np.arange(m.elems.shape[0]) % 2 == 0, 1.0, E)
    if nu is not None:
        m.nu = np.where(np.arange(m.elems.shape[0]) % 2 == 0, m.nu, nu)
    return m


@pytest.mark.parametrize("make,prec,tables", [
    (lambda: _contrast(small2d(17, seed=1), 10.0), V.FP32_PRECOND, True),
    (lambda: _contrast(small2d(17, seed=1), 10.5), V.FP32_PRECOND, False),
    (lambda: _contrast(small2d(17, seed=1, nu=0.0), nu=0.495), V.FP32_PRECOND, False),
    (lambda: _contrast(small2d(17, seed=1), 100.0), V.FP64, True),
    (lambda: _contrast(small3d(8, seed=1), 100.0), V.FP32_PRECOND, True),
])
def test_tables_by_stiffness_contrast(make, prec, tables):
    """The FP32 cycle in 2D tabulates up to a contrast of 10 (of E, or of lambda + 2 mu),
    alone and as part of a pack; FP64 and 3D whatever the contrast."""
    m = make()
    even = small2d(9, seed=2) if m.dim == 2 else small3d(5, seed=2)
    parts = [V.Solver.from_mesh(x, precision=prec, host_only=1) for x in (even, m)]
    for s in (V.Solver.from_mesh(m, precision=prec), V.PackedSolver(parts)):
        ph = s.profile_iteration(1)
        lo = [p for p in ph if p["name"] == "bottom"][0]["level"]
        smoothed = [p for p in ph if p["name"] == "gs_bwd" and p["level"] >= 1]
        dense = [p for p in ph if p["name"].startswith("dense")]
        if tables:
            assert not smoothed and len(dense) == (2 if lo > 1 else 0)
        else:
            assert not dense and len(smoothed) == lo - 1
        s.free()
