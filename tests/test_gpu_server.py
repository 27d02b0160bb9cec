"""Serving engine (vasmg_server_*): continuous batching of independent solve
requests on one GPU. Every served result matches the oracle's solve of the same
request (FP64: 1e-8 relative error, +-1 iteration; FP32 V-cycle: +-1 iteration
of the oracle's FP32 mode, 1e-5 of its FP64 solution). Each result is the same
alone and in the mix (bitwise:
the kernels are deterministic and autotuning is off in the server), the HBM
budget bounds the bytes resident at once, a request that cannot fit or cannot be
set up fails alone while the others complete, and every request's timestamps
are ordered submit <= setup <= admission <= done."""
import numpy as np
import pytest

from oracle import Oracle
from workloads import small2d, small3d

torch = pytest.importorskip("torch")
from paper_2505_09064_amd import vasmg as V  # noqa: E402

pytestmark = pytest.mark.gpu


def _requests():
    out = []
    for i in range(8):
        if i % 2 == 0:
            m = small2d(9 + 4 * i, seed=i, nu=0.3 + 0.02 * i,
                        fix="symmetry" if i == 4 else "boundary")
        else:
            m = small3d(5 + i // 2, seed=i, fix="symmetry" if i == 5 else "x0")
        rng = np.random.default_rng(i)
        m.E = np.where(rng.random(m.elems.shape[0]) < 0.5, 1.0, 100.0)
        out.append(m)
    return out


_oracle_cache = {}


def _check_against_oracle(i, m, x, info, precision):
    """A served result against the oracle's solve of the same request: FP64
    within 1e-8 relative solution error and +-1 iteration; the FP32 V-cycle
    within +-1 iteration of the oracle's FP32 mode and 1e-5 of its FP64
    solution, reaching rtol in the FP64 true residual."""
    if i not in _oracle_cache:
        o = Oracle(m.coords, m.elems, m.E, m.nu, m.fixed)
        xo, io = o.solve(m.rhs[0], 1e-6)
        _, io32 = o.solve(m.rhs[0], 1e-6, precision="fp32")
        _oracle_cache[i] = (xo, io, io32)
    xo, io, io32 = _oracle_cache[i]
    err = np.linalg.norm(x - xo) / np.linalg.norm(xo)
    assert info["rel_res_true"] < 1e-6
    if precision == V.FP64:
        assert abs(info["iterations"] - io["iterations"]) <= 1, (i, info["iterations"], io["iterations"])
        assert err <= 1e-8, (i, err)
    else:
        assert abs(info["iterations"] - io32["iterations"]) <= 1, (i, info["iterations"],
                                                                   io32["iterations"])
        assert err <= 1e-5, (i, err)


def _alone(m, **opt):
    s = V.Solver.from_mesh(m, autotune=0, **opt)
    x, info = s.solve(m.rhs[0], 1e-6)
    s.free()
    return x, info


@pytest.mark.parametrize("precision", [V.FP64, V.FP32_PRECOND])
def test_results_same_alone_and_in_the_mix(precision):
    reqs = _requests()
    srv = V.Server(slots=3, setup_workers=3, precision=precision)
    ids = [srv.submit(m, m.rhs[0], 1e-6) for m in reqs]
    got = [srv.wait(i) for i in ids]
    st = srv.stats()
    srv.close()
    assert st["completed"] == len(reqs) and st["peak_bytes"] <= st["budget_bytes"]
    for i, (m, (x, res)) in enumerate(zip(reqs, got)):
        assert res["status"] == V.OK, res
        _check_against_oracle(i, m, x, res["info"], precision)
        xa, ia = _alone(m, precision=precision)
        assert res["info"]["iterations"] == ia["iterations"]
        assert np.array_equal(x, xa), np.abs(x - xa).max()
        assert res["info"]["rel_res_true"] < 1e-6
        t = [res[k] for k in ("t_submit_ms", "t_setup_start_ms", "t_setup_end_ms", "t_admit_ms",
                              "t_done_ms")]
        assert all(a <= b for a, b in zip(t, t[1:])), t
        assert 0 <= res["slot"] < 3 and res["device_bytes"] > 0


def test_device_setup_workers():
    """Setup workers that form the Galerkin products on the device (options
    setup_device = 1, transient device memory ordered on each worker's stream)
    while other requests solve and capture graphs: every result equals the same
    request solved alone from a device setup, bit for bit, and takes the
    iterations of a host setup. The size limits of the host setup are off here,
    so every request takes the device setup."""
    reqs = _requests()
    srv = V.Server(slots=3, setup_workers=3, setup_device=1, host_setup_max_dofs=(0, 0))
    ids = [srv.submit(m, m.rhs[0], 1e-6) for m in reqs]
    got = [srv.wait(i) for i in ids]
    srv.close()
    for i, (m, (x, res)) in enumerate(zip(reqs, got)):
        assert res["status"] == V.OK, res
        assert res["setup_device"] == 1
        _check_against_oracle(i, m, x, res["info"], V.FP64)
        xa, ia = _alone(m, setup_device=1)
        assert np.array_equal(x, xa), np.abs(x - xa).max()
        _, ih = _alone(m)
        assert res["info"]["iterations"] == ih["iterations"]
        assert res["info"]["rel_res_true"] < 1e-6


def test_small_requests_set_up_on_the_host():
    """With setup_device = 1, requests at or below the dimension's DOF limit are
    set up on the host (their results equal the host-setup solve alone, bit for
    bit) and larger ones on the device (equal to the device-setup solve alone)."""
    reqs = [small2d(9, seed=1), small3d(5, seed=2), small2d(13, seed=3), small3d(7, seed=4)]
    lim2, lim3 = 2 * 9 * 9, 3 * 6 * 6 * 6          # 9x9 and 5^3 vertices at or below
    srv = V.Server(slots=2, setup_workers=2, setup_device=1, host_setup_max_dofs=(lim2, lim3))
    ids = [srv.submit(m, m.rhs[0], 1e-6) for m in reqs]
    got = [srv.wait(i) for i in ids]
    srv.close()
    for i, (m, (x, res)) in enumerate(zip(reqs, got)):
        assert res["status"] == V.OK, res
        lim = lim2 if m.dim == 2 else lim3
        on_device = int(m.coords.size > lim)
        assert res["setup_device"] == on_device, (i, m.coords.size, res["setup_device"])
        xa, _ = _alone(m, setup_device=on_device)
        assert np.array_equal(x, xa), (i, np.abs(x - xa).max())
    assert [r["setup_device"] for _, r in got] == [0, 0, 1, 1]


def test_budget_bounds_resident_bytes():
    reqs = _requests()
    # the estimate of each request, from a host-only handle
    est = []
    for m in reqs:
        s = V.Solver.from_mesh(m, host_only=1, autotune=0)
        b = V.C.c_int64()
        V._check(V.lib().vasmg_device_bytes(s._h, V.C.byref(b)))
        est.append(b.value)
        s.free()
    budget = int(max(est) * 1.5)
    srv = V.Server(slots=4, setup_workers=2, hbm_budget_bytes=budget)
    ids = [srv.submit(m, m.rhs[0], 1e-6) for m in reqs]
    res = [srv.wait(i)[1] for i in ids]
    st = srv.stats()
    srv.close()
    assert all(r["status"] == V.OK for r in res)
    assert st["peak_bytes"] <= budget
    # no two requests whose bytes exceed the budget together were resident at once
    for i in range(len(res)):
        for j in range(i + 1, len(res)):
            a, b = res[i], res[j]
            if a["device_bytes"] + b["device_bytes"] > budget:
                assert a["t_done_ms"] <= b["t_admit_ms"] or b["t_done_ms"] <= a["t_admit_ms"]


def test_server_config_validation():
    for kw in (dict(pack_max_dofs=-1), dict(pack_max_parts=300), dict(pack_wait_ms=-5),
               dict(host_setup_max_dofs=(-1, 0)), dict(host_setup_max_dofs=(0, -1))):
        with pytest.raises(V.VasmgError) as ei:
            V.Server(slots=1, setup_workers=1, **kw)
        assert ei.value.status == V.EINVAL, kw


def test_failing_requests_fail_alone():
    ok1, big, ok2 = small2d(9, seed=1), small3d(12, seed=2), small2d(11, seed=3)
    bad = small2d(9, seed=4)
    bad.elems[3, [1, 2]] = bad.elems[3, [2, 1]]           # inverted triangle
    srv = V.Server(slots=2, setup_workers=2, hbm_budget_bytes=6 << 20)
    ids = [srv.submit(m, m.rhs[0], 1e-6) for m in (ok1, big, bad, ok2)]
    out = [srv.wait(i) for i in ids]
    srv.close()
    assert out[0][1]["status"] == V.OK and out[3][1]["status"] == V.OK
    assert out[1][1]["status"] == V.ENOMEM and out[1][0] is None
    assert out[2][1]["status"] == V.EINVAL
    xa, _ = _alone(ok2)
    assert np.array_equal(out[3][0], xa)


def test_uploaded_bytes_within_estimate():
    m = small3d(9, seed=5)
    s = V.Solver.from_mesh(m, host_only=1, autotune=0)
    est, act = V.C.c_int64(), V.C.c_int64()
    V._check(V.lib().vasmg_device_bytes(s._h, V.C.byref(est)))
    V._check(V.lib().vasmg_upload(s._h, None))
    V._check(V.lib().vasmg_device_bytes(s._h, V.C.byref(act)))
    assert 0 < act.value <= est.value
    x, info = s.solve(m.rhs[0], 1e-6)
    xa, ia = _alone(m)
    assert np.array_equal(x, xa)
    assert V.lib().vasmg_upload(s._h, None) == V.EINVAL      # already on the device
    s.free()


@pytest.mark.parametrize("precision", [V.FP64, V.FP32_PRECOND])
def test_packed_serving(precision):
    """Packing on (pack_max_dofs, a batching window long enough for every setup
    to finish, one slot): the 2D and the 3D requests are each solved as one
    pack, and every result still matches the oracle's solve of its own request
    and the request solved alone (FP64: 1e-10 relative, +-1 iteration; the dot
    products sum in another order)."""
    reqs = _requests()
    srv = V.Server(slots=1, setup_workers=4, precision=precision, pack_max_dofs=100000,
                   pack_max_parts=8, pack_wait_ms=5000)
    ids = [srv.submit(m, m.rhs[0], 1e-6) for m in reqs]
    got = [srv.wait(i) for i in ids]
    st = srv.stats()
    srv.close()
    assert st["completed"] == len(reqs) and st["peak_bytes"] <= st["budget_bytes"]
    sizes = [res["pack_size"] for _, res in got]
    assert max(sizes) > 1, sizes
    for i, (m, (x, res)) in enumerate(zip(reqs, got)):
        assert res["status"] == V.OK and res["info"]["status"] == V.OK, res
        _check_against_oracle(i, m, x, res["info"], precision)
        xa, ia = _alone(m, precision=precision)
        assert abs(res["info"]["iterations"] - ia["iterations"]) <= 1
        if precision == V.FP64:
            assert np.linalg.norm(x - xa) / np.linalg.norm(xa) <= 1e-10
        t = [res[k] for k in ("t_submit_ms", "t_setup_start_ms", "t_setup_end_ms", "t_admit_ms",
                              "t_done_ms")]
        assert all(a <= b for a, b in zip(t, t[1:])), t
    # requests packed together share their admission and completion times
    by_admit = {}
    for _, res in got:
        by_admit.setdefault(res["t_admit_ms"], []).append(res)
    for group in by_admit.values():
        assert all(r["pack_size"] == len(group) for r in group)
        assert len({r["t_done_ms"] for r in group}) == 1


def test_small_requests_pack_under_a_modest_budget():
    """Eight small requests, each a few MiB of levels, under a budget of 1 GiB: the
    dense tables and their construction (tens to hundreds of MiB a request) do not
    keep them apart. One worker sets up, so that all wait while the first does."""
    ms = [small3d(9, seed=i) for i in range(8)]
    budget = 1 << 30
    srv = V.Server(slots=1, setup_workers=1, pack_max_dofs=100000, pack_max_parts=8,
                   pack_wait_ms=5000, hbm_budget_bytes=budget)
    ids = [srv.submit(m, m.rhs[0], 1e-8) for m in ms]
    got = [srv.wait(i) for i in ids]
    st = srv.stats()
    srv.close()
    assert st["peak_bytes"] <= budget
    assert max(res["pack_size"] for _, res in got) >= 6, [res["pack_size"] for _, res in got]
    for m, (x, res) in zip(ms, got):
        with V.Solver.from_mesh(m) as s:
            xa, ia = s.solve(m.rhs[0], 1e-8)
        assert res["status"] == V.OK and abs(res["info"]["iterations"] - ia["iterations"]) <= 1
        assert np.linalg.norm(x - xa) / np.linalg.norm(xa) <= 1e-10
