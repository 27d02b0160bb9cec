"""Solutions of FP32-cycle solves in 2D with materials 1:100, pinned.

PCG amplifies the rounding of its FP32 preconditioner in these problems (15 to 40
products, some of the spectrum converged long before) to 1e-9 .. 1e-8 of the
solution, so another order of the cycle's FP32 sums gives another of many equally
converged iterates, and a caller who compares solutions between versions of the
library sees them change. The pinned values are the library's own, from the cycle
launched level by level: 32 seeded random-sign projections of each solution, whose
distance estimates the distance of the whole vectors.

Run as a program to write the file: python tests/test_gpu_fp32_order.py > tests/golden/fp32_order_2d.json
"""
import importlib.util
import json
import os
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.append(ROOT)

from workloads import small2d  # noqa: E402

torch = pytest.importorskip("torch")
from paper_2505_09064_amd import vasmg as V  # noqa: E402

pytestmark = pytest.mark.gpu

GOLD = os.path.join(ROOT, "tests", "golden")
GOLDEN = os.path.join(GOLD, "fp32_order_2d.json")
_spec = importlib.util.spec_from_file_location("make_oracle_golden", os.path.join(GOLD, "make_oracle_golden.py"))
_gold = importlib.util.module_from_spec(_spec)
_spec.loader.exec_module(_gold)

# name: kind, vertices per side of each mesh, seed
CASES = {
    "pack of 9 to 14": ("pack", (9, 12, 10, 14), 105),
    "pack of 8 to 17": ("pack", (8, 13, 17, 11), 136),
    "solve 52": ("solve", (52,), 114),
    "5 columns, 40": ("block", (40,), 130),
    "device set-up, 45": ("device set-up", (45,), 111),
}


def mixed2d(n, seed, fix="x0"):
    """small2d with E in {1, 100} on 4 x 4 squares."""
    m = small2d(n, seed=seed, fix=fix, nu=0.35)
    table = np.where(np.random.default_rng(seed).random((4, 4)) < 0.5, 100.0, 1.0)
    c = m.coords[m.elems].mean(axis=1)
    i = np.minimum((c * 4).astype(int), 3)
    m.E = table[i[:, 0], i[:, 1]]
    return m


def solve(kind, sides, seed):
    """(solutions, iterations) at rtol 1e-6."""
    ms = [mixed2d(n, seed + k, "symmetry" if k % 3 == 2 else "x0") for k, n in enumerate(sides)]
    kw = dict(precision=V.FP32_PRECOND)
    if kind == "pack":
        pk = V.PackedSolver([V.Solver.from_mesh(m, host_only=1, **kw) for m in ms])
        xs, infos = pk.solve_packed([m.rhs[0] for m in ms], 1e-6)
        pk.free()
        return np.concatenate([x.ravel() for x in xs]), [i["iterations"] for i in infos]
    m = ms[0]
    if kind == "block":
        f = np.random.default_rng(seed).normal(size=(5,) + m.coords.shape) * np.abs(m.rhs[0]).max()
        with V.Solver.from_mesh(m, block_rhs=4, **kw) as s:
            x, infos = s.solve(f, 1e-6)
        return x, [i["iterations"] for i in infos]
    with V.Solver.from_mesh(m, setup_device=1 if kind == "device set-up" else 0, **kw) as s:
        x, info = s.solve(m.rhs[0], 1e-6)
    return x, [info["iterations"]]


@pytest.mark.parametrize("name", list(CASES))
def test_solution_is_the_pinned_one(name):
    """1e-9 of the solution, the last digit that FP64 outputs are held to, and the
    same iterations."""
    with open(GOLDEN) as f:
        g = json.load(f)[name]
    x, its = solve(*CASES[name])
    e = np.linalg.norm(_gold.sketch(x) - np.array(g["sketch"])) / np.sqrt(_gold.SKETCH_ROWS) / g["norm"]
    print(name, its, f"{e:.1e}")
    assert its == g["iterations"] and e <= 1e-9


if __name__ == "__main__":
    out = {}
    for case_name, spec in CASES.items():
        sol, n_its = solve(*spec)
        out[case_name] = dict(iterations=n_its, norm=float(np.linalg.norm(sol)), sketch=_gold.sketch(sol).tolist())
    json.dump(out, sys.stdout, indent=1)
