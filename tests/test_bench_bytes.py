"""The byte models of the benchmark's rooflines against the arrays that the
kernels read and write, and the batch's model against the single run's: one
place holds both."""
import ast
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

INFO = dict(n_nodes=1_100, n_free=1_000, nnz=14_000, nnz_field=15_500)
N, NF, NNZ, NNZ_D, ND = 1_100, 1_000, 14_000, 1_500, 100


@pytest.fixture(scope="module")
def bench():
    import importlib.util
    spec = importlib.util.spec_from_file_location("bench_module", os.path.join(ROOT, "bench.py"))
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


def _full(e32):
    real = 4 if e32 else 8
    rows = 4 + 8 + 8 + 8 + 3 * 8 + 4 * real    # map, phi, charge, load; x, b, r; E
    rows += 32 if e32 else 0                    # row sums of R
    return NF * rows + 4 * NNZ + NNZ_D * (4 + 3 * real) + ND * (8 + 4 * real)


@pytest.mark.parametrize("e32", [False, True])
def test_passes(bench, e32):
    B = bench.pass_bytes(INFO, e32)
    assert B["full"] == _full(e32)
    assert B["inc"] == NF * (4 + 8 + 8 + 2 * 8 + 2 * 8 + 8 + 8)
    assert B["iter"] == NF * (2 * 32 + 2 * 8 + 2 * 8 + 7 * 4)
    rows = [dict(cg_iters=k) for k in (0, 3, 0, 0)]
    want = B["full"] + 3 * B["inc"] + B["back"] + B["full"]
    assert bench.solve_bytes(INFO, rows, lean=False, iterations=False, e32=e32) == want
    assert bench.solve_bytes(INFO, rows, lean=False, e32=e32) == want + 3 * B["iter"]
    # (steps 1 and 3 follow one without iterations; 3 has no step after it)
    lean = B["full"] + B["lean"] + B["prep"] + 2 * B["inc"] + B["back"] + B["full"] + 3 * B["iter"]
    assert bench.solve_bytes(INFO, rows, e32=e32) == lean


def test_metal_iteration(bench):
    # value and column; a record each way, p and x each way
    assert bench.metal_iter_bytes(100, 1500) == 1500 * (8 + 4) + 100 * (2 * 32 + 4 * 8)


def test_legs_hold_no_model_of_their_own():
    """The batch and metal legs take their bytes from the functions above."""
    with open(os.path.join(ROOT, "bench.py")) as f:
        legs = {n.name: n for n in ast.parse(f.read()).body if isinstance(n, ast.FunctionDef)}
    calls = {k: {c.func.id for c in ast.walk(v) if isinstance(c, ast.Call)
                 and isinstance(c.func, ast.Name)} for k, v in legs.items()}
    assert {"solve_bytes", "operator_bytes"} <= calls["run_batch_leg"]
    assert "metal_iter_bytes" in calls["run_metal_leg"]
