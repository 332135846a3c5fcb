"""bench.py's accounting of the mode products (CPU): what is set against a
matrix-core ceiling is the work of an axis's parity groups, and the profiler's
names of the library's kernels have the form in which the library reports them."""

import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture()
def bench(monkeypatch):
    monkeypatch.setattr(sys, "argv", ["bench.py"])
    if ROOT not in sys.path:
        sys.path.insert(0, ROOT)
    import bench as b
    return b


def test_groups_divide_the_contraction(bench):
    grid, N = (512, 512, 512), 512 ** 3
    for g in (1, 2, 4):
        groups = {c: g for c in bench.MODEPROD}
        assert bench.launch_work("modeprod_x_bwd", grid, 3, groups=groups) == \
            ("flop", 3 * 2.0 * N * 512 / g)
        # the Hadamard factor is not folded
        assert bench.launch_work("modeprod_z_fwd", grid, 1, groups=groups) == \
            ("flop", 2.0 * N * 512 / g + N)
    # without groups: the plain products of an application add up to 4N(nx+ny+nz) + N
    one = [{"iterations": 1, "pinv_applications": 1}]
    grid, N = (48, 32, 80), 48 * 32 * 80
    assert sum(bench.solve_work(c, grid, one)[1] for c in bench.MODEPROD) == \
        4.0 * N * (48 + 32 + 80) + N


def test_small_solve_folds_in_two(bench):
    res = [{"iterations": 1, "pinv_applications": 2}]
    N = 64 * 64
    assert bench.solve_work("small_solve", (64, 64, 1), res) == ("flop", 2 * (4.0 * N * 128 + N))
    for g in (2, 4):     # (the one-kernel solve folds in at most two)
        groups = {c: g for c in bench.PRODUCT_ORDER[2]}
        assert bench.solve_work("small_solve", (64, 64, 1), res, groups=groups) == \
            ("flop", 2 * (4.0 * N * 128 / 2 + N))


def test_profiler_names_of_unnamed_namespaces(bench):
    n = bench.profiler_kernel_name
    assert n("void kp::(anonymous namespace)::mp_fold<0, double, double, 4, 1, 2, 2, 1>"
             "(kp::(anonymous namespace)::FoldArgs)") == \
        "kp::mp_fold<0, double, double, 4, 1, 2, 2, 1>"
    assert n("void kp::(anonymous namespace)::mp_oz<6, 2, true, 8, 512, 32>"
             "(kp::(anonymous namespace)::OzArgs)") == "kp::mp_oz<6, 2, true, 8, 512, 32>"
    names = {"modeprod_x_fwd": "kp::mp_oz<6, 4, true, 4, 512, 32>|131072"}
    assert bench.launch_identity("modeprod_x_fwd", "i8x6", (512,) * 3, 1, [13] * 6, names) == \
        "kp::mp_oz<6, 4, true, 4, 512, 32>|131072"
    assert bench.launch_identity("small_solve", "f64", (64, 64, 1), 1, [0] * 4) == \
        n("void kp::(anonymous namespace)::k_small_solve<2>(kp::Geom, kp::SmallOps)")
