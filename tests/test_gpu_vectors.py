"""The sums and updates after an application, with Z held as FP32 values (the
FP32, BF16 and BF16X6 products) and as FP64 ones, and the flexible beta."""

import numpy as np
import pytest

from gpu_util import assert_close, grid_dims, oracle_pinv, to_dev, to_host

pytestmark = pytest.mark.gpu


def _plan(shape, bcs, prec="f64"):
    from paper_2501_03377_amd import Plan
    nx, ny, nz = grid_dims(shape)
    return Plan(nx, ny, nz, bcs, prec=prec, max_batch=1)


# an odd number of points (no pairs), an even one below a block's share, and
# one of more than one block and stencil tile
SHAPES = [((7, 9, 11), ("D", "N", "DN")), ((12, 16, 20), ("P", "N", "P")),
          ((33, 21), ("ND", "D")), ((20, 40, 72), ("D", "P", "D"))]


# Every sum, scale and test of a solve scales exactly with a power of two, and
# the stored FP32 values stay the same: the two runs agree bit for bit, though
# FP32 could not hold the larger Z.
@pytest.mark.parametrize("flex", [False, True])
@pytest.mark.parametrize("prec", ["f32", "bf16", "bf16x6"])
@pytest.mark.parametrize("shape,bcs", SHAPES)
def test_solve_scales_exactly(shape, bcs, prec, flex):
    from paper_2501_03377_amd import KP_FLAG_FLEX_BETA
    rng = np.random.default_rng(61)
    eta = rng.standard_normal(shape)
    plan = _plan(shape, bcs, prec)
    flags = KP_FLAG_FLEX_BETA if flex else 0
    runs = []
    for e in (0, 200):
        u, res, hist, rc = plan.solve(to_dev(eta * 2.0 ** e), tol=1e-11, max_iter=60, flags=flags)
        assert rc == 0
        runs.append((to_host(u) * 2.0 ** -e, np.asarray(hist)))
    plan.close()
    assert np.array_equal(runs[0][0], runs[1][0])
    assert np.array_equal(runs[0][1], runs[1][1])
    # the error test or bound at 1e-11 (an estimate: ten times that)
    assert_close(runs[0][0], oracle_pinv(eta, bcs), 1e-10, (shape, bcs, prec))


# A fixed symmetric preconditioner: the flexible beta is the ordinary one up to
# the loss of orthogonality, some eps times the condition number (below 1e5
# here) per step.
@pytest.mark.parametrize("shape,bcs", SHAPES)
def test_flexible_beta_is_the_ordinary_one(shape, bcs):
    from paper_2501_03377_amd import KP_FLAG_FLEX_BETA
    rng = np.random.default_rng(62)
    eta = rng.standard_normal(shape)
    plan = _plan(shape, bcs)
    plan.set_preconditioner("jacobi", steps=3, omega=1.3)
    hists = [np.asarray(plan.solve(to_dev(eta), tol=1e-13, max_iter=8, flags=f)[2]).ravel()
             for f in (0, KP_FLAG_FLEX_BETA)]
    plan.close()
    assert hists[0].size == hists[1].size and hists[0][-1] > 0.0
    assert np.max(np.abs(hists[1] / hists[0] - 1.0)) < 1e-8


# rows of whole pairs (the odd ones take the other kernel): a single pair, and
# several blocks, under every pair of ends along x
@pytest.mark.parametrize("bcx", ["P", "D", "N", "DN", "ND"])
@pytest.mark.parametrize("shape", [(3, 5, 4), (7, 4), (9, 34, 66)])
def test_field_in_pairs(shape, bcx):
    import oracle
    rng = np.random.default_rng(63)
    bcs = (bcx, "ND", "P")[:len(shape)]
    u = rng.standard_normal(shape)
    faces = rng.standard_normal((len(shape), 2))
    faces[[b == "P" for b in bcs]] = 0.0
    plan = _plan(shape, bcs)
    eps = to_host(plan.field(to_dev(u), faces))
    plan.close()
    ref = oracle.field(u.T, bcs, faces)
    for a in range(len(shape)):
        assert np.array_equal(eps[a], ref[a].T), (bcs, a)
