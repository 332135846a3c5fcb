"""A solve's result does not depend on what its plan solved before, from which
the plan only sizes the first chunk of launches, nor on whether its last
iteration is the last one allowed."""

import numpy as np
import pytest

from gpu_util import assert_close, grid_dims, oracle_laplacian, to_dev, to_host

pytestmark = pytest.mark.gpu


def _plan(shape, bcs, prec="f64", max_batch=1):
    from paper_2501_03377_amd import Plan
    nx, ny, nz = grid_dims(shape)
    return Plan(nx, ny, nz, bcs, prec=prec, max_batch=max_batch)


# axes of more than 32 points: the certificate's box does not hold every mode, so
# that its bound lies above the error estimate of the next application
CASES = [("f64", (20, 36, 40), ("D", "N", "DN")), ("f64", (40, 48, 36), ("N", "P", "N")),
         ("i8x6", (48, 48, 64), ("P", "D", "N"))]


def _rough(shape, bcs, seed):
    """L w for white noise w: relative to the solution as large as the residual's
    rounding is to its error, or larger, so that the residual test passes first."""
    return oracle_laplacian(np.random.default_rng(seed).standard_normal(shape), bcs)


# A tolerance just above the error estimate and below both bounds: with one
# iteration allowed only the application that closes it can stop the solve.
@pytest.mark.parametrize("prec,shape,bcs", CASES)
def test_last_iteration_allowed_is_whole(prec, shape, bcs):
    from paper_2501_03377_amd import KP_NOT_CONVERGED
    eta = to_dev(_rough(shape, bcs, 71))
    plan = _plan(shape, bcs, prec)
    _, (probe,), _, rc = plan.solve(eta, tol=1e-300, max_iter=1)
    plan.close()
    assert rc == KP_NOT_CONVERGED and probe["pinv_applications"] == 2, probe
    tol = probe["err_est"] * (1 + 1e-9)
    assert 0.0 < probe["rel_res"] <= tol
    for later in (False, True):
        plan = _plan(shape, bcs, prec)
        if later:
            _, (easy,), _, rc = plan.solve(eta, tol=1e-3, max_iter=20)
            assert rc == 0 and easy["iterations"] == easy["pinv_applications"] == 1
        _, (r,), _, rc = plan.solve(eta, tol=tol, max_iter=1)
        plan.close()
        assert rc == 0 and r["iterations"] == 1 and r["pinv_applications"] == 2, (later, r)
        assert r["err_est"] == probe["err_est"] and r["true_rel_res"] == probe["true_rel_res"]


# A certificate that the plan's last solve did not need is launched only when the
# residual test asks for it: the solve that needs one, whether it holds or not,
# ends with the same bits as on a new plan, where it is launched at once.
@pytest.mark.parametrize("prec,shape,bcs", CASES)
def test_deferred_certificate(prec, shape, bcs):
    eta = to_dev(_rough(shape, bcs, 72))
    new = lambda tol: _solve_on(_plan(shape, bcs, prec), eta, tol)
    _, probe = new(1e-300)
    # what the free bound ||R|| / (lambda_min ||U||) gives, from a solve that it stops
    _, free = new(1e-3)
    assert free["iterations"] == free["pinv_applications"] == 1 and free["err_est"] <= 1e-3
    _, held = new(0.9 * free["err_est"])
    assert held["pinv_applications"] == 1 and held["err_est"] < 0.9 * free["err_est"], held
    assert probe["err_est"] < held["err_est"]
    for tol, applications in ((0.9 * free["err_est"], 1),
                              (0.5 * (probe["err_est"] + held["err_est"]), 2)):
        ref, r = new(tol)
        assert r["iterations"] == 1 and r["pinv_applications"] == applications, r
        plan = _plan(shape, bcs, prec)
        plan.solve(eta, tol=1e-3, max_iter=20)
        u, q = _solve_on(plan, eta, tol)
        assert q == r
        assert np.array_equal(u, ref), tol


def _solve_on(plan, eta, tol):
    u, (r,), _, _ = plan.solve(eta, tol=tol, max_iter=20 if tol > 1e-300 else 1)
    plan.close()
    return to_host(u), r


# A start whose mean is far larger than the solution (a singular set): the
# iterates keep it, and the error tests count on that, over every chunk of
# launches of the solve (an easy solve before makes them one iteration long).
@pytest.mark.parametrize("easy_first", [False, True])
@pytest.mark.parametrize("shape,bcs", [((16, 24, 32), ("N", "P", "N")), ((40, 56), ("P", "N"))])
def test_warm_start_with_a_large_mean(shape, bcs, easy_first):
    from paper_2501_03377_amd import KP_FLAG_WARM_START
    w = np.random.default_rng(73).standard_normal(shape)
    w -= w.mean()
    eta = to_dev(oracle_laplacian(w, bcs))
    plan = _plan(shape, bcs, "f32")
    if easy_first:
        _, (easy,), _, rc = plan.solve(eta, tol=1e-3, max_iter=20)
        assert rc == 0 and easy["iterations"] == 1
    start = np.random.default_rng(74).standard_normal(shape)
    u, (r,), _, rc = plan.solve(eta, tol=1e-10, max_iter=20, flags=KP_FLAG_WARM_START,
                                out=to_dev(start + 100.0))
    plan.close()
    assert rc == 0 and r["iterations"] >= 2, r
    assert 0.0 < r["err_est"] <= 1e-10
    assert_close(to_host(u), w, 1e-10, (shape, bcs))
    plan = _plan(shape, bcs, "f32")
    _, (q,), _, _ = plan.solve(eta, tol=1e-10, max_iter=20, flags=KP_FLAG_WARM_START,
                               out=to_dev(start - start.mean()))
    plan.close()
    # (the start's rounding differs, far below the tolerance)
    assert r["iterations"] <= q["iterations"] + 1, (r, q)


# A batch at its limit of one iteration, in which one right-hand side stops, one
# runs on and one makes no iteration: the exit step that rides on the last
# kernel of such a chunk (a later solve), and the one of its own (a first solve).
@pytest.mark.parametrize("prec", ["f64", "i8x6"])
@pytest.mark.parametrize("bcs", [("D", "N", "P"), ("N", "P", "N")])
def test_batch_at_a_limit_of_one_iteration(prec, bcs):
    import torch
    from paper_2501_03377_amd import KP_FLAG_RESIDUAL_ONLY, KP_NOT_CONVERGED
    shape = (16, 32, 48)
    x = np.cos(np.pi * (np.arange(48) + 0.5) / 48) if bcs[0] == "N" else \
        np.sin(np.pi * np.arange(1, 49) / 49)
    smooth = np.broadcast_to(x, shape)     # (its residual is all rounding of a large u)
    eta = to_dev(np.stack([_rough(shape, bcs, 75), smooth, np.zeros(shape)]))
    plan = _plan(shape, bcs, prec, 3)
    _, probe, _, _ = plan.solve(eta, tol=1e-300, max_iter=1, flags=KP_FLAG_RESIDUAL_ONLY)
    plan.close()
    rough, far = probe[0]["rel_res"], probe[1]["rel_res"]
    assert 0.0 < 4 * rough < far, (rough, far)
    tol, got = np.sqrt(rough * far), []
    for later in (False, True):
        plan = _plan(shape, bcs, prec, 3)
        if later:
            _, easy, _, rc = plan.solve(eta, tol=1e-3, max_iter=20, flags=KP_FLAG_RESIDUAL_ONLY)
            assert rc == 0 and [r["iterations"] for r in easy] == [1, 1, 0]
        u = torch.full_like(eta, float("nan"))
        _, res, hist, rc = plan.solve(eta, tol=tol, max_iter=1, flags=KP_FLAG_RESIDUAL_ONLY,
                                      out=u)
        plan.close()
        assert rc == KP_NOT_CONVERGED
        assert [r["status"] for r in res] == [0, KP_NOT_CONVERGED, 0], res
        assert [r["iterations"] for r in res] == [1, 1, 0]
        assert [r["pinv_applications"] for r in res][:2] == [1, 2]
        uh = to_host(u)
        assert np.array_equal(uh[2], np.zeros(shape))
        for b in range(2):   # the residual of what is returned, to its rounding
            r = to_host(eta)[b] - oracle_laplacian(uh[b], bcs)
            assert np.linalg.norm(r) <= 1e-10 * np.linalg.norm(to_host(eta)[b])
        got.append((uh, res, np.asarray(hist)))
    assert np.array_equal(got[0][0], got[1][0])
    assert got[0][1] == got[1][1] and np.array_equal(got[0][2], got[1][2])
