"""Replays of captured graphs: a plan launches a new combination directly the
first time, captures it the second time and replays it from the third on.  Each
test counts the graphs where it takes a replay for granted, and every replay is
compared with the direct launches, with the program's own work between them."""

import numpy as np
import pytest

import oracle
import synth
from gpu_util import assert_close, grid_dims, oracle_solve, to_dev, to_host

pytestmark = pytest.mark.gpu


def _plan(shape, bcs, prec="f64", max_batch=1):
    from paper_2501_03377_amd import Plan
    nx, ny, nz = grid_dims(shape)
    return Plan(nx, ny, nz, bcs, prec=prec, max_batch=max_batch)


def _graphs(plan):
    from paper_2501_03377_amd.kpcg import kp_plan_graph_count
    return kp_plan_graph_count(plan._h)


def _batch(prec, bcs, seed):
    """Right-hand sides that iterate next to ones that never do: all null space
    or zero, and one with an infinity."""
    shape = (16, 32, 16) if prec.startswith("i8") else (12, 10, 16)
    rng = np.random.default_rng(seed)
    eta = np.stack([rng.standard_normal(shape),
                    np.full(shape, 2.5 if oracle.is_singular(bcs) else 0.0),
                    rng.standard_normal(shape), np.ones(shape)])
    eta[3, 1, 2, 3] = np.inf
    return shape, eta


# The whole solve in one graph (the same buffers every time).  Two direct solves
# first: the first chunk of a plan's later solves differs from its first one's.
@pytest.mark.parametrize("prec", ["f64", "f32", "bf16x6", "i8x6"])
@pytest.mark.parametrize("bcs", [("D", "N", "P"), ("N", "N", "N")])
@pytest.mark.parametrize("flags", [0, "diagnostics"])
def test_whole_solve_with_rhs_that_make_no_iteration(prec, bcs, flags):
    import torch
    from paper_2501_03377_amd import KP_ENONFINITE, KP_FLAG_DIAGNOSTICS, KP_FLAG_NO_GRAPH
    shape, eta = _batch(prec, bcs, 81)
    flags = KP_FLAG_DIAGNOSTICS if flags else 0
    plan = _plan(shape, bcs, prec, 4)
    e, u = to_dev(eta), torch.empty_like(to_dev(eta))

    def solve(fl):
        u.fill_(float("nan"))
        _, res, hist, rc = plan.solve(e, tol=1e-10, max_iter=20, flags=flags | fl, out=u,
                                      raise_on_error=False)
        torch.cuda.synchronize()
        assert rc == KP_ENONFINITE
        return to_host(u), repr(res), np.asarray(hist)     # (repr: results hold NaN)

    solve(KP_FLAG_NO_GRAPH)
    ref = solve(KP_FLAG_NO_GRAPH)
    for b in (0, 2):
        assert_close(ref[0][b], oracle_solve(eta[b], bcs), 1e-10, b)
    for b in (1, 3):
        assert np.array_equal(ref[0][b], np.zeros(shape))
    counts = []
    for call in range(5):
        got = solve(0)
        counts.append(_graphs(plan))
        assert np.array_equal(got[0], ref[0]) and got[1] == ref[1], call
        assert np.array_equal(got[2], ref[2], equal_nan=True), call
        if call == 3:                       # the program's own work, and a direct solve
            torch.randn_like(e).sum().item()
            solve(KP_FLAG_NO_GRAPH)
    assert counts == [0, 1, 1, 1, 1]
    plan.close()


# The iterations alone in a graph (no call repeats the buffers of the one before):
# one graph per right-hand side's buffer where the iterations read it (a
# nonsingular set's R_0), one for all where they do not; a repeat then captures the
# whole solve beside it.
@pytest.mark.parametrize("prec", ["f64", "f32", "i8x6"])
@pytest.mark.parametrize("bcs", [("D", "N", "P"), ("N", "N", "N")])
def test_iterations_of_alternating_right_hand_sides(prec, bcs):
    import torch
    from paper_2501_03377_amd import KP_FLAG_NO_GRAPH
    shape = (16, 32, 48)
    etas = [synth.charge_field(shape, ncharges=200, seed=82 + k) for k in range(2)]
    plan = _plan(shape, bcs, prec)
    dev = [to_dev(a) for a in etas]
    u = torch.empty_like(dev[0])

    def solve(k, fl=0):
        u.fill_(float("nan"))
        _, res, hist, rc = plan.solve(dev[k], tol=1e-10, max_iter=20, flags=fl, out=u)
        torch.cuda.synchronize()
        assert rc == 0
        return to_host(u), res, np.asarray(hist)

    ref = None
    for _ in range(2):
        ref = [solve(k, KP_FLAG_NO_GRAPH) for k in (0, 1)]
    for k in (0, 1):
        assert_close(ref[k][0], oracle_solve(etas[k], bcs), 1e-10, k)
    for call in range(8):
        got = solve(call % 2)
        want = ref[call % 2]
        assert np.array_equal(got[0], want[0]) and got[1] == want[1], call
        assert np.array_equal(got[2], want[2]), call
    chunks = 1 if oracle.is_singular(bcs) else 2
    assert _graphs(plan) == chunks
    for call in range(4):                   # the last buffers again: the whole solve
        got = solve(1)
        assert np.array_equal(got[0], ref[1][0]) and got[1] == ref[1][1], call
    assert _graphs(plan) == chunks + 1
    plan.close()


# A batch on the int8 split, replayed.
@pytest.mark.parametrize("prec", ["i8x6", "i8x7"])
def test_int8_batch_replays(prec):
    import torch
    from paper_2501_03377_amd import KP_FLAG_NO_GRAPH
    shape, bcs = (16, 48, 32), ("P", "D", "N")
    eta = np.stack([synth.charge_field(shape, ncharges=100, seed=84 + b) for b in range(3)])
    plan = _plan(shape, bcs, prec, 3)
    e = to_dev(eta)
    u = torch.empty_like(e)
    out = []
    for call in range(6):
        u.fill_(float("nan"))
        _, res, _, rc = plan.solve(e, tol=1e-10, flags=KP_FLAG_NO_GRAPH if call < 2 else 0, out=u)
        assert rc == 0
        out.append((to_host(u), res))
    assert _graphs(plan) == 1
    for b in range(3):
        assert_close(out[1][0][b], oracle_solve(eta[b], bcs), 1e-10, b)
    for got in out[2:]:
        assert np.array_equal(got[0], out[1][0]) and got[1] == out[1][1]
    plan.close()
