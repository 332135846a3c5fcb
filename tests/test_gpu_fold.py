"""The folded mode products (FP64 and the int8 splits): parity groups on every
boundary condition at the sizes where the fold can go wrong, and the tile
shapes chosen by size."""

import numpy as np
import pytest

from gpu_util import assert_close, grid_dims, oracle_pinv, to_dev, to_host
from oracle.spectral import axis_eigenpairs

pytestmark = pytest.mark.gpu


def _plan(shape, bcs, max_batch=1, prec="f64"):
    from paper_2501_03377_amd import Plan
    nx, ny, nz = grid_dims(shape)
    return Plan(nx, ny, nz, bcs, prec=prec, max_batch=max_batch)


def _tol(shape, bcs):
    """1e-12 for the products, plus the oracle's own error: LAPACK's smallest
    nonzero eigenvalue sum mu is off by about 12 eps / mu relative."""
    lam = [axis_eigenpairs(n, bc)[0] for n, bc in zip(shape[::-1], bcs)]
    low = sum(l[0] for l in lam)
    mu = low if low > 1e-13 else min(l[l > 1e-12].min() for l in lam)
    return 1e-12 + 12 * np.finfo(float).eps / mu


# x, y and z extents: odd (a centre without a mirror image), even but not a
# multiple of 4 or 8 (chunks that cross a group's end, unaligned groups),
# quarters of odd length (36, 52, 68), one k-block and one more (64 / 68), the
# smallest that folds (17 and 18 in two, 36 in four) and the largest that does
# not (16)
@pytest.mark.parametrize("shape,bcs", [
    ((16, 17, 18), ("D", "N", "P")),
    ((36, 35, 34), ("D", "P", "P")),
    ((33, 52, 68), ("P", "P", "N")),
    ((20, 66, 100), ("P", "D", "N")),
    ((72, 31, 50), ("N", "P", "P")),
    ((40, 48, 64), ("P", "D", "P")),
    ((64, 129), ("N", "P")),
    ((260, 130), ("D", "P")),
    ((24, 16, 512), ("P", "DN", "D")),
    ((16, 500, 24), ("ND", "P", "N")),
])
def test_folded_pinv_matches_the_oracle(shape, bcs):
    rng = np.random.default_rng(51)
    r = rng.standard_normal(shape)
    plan = _plan(shape, bcs)
    z = to_host(plan.apply_pinv(to_dev(r)))
    plan.close()
    assert_close(z, oracle_pinv(r, bcs), _tol(shape, bcs), (shape, bcs))


# a large batch takes other tile shapes than one right-hand side (from 16-row
# tiles to full-width ones); each output is summed in the same order in all
@pytest.mark.parametrize("shape,bcs,batch", [
    ((16, 16, 512), ("P", "D", "N"), 96),
    ((16, 16, 512), ("DN", "P", "P"), 96),
    ((8, 75, 256), ("D", "N", "DN"), 64),
    ((64, 64, 64), ("P", "D", "N"), 48),
    ((48, 96, 192), ("P", "N", "D"), 24),
])
def test_tile_shapes_agree_bitwise(shape, bcs, batch):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(52)
    r = torch.randn((batch,) + shape, dtype=torch.float64, device="cuda", generator=gen)
    plan = _plan(shape, bcs, max_batch=batch)
    zb = plan.apply_pinv(r)
    for b in (0, batch // 2, batch - 1):
        assert torch.equal(plan.apply_pinv(r[b].contiguous()), zb[b]), b
    plan.close()


# the int8 kernel's thread and k-block shapes: 256 and 512 threads (axes up to
# 256 and beyond), 1 to 16 pairs a thread, partly filled k-blocks (16, 48, 80,
# 144, 272), fragments past the group (80, 208), one, two and four groups, and
# rows that end inside a tile (2D, 48 rows)
@pytest.mark.parametrize("prec", ["i8x6", "i8x7"])
@pytest.mark.parametrize("shape,bcs", [
    ((16, 32, 48), ("P", "N", "DN")),
    ((64, 80, 96), ("D", "P", "N")),
    ((112, 16, 128), ("P", "D", "ND")),
    ((48, 144, 192), ("N", "P", "D")),
    ((16, 208, 256), ("P", "DN", "N")),
    ((32, 16, 272), ("P", "D", "P")),
    ((16, 16, 320), ("N", "P", "D")),
    ((16, 384, 32), ("D", "P", "DN")),
    ((16, 32, 512), ("P", "N", "D")),
    ((16, 32, 512), ("DN", "D", "P")),
    ((512, 16, 16), ("ND", "P", "N")),
    ((48, 80), ("P", "D")),
])
def test_folded_int8_pinv_matches_the_oracle(shape, bcs, prec):
    rng = np.random.default_rng(53)
    r = rng.standard_normal(shape)
    plan = _plan(shape, bcs, prec=prec)
    z = to_host(plan.apply_pinv(to_dev(r)))
    plan.close()
    assert_close(z, oracle_pinv(r, bcs), _tol(shape, bcs), (shape, bcs))


def test_int8_tiles_of_128_rows():
    """Short axes with many rows take 128-row tiles: a batch of plans' largest
    size against the oracle, and bitwise equal to its single solves."""
    import torch
    shape, bcs, batch = (16, 32, 320), ("DN", "P", "N"), 8
    rng = np.random.default_rng(54)
    r = rng.standard_normal((batch,) + shape)
    plan = _plan(shape, bcs, max_batch=batch, prec="i8x6")
    zb = plan.apply_pinv(to_dev(r))
    for b in (0, batch - 1):
        assert_close(to_host(zb[b]), oracle_pinv(r[b], bcs), _tol(shape, bcs), b)
        assert torch.equal(plan.apply_pinv(to_dev(r[b])), zb[b])
    plan.close()


# the one-kernel solve: axes of one and two fragments per group (16 | 17, 32 |
# 33, 63), odd ones, and periodic ones whose products fold in four (36, 52);
# with a tolerance out of reach it iterates to the limit, or until its residual
# is all rounding (a breakdown), and stays accurate
@pytest.mark.parametrize("shape,bcs", [
    ((16, 33), ("D", "P")), ((31, 48), ("N", "D")), ((32, 17), ("P", "N")),
    ((34, 63), ("DN", "P")), ((49, 47), ("P", "ND")), ((36, 52), ("P", "P")),
    ((63, 15), ("D", "D")), ((64, 33), ("ND", "DN")), ((3, 4), ("P", "N")),
])
@pytest.mark.parametrize("tol,max_iter", [(1e-12, 20), (1e-18, 3)])
def test_one_kernel_solve_at_tile_edges(shape, bcs, tol, max_iter):
    rng = np.random.default_rng(55)
    eta = rng.standard_normal((2,) + shape)
    if all(b in "PN" for b in bcs):
        eta -= eta.mean(axis=(1, 2), keepdims=True)
    plan = _plan(shape, bcs, max_batch=2)
    u, res, _, rc = plan.solve(to_dev(eta), tol=tol, max_iter=max_iter,
                              raise_on_error=tol == 1e-12)
    plan.close()
    assert tol < 1e-12 or rc == 0
    assert all(r["iterations"] <= max_iter for r in res)
    for b in range(2):
        assert_close(to_host(u)[b], oracle_pinv(eta[b], bcs), 1e-10, (shape, bcs, b))
