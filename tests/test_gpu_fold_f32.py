"""The FP32 products' tile shapes, which are chosen by size: a large batch takes
other shapes than one right-hand side (and in a solve other kernels than in the
pseudoinverse alone: sums in FP32 at the end), and every output is summed in the
same order in all of them."""

import numpy as np
import pytest

from gpu_util import assert_close, grid_dims, oracle_pinv, to_dev, to_host

pytestmark = pytest.mark.gpu

# rows of whole 16-byte pieces and ragged ones (75, 130, 50, 33); the shapes of
# one right-hand side are the smallest, those of the batches reach from four
# row groups to the full width
CASES = [((16, 16, 512), ("P", "D", "N"), 512), ((8, 75, 256), ("D", "N", "DN"), 64),
         ((33, 50, 130), ("N", "P", "P"), 64), ((48, 96, 192), ("P", "N", "D"), 24),
         ((36, 300), ("ND", "P"), 128), ((20, 30, 384), ("N", "N", "N"), 100)]


@pytest.mark.parametrize("shape,bcs,batch", CASES)
def test_f32_tile_shapes_agree_bitwise(shape, bcs, batch):
    import torch
    from paper_2501_03377_amd import Plan
    nx, ny, nz = grid_dims(shape)
    gen = torch.Generator(device="cuda").manual_seed(57)
    r = torch.randn((batch,) + shape, dtype=torch.float64, device="cuda", generator=gen)
    plan = Plan(nx, ny, nz, bcs, prec="f32", max_batch=batch)
    zb = plan.apply_pinv(r)
    ub, res, _, rc = plan.solve(r, tol=1e-10, max_iter=20)
    assert rc == 0
    for b in (0, batch // 2, batch - 1):
        one = r[b].contiguous()
        assert torch.equal(plan.apply_pinv(one), zb[b]), b
        u, (q,), _, _ = plan.solve(one, tol=1e-10, max_iter=20)
        assert torch.equal(u, ub[b]) and q["iterations"] == res[b]["iterations"], b
    plan.close()
    # a relative residual of 1e-10 and an error bound or estimate of as much
    assert_close(to_host(ub[0]), oracle_pinv(to_host(r[0]), bcs), 1e-9, (shape, bcs))
