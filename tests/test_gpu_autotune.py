"""The autotuner times the kernels that a solve launches."""

import pytest

from gpu_util import grid_dims

pytestmark = pytest.mark.gpu


# The tuner works on the plan's workspace: it clears the first product's input
# (FP64) and the two buffers between products, and its products of zeros write
# zeros.  The last product of a solve writes its sums as FP32, half of an FP64
# grid, so that is what the tuner may have written; the rest stays as it was.
@pytest.mark.parametrize("prec", ["bf16", "bf16x6"])
@pytest.mark.parametrize("shape,bcs", [((16, 24, 40), ("P", "D", "N")), ((40, 64), ("D", "P"))])
def test_autotuned_last_product_is_a_solves(shape, bcs, prec):
    import torch
    from paper_2501_03377_amd import Plan
    from paper_2501_03377_amd.kpcg import kp_plan_set_workspace
    nx, ny, nz = grid_dims(shape)
    plan = Plan(nx, ny, nz, bcs, prec=prec, max_batch=1)
    ws = torch.full((plan.workspace_bytes,), 0xff, dtype=torch.uint8, device="cuda")
    assert kp_plan_set_workspace(plan._h, ws.data_ptr(), ws.numel()) == 0
    plan.autotune(batch=1, reps=1)
    torch.cuda.synchronize()
    n = nx * ny * nz
    between = 2 if prec == "bf16" else 4
    assert int((ws == 0).sum()) == n * (8 + 2 * between + 4)
    assert int((ws == 0xff).sum()) == ws.numel() - n * (8 + 2 * between + 4)
    plan.close()
