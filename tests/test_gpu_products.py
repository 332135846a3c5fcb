"""What a plan reports about its mode products (kp_plan_product_kernel)."""

import re

import pytest

pytestmark = pytest.mark.gpu

CLASSES = ["modeprod_%s_%s" % (a, d) for d in ("fwd", "bwd") for a in "xyz"]


# (n, condition) of each axis with its groups: periodic axes of whole quarters fold
# in four where that saves padded work (64), else in two (34, 68 in four), the
# Dirichlet and Neumann ones in two from 17 points on, the mixed ones never; FP32
# and BF16 products are plain
@pytest.mark.parametrize("prec,n,bcs,groups", [
    ("f64", (64, 34, 17), ("P", "P", "D"), (4, 2, 2)),
    ("f64", (16, 128, 68), ("N", "DN", "P"), (1, 1, 4)),
    ("f64", (70, 33, 1), ("ND", "N"), (1, 2)),
    ("i8x6", (512, 256, 48), ("P", "D", "DN"), (4, 2, 1)),
    ("f32", (64, 34, 18), ("P", "P", "D"), (1, 1, 1)),
    ("bf16", (64, 32, 16), ("P", "P", "D"), (1, 1, 1)),
])
def test_reported_products(prec, n, bcs, groups):
    from paper_2501_03377_amd import KpError, Plan
    plan = Plan(*n, bcs, prec=prec, max_batch=2)
    dim = 3 if n[2] > 1 else 2
    for c in CLASSES:
        axis = "xyz".index(c.split("_")[1])
        if axis >= dim:
            with pytest.raises(KpError):
                plan.product_kernel(c)
            continue
        got = {b: plan.product_kernel(c, batch=b) for b in (1, 2)}
        assert {g for g, _ in got.values()} == {groups[axis]}, c
        for b, (_, name) in got.items():
            if prec == "bf16":
                assert name == ""
                continue
            m = re.fullmatch(r"kp::mp_(fold|oz)<([^<>]*)>\|(\d+)", name)
            assert m and (m.group(1) == "oz") == (prec == "i8x6"), name
            # whole blocks; the template's group count is the reported one
            assert int(m.group(3)) % 256 == 0
            args = m.group(2).split(", ")
            assert int(args[1] if prec == "i8x6" else args[3]) == groups[axis], name
    for bad in ("stencil_dot", "update_p"):
        with pytest.raises(KpError):
            plan.product_kernel(bad)
    with pytest.raises(KpError):
        plan.product_kernel(CLASSES[0], batch=3)     # beyond max_batch
    plan.close()
