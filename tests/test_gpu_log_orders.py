"""The logarithmic potential against the same sums of the same order
(tests/order_reference.py), at the edges of the constants' loops: orders around the
8 coefficients that a lane has in flight and the 32 lanes of a box, trees of 2 to 6
levels.  The truncation is the same on both sides, so the bars are those of rounding:
1e-12 in FP64 (the parity bar), 1e-6 in mixed precision."""
import numpy as np
import pytest

from paper_1311_1006_amd import workloads as W

from gpu_util import dev, e2, host
from order_reference import Order

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,L", [(16, 2), (3000, 3), (9000, 5), (20000, 6)])
@pytest.mark.parametrize("p", [1, 2, 8, 9, 10, 32, 33, 48, 64])
def test_log_of_one_order(orc, n, L, p):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1311_1006_amd as F
    z, _, _ = W.uniform(n, seed=n + L)
    q = np.random.default_rng(p).standard_normal(n)
    ref = Order(orc, z, q + 0j, L, 0.5, p).log()
    tree = F.build_tree(dev(z), L)
    for prec, bar in (("fp64", 1e-12), ("mixed", 1e-6)):
        u = host(F.evaluate_log(F.plan(tree, p, 0.5, prec), torch.from_numpy(q).to("cuda")))
        assert e2(u, ref) <= bar, prec
