"""The constant terms of the logarithmic local expansions at the edges of their
loops: orders around the 8 coefficients that a lane has in flight and the 32
lanes of a box, trees of 2 to 8 levels (a leaf adds up its ancestors' terms),
against the direct sum.

The bar: under the theta-criterion every shift's terms fall by 2 theta / (1 +
theta) = 2/3 per order, and the directly truncated series is used at no more than
p terms, so the error relative to the sum of |q log| is at most (2/3)^p / (1 -
2/3) for either expansion; the random signs' 2-norm of u is taken against that
sum, which is at most sqrt(n) times larger.  Observed errors lie far below;
rounding adds 1e-12 in FP64 (the parity bar) and 1e-6 in mixed precision.  Leaves
hold two points or more: a leaf without extent can overflow FP32 coefficients."""
import numpy as np
import pytest

from paper_1311_1006_amd import workloads as W

from gpu_util import dev, e2, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1311_1006_amd as F
    F.lib()
    return F


@pytest.mark.parametrize("n,L", [(16, 2), (3000, 3), (20000, 6), (40000, 8)])
@pytest.mark.parametrize("p", [1, 2, 8, 9, 10, 32, 33, 48, 64])
def test_log_constants_by_order(F, orc, n, L, p):
    import torch
    z, _, _ = W.uniform(n, seed=n + L)
    q = np.random.default_rng(p).standard_normal(n)
    sub = np.arange(0, n, max(1, n // 2000))
    ref = orc.direct_log_points(z, q, z[sub])
    tree = F.build_tree(dev(z), L)
    for prec, floor in (("fp64", 1e-12), ("mixed", 1e-6)):
        u = host(F.evaluate_log(F.plan(tree, p, 0.5, prec), torch.from_numpy(q).to("cuda")))
        assert e2(u[sub], ref) <= 2 * 3 * (2 / 3) ** p * np.sqrt(n) + floor, prec
