"""L2P of the logarithmic potential on both sides of the line between 32 lanes per
leaf and a workgroup per leaf (64 points per leaf on average), a single leaf and
leaves of several times 256 points among them, against the same sums of the same
order (tests/order_reference.py): rounding, 1e-12 in FP64 and 1e-6 in mixed precision."""
import numpy as np
import pytest

from paper_1311_1006_amd import workloads as W

from gpu_util import dev, e2, host
from order_reference import Order

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,L", [(700, 1), (1024, 3), (1025, 3), (4096, 4), (4100, 4), (5000, 2)])
@pytest.mark.parametrize("p", [5, 33])
def test_log_l2p(orc, n, L, p):
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
