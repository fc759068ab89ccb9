"""The in-LDS tree stage for densities that crowd towards the largest coordinate (the
last of its equal-width buckets), against the oracle's tree to the bit."""
import numpy as np
import pytest

from gpu_util import same_tree

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["both", "one"])
@pytest.mark.parametrize("n,L", [(1024, 3), (1025, 3), (4096, 4), (16385, 6), (300001, 8)])
def test_crowded_at_the_end(orc, kind, n, L):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1311_1006_amd as F
    rng = np.random.default_rng(n)
    x, y = 1.0 - rng.random(n) ** 3, rng.random(n)
    if kind == "both":
        y = 1.0 - y ** 3
    same_tree(orc, F, (x + 1j * y).astype(np.complex128), L)
