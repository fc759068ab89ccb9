"""The FP64 logarithm of the near field as the device computes it, one value per
problem: many problems of two points, one of them with a strength, so that the
potential at the other is log r alone.  Distances have 26 significant bits, so that
r^2 is rounded once at most; the bound is the one of tests/test_near_log.py, 0.6
units in the last place of the result."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["intervals", "one", "exponents"])
def test_one_logarithm(kind):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1311_1006_amd as F
    n, rng = 20000, np.random.default_rng(4)
    if kind == "intervals":
        d = 0.85 + 0.4 * rng.random(n)
    elif kind == "one":
        d = 1.0 + rng.uniform(-1, 1, n) * 2.0 ** rng.uniform(-24, -7, n)
    else:
        d = 2.0 ** rng.uniform(-500, 500, n)
    f, e = np.frexp(d)
    d = np.ldexp(np.round(f * 2.0 ** 26) * 2.0 ** -26, e)
    z = np.zeros(2 * n, np.complex128)
    z[1::2] = d
    q = np.zeros(2 * n)
    q[1::2] = 1.0
    tree = F.build_tree(torch.from_numpy(z).cuda(), [1] * n, offsets=list(range(0, 2 * n + 1, 2)))
    u = F.evaluate_log(F.plan(tree, 4, 0.5, "fp64"), torch.from_numpy(q).cuda()).cpu().numpy()[::2]
    # the kernel's r^2, rounded once: the smallest normal number is added to it
    r2 = (d.astype(np.longdouble) ** 2 + np.finfo(np.float64).tiny).astype(np.float64)
    ref = np.log(r2.astype(np.longdouble)) / 2
    live = ref != 0
    ulp = np.spacing(np.abs(ref[live]).astype(np.float64))
    err = np.abs((u[live].astype(np.longdouble) - ref[live]) / ulp)
    assert np.all(u[~live] == 0)
    assert float(err.max()) <= 0.6
