"""Leaves of many points where the near field runs on the second stream and gathers
the strengths itself (more than 64 points per leaf), and its neighbours: one
stream below 16,385 points with split lists and below 2049 points with more than 32
terms.  Every form of the evaluation against the direct sum (converged orders;
1e-12 FP64, 1e-6 mixed) and against each other to the bit."""
import numpy as np
import pytest

from paper_1311_1006_amd import workloads as W

from gpu_util import dev, e2, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,bar", [("fp64", 1e-12), ("mixed", 1e-6)])
@pytest.mark.parametrize("n,L,p", [(2048, 3, 44), (2049, 3, 44), (9000, 4, 48), (2049, 2, 64), (16384, 4, 46),
                                   (16385, 4, 32), (33000, 6, 46)])
def test_evaluations_agree(orc, prec, bar, n, L, p):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1311_1006_amd as F
    z, m, _ = W.uniform(n, seed=n + p)
    tree, md = F.build_tree(dev(z), L), dev(m)
    pl = F.plan(tree, p, 0.5, prec)
    phi = host(F.evaluate(pl, md))                     # lists pending
    sub = np.arange(0, n, max(1, n // 2000))
    # 32 terms leave 2^-32 and a constant
    assert e2(phi[sub], orc.direct_points(z, m, z[sub])) <= (bar if p > 32 else max(bar, 1e-8))
    assert np.array_equal(host(F.evaluate(pl, md)), phi)
    out = dev(np.zeros(n, np.complex128))
    F.evaluate_static(pl, md, out)
    assert np.array_equal(host(out), phi)
    g = F.plan(tree, p, 0.5, prec, graph=True)
    gout = dev(np.zeros(n, np.complex128))
    other = dev(m[::-1])
    for _ in range(3):                                 # replays, eager work of other strengths between
        gout.zero_()
        F.evaluate(g, md, gout)
        F.evaluate(pl, other)
        assert np.array_equal(host(gout), phi)
    near, far = F.evaluate_parts(pl, md)
    assert e2(host(near) + host(far), phi) <= 1e-15


def every_form(F, pl, m, g, q, y):
    """Each evaluation of the plan's multipoles and local expansions, on the host."""
    import torch
    md = dev(m)
    out = {"phi": F.evaluate(pl, md)}
    near, far = F.evaluate_parts(pl, md)
    out["parts"] = near + far
    out["field"], out["dphi"] = F.evaluate_field(pl, md)
    out["gm"], out["gz"] = F.evaluate_adjoint(pl, md, dev(g))
    out["u"] = F.evaluate_log(pl, torch.from_numpy(q).cuda())
    out["points"], out["dpoints"] = F.evaluate_points(pl, md, dev(y), field=True)
    return {k: host(v) for k, v in out.items()}


@pytest.mark.parametrize("prec,bar", [("fp64", 1e-12), ("mixed", 1e-6)])
@pytest.mark.parametrize("n,L,p", [(4096, 3, 46), (4097, 3, 46), (16385, 4, 46), (4097, 3, 16), (9001, 3, 30),
                                   (65537, 5, 17)])
def test_p2m_and_l2p_of_their_own(orc, prec, bar, n, L, p):
    # 256 points per leaf and more: against the direct sums (0.5^p and a constant
    # of ten, the derivative p times that) and level by level
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1311_1006_amd as F
    z, m, _ = W.uniform(n, seed=n + p)
    rng = np.random.default_rng(n)
    g, q, y = rng.normal(size=n) + 1j * rng.normal(size=n), rng.normal(size=n), W.uniform(501, seed=3)[0]
    tree = F.build_tree(dev(z), L)
    got = every_form(F, F.plan(tree, p, 0.5, prec), m, g, q, y)
    lev = every_form(F, F.plan(tree, p, 0.5, prec, levelwise=True), m, g, q, y)
    for k in got:
        assert e2(got[k], lev[k]) <= bar, k
    assert np.array_equal(got["phi"], got["field"])
    sub = np.arange(0, n, max(1, n // 700))
    tol = max(bar, 10 * 0.5 ** p)
    assert e2(got["phi"][sub], orc.direct_points(z, m, z[sub])) <= tol
    assert e2(got["parts"], got["phi"]) <= 1e-15
    assert e2(got["dphi"][sub], orc.direct_deriv_points(z, m, z[sub])) <= p * tol
    assert e2(got["u"][sub], orc.direct_log_points(z, q, z[sub])) <= tol
    assert e2(got["points"], orc.direct_points(z, m, y)) <= tol
    if n < 10000:
        gm, gz = orc.grad_direct(z, m, g)
        assert e2(got["gm"], gm) <= tol and e2(got["gz"], gz) <= p * tol


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("sizes,Ls", [((4097, 300, 5000), (3, 3, 3)), ((4097, 9000), (3, 3)),
                                      ((4097, 700, 40, 17000, 700), (3, 2, 1, 4, 4)), ((40, 17000), (1, 4)),
                                      ((70000, 3000), (5, 5)), ((3000, 70000, 500), (5, 5, 4))])
@pytest.mark.parametrize("p", [16, 46])
def test_fat_and_thin_problems_in_one_call(prec, sizes, Ls, p):
    # problems with and without launches of their own, of one depth and of several,
    # against each alone (run level by level where the depths differ): to the bit
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1311_1006_amd as F
    zs = [W.uniform(n, seed=n + i)[0] for i, n in enumerate(sizes)]
    ms = [W.uniform(n, seed=n + i)[1] for i, n in enumerate(sizes)]
    off = np.concatenate([[0], np.cumsum(sizes)]).tolist()
    pl = F.plan(F.build_tree(dev(np.concatenate(zs)), list(Ls), offsets=off), p, 0.5, prec)
    mc = dev(np.concatenate(ms))
    phi, (fphi, dphi) = host(F.evaluate(pl, mc)), (host(x) for x in F.evaluate_field(pl, mc))
    assert np.array_equal(phi, fphi)
    for b, n in enumerate(sizes):
        one = F.plan(F.build_tree(dev(zs[b]), Ls[b]), p, 0.5, prec, levelwise=len(set(Ls)) > 1)
        part = slice(off[b], off[b + 1])
        assert np.array_equal(phi[part], host(F.evaluate(one, dev(ms[b])))), b
        assert np.array_equal(dphi[part], host(F.evaluate_field(one, dev(ms[b]))[1])), b
