"""FP64 batches of problems with operators of at most 32 x 32.

Their M2L takes the kernel that a single plan takes for them (packed columns), which the
executed flops show: k in steps of 4 up to d instead of whole 64-element chunks.  Results
against the oracle's Algorithm 3 (1e-10, as the pass elsewhere) and each problem's own plan:
one and two 16-row blocks, several operator sets and levels, more jobs than a wave has
lanes, a problem without points, a level of larger operators beside the small ones.
"""
import numpy as np
import pytest

from parity_util import rel

pytestmark = pytest.mark.gpu


def test_batch_of_small_operators(oracle_lib):
    import torch

    from paper_1408_0210_amd import eifmm as E
    from paper_1408_0210_amd import workloads as W
    spec = [("gauss", 1.0, 1e-6, 4, 9000), ("mq", 1.0, 1e-6, 3, 1500), ("gauss", 1.0, 1e-6, 3, 2500),
            ("gauss", 1.0, 1e-3, 4, 5000), ("mq", 2.0, 1e-4, 4, 4000), ("gauss", 1.0, 1e-6, 2, 0),
            ("laplace", 0.0, 1e-3, 3, 3000), ("gauss", 2.0, 1e-5, 5, 20000)]
    probs, xs, ss = [], [], []
    for i, (kern, param, tau, depth, n) in enumerate(spec):
        x = W.uniform_points(n, 300 + i)
        x[:, ::3] *= 0.3  # boxes without points
        probs.append(dict(kernel=kern, param=param, n=n, tau=tau, depth=depth))
        xs.append(torch.from_numpy(np.ascontiguousarray(x)).cuda())
        ss.append(torch.from_numpy(W.potentials(n, 320 + i)).cuda())
    B = E.Batch(probs)
    B.set_points(xs)
    for rep in range(2):
        fs = B.evaluate(ss)
    for i, q in enumerate(probs):
        if q["n"] == 0:
            continue
        plan = E.Plan(q["kernel"], q["param"], [0, 0, 0], 1.0, q["n"], q["depth"], q["tau"])
        plan.set_points(xs[i])
        own = plan.evaluate(ss[i]).cpu().numpy()
        f = fs[i].cpu().numpy()
        assert rel(f, own) < 1e-12, (i, q)
        ref = oracle_lib.Plan(q["kernel"], q["param"], [0, 0, 0], 1.0, q["depth"], q["tau"])
        e = rel(f, ref.evaluate(xs[i].cpu().numpy(), ss[i].cpu().numpy()))
        assert e < 1e-10, (i, q, e)
        sb, sp = B.stats(i), plan.stats()
        if q["depth"] > 3 or sp["d"][2] <= 32:  # (else a single plan takes level 2 by offset)
            assert min(sp["d"].values()) <= 32, (i, sp["d"])
            assert sb["m2l_flops_exec"] == sp["m2l_flops_exec"], (i, q)
        plan.close()
    B.close()


def test_small_operators_not_finite_potential():
    """A potential that is not a number reaches, through the M2L, points that are not near."""
    import torch

    from paper_1408_0210_amd import eifmm as E
    from paper_1408_0210_amd import workloads as W
    n = 2000
    x = W.uniform_points(n, 340)
    x[:, 0] = 0.01
    s = W.potentials(n, 341)
    s[0] = np.nan
    far = x.max(0) > 0.5  # two leaves of depth 3 and more away from the corner
    sig, pts = torch.from_numpy(s).cuda(), torch.from_numpy(x).cuda()
    plan = E.Plan("gauss", 1.0, [0, 0, 0], 1.0, n, 3, 1e-6)
    plan.set_points(pts)
    f = plan.evaluate(sig).cpu().numpy()
    assert np.isnan(f[far]).all()
    plan.close()
    B = E.Batch([dict(kernel="gauss", param=1.0, n=n, tau=1e-6, depth=3)])
    B.set_points([pts])
    assert np.isnan(B.evaluate([sig])[0].cpu().numpy()[far]).all()
    B.close()


@pytest.mark.parametrize("kernel,param,tau,depth", [
    ("sqdist", 0.0, 1e-6, 3), ("gauss", 0.02, 1e-4, 2), ("laplace", 0.0, 1e-3, 2)])
def test_batch_of_one_kind_of_level(kernel, param, tau, depth):
    """Only small operators, only steep levels, only levels of seven digits: the other
    launches are empty."""
    import torch

    from paper_1408_0210_amd import eifmm as E
    from paper_1408_0210_amd import workloads as W
    ns = (1500, 700)
    xs = [torch.from_numpy(W.uniform_points(n, 360 + n)).cuda() for n in ns]
    ss = [torch.from_numpy(W.potentials(n, 370 + n)).cuda() for n in ns]
    B = E.Batch([dict(kernel=kernel, param=param, n=n, tau=tau, depth=depth) for n in ns])
    B.set_points(xs)
    for rep in range(2):
        fs = B.evaluate(ss)
    for i, n in enumerate(ns):
        plan = E.Plan(kernel, param, [0, 0, 0], 1.0, n, depth, tau)
        plan.set_points(xs[i])
        own = plan.evaluate(ss[i]).cpu().numpy()
        assert rel(fs[i].cpu().numpy(), own) < 1e-12, (kernel, i)
        plan.close()
    B.close()
