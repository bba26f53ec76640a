"""Mixed batches take each problem's P2M as its own plan does.

W of the leaf level is P2M alone, so it has the same bits in a batch as from a plan of the
same problem: problems whose levels are all compressed (P2M by segments and the FP64
exponential of the kernel values) and problems that round What to FP32 (one sum per leaf,
the library's exponential), of one kernel in one batch, on crowded leaves.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_mixed_batch_p2m_as_plan():
    import torch

    from paper_1408_0210_amd import eifmm as E
    from paper_1408_0210_amd import workloads as W
    spec = [("yukawa", 1.0, 1e-4, 1e-3, 3, 6000), ("yukawa", 1.0, 1e-4, 0.0, 3, 5000),
            ("gauss", 0.05, 1e-4, 1e-3, 2, 4000), ("yukawa", 1.0, 1e-4, 1e-3, 2, 3000),
            ("gauss", 0.05, 1e-4, 0.0, 2, 2000), ("laplace", 0.0, 1e-4, 1e-3, 3, 3000)]
    probs, xs, ss = [], [], []
    for i, (kern, param, tau, ctol, depth, n) in enumerate(spec):
        probs.append(dict(kernel=kern, param=param, n=n, tau=tau, depth=depth, compress_tol=ctol))
        xs.append(torch.from_numpy(W.cluster_points(n, 3, 0.05, 400 + i, 420 + i)).cuda())
        ss.append(torch.from_numpy(W.potentials(n, 440 + i)).cuda())
    B = E.Batch(probs, precision="mixed")
    B.set_points(xs)
    fs = B.evaluate(ss)
    for i, q in enumerate(probs):
        plan = E.Plan(q["kernel"], q["param"], [0, 0, 0], 1.0, q["n"], q["depth"], q["tau"],
                      precision="mixed", compress_tol=q["compress_tol"])
        plan.set_points(xs[i])
        own = plan.evaluate(ss[i]).cpu().numpy()
        f = fs[i].cpu().numpy()
        k = q["depth"]
        assert np.array_equal(B.export_expansion(i, "W", k), plan.export_expansion("W", k)), (i, q)
        assert np.linalg.norm(f - own) < 1e-6 * np.linalg.norm(own), (i, q)
        plan.close()
    B.close()
