"""The near field's exponential over its whole range, down to the denormals and to zero.

One source and many targets, a tree of one box: f is one kernel value per target.  The
exponent x carries a few roundings (r^2, the product with the parameter), which the
exponential turns into a relative error of |x| each; the value itself adds a few more:
(6 + 6 |x|) 2^-53 relative, plus the spacing of the denormals.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel,param", [("gauss", 1.0), ("gauss", 0.01), ("gauss", 0.0025),
                                          ("yukawa", 1.0), ("yukawa", 500.0), ("yukawa", 0.0),
                                          ("advdiff", 3.0)])
def test_kernel_values(kernel, param):
    import torch

    from paper_1408_0210_amd import eifmm as E
    n = 4001
    t = np.linspace(0.0, 1.0, n)[1:]
    tgt = np.ascontiguousarray(np.stack([t, t * t, 0.7 * t]))
    src = np.zeros((3, 1))
    plan = E.Plan(kernel, param, [0, 0, 0], 1.0, 1, 0, 1e-6, n_targets=tgt.shape[1])
    plan.set_points(torch.from_numpy(src).cuda(), torch.from_numpy(tgt).cuda())
    f = plan.evaluate(torch.ones(1, dtype=torch.float64, device="cuda")).cpu().numpy()
    z = tgt.astype(np.longdouble)
    r2 = (z ** 2).sum(0)
    r = np.sqrt(r2)
    x = {"gauss": -r2 / np.longdouble(param) if param else 0 * r2, "yukawa": -param * r,
         "advdiff": param * (z[0] - r)}[kernel]
    want = np.exp(x) / (1 if kernel == "gauss" else r)
    # the argument of advdiff cancels: its roundings are relative to r
    size = param * r if kernel == "advdiff" else np.abs(x)
    tol = (6 + 6 * size) * np.longdouble(2) ** -53 * want + np.longdouble(2) ** -1073
    assert (np.abs(f - want) <= tol).all()
    plan.close()
