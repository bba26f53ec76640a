"""FP64 M2L of operators of at most 32 x 32 (FP64 matrix cores, no digits).

Against the oracle's Algorithm 3 (FP64, the same tables up to rounding) with one and with
two 16-row blocks, k walked in 2 to 8 steps (even and odd), tiles with few and many valid
columns, several right-hand sides, empty boxes and a potential that is not a number.  The
tolerance is the pass's elsewhere (1e-10); an operand out of place shows as 1e-3 or more.
"""
import numpy as np
import pytest

from parity_util import rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel,param,tau,ctol,depth,n,nrhs", [
    ("sqdist", 0.0, 1e-6, 0.0, 3, 1500, 1), ("laplace", 0.0, 1e-1, 0.0, 4, 3000, 3),
    ("gauss", 1.0, 1e-3, 0.0, 3, 1500, 1), ("gauss", 1.0, 1e-6, 0.0, 4, 9000, 1),
    ("gauss", 1.0, 1e-6, 0.0, 2, 40, 2), ("gauss", 1.0, 1e-7, 0.0, 3, 2000, 1),
    ("laplace", 0.0, 1e-4, 3e-2, 3, 1500, 2), ("advdiff", 1.0, 2e-1, 0.0, 3, 1500, 1)])
def test_small_m2l_matches_oracle(kernel, param, tau, ctol, depth, n, nrhs, oracle_lib):
    import torch

    from paper_1408_0210_amd import eifmm as E
    from paper_1408_0210_amd import workloads as W
    x = W.uniform_points(n, 51)
    x[:, ::4] *= 0.2  # boxes without points, and full ones
    sig = np.stack([W.potentials(n, 52 + r) for r in range(nrhs)])
    plan = E.Plan(kernel, param, [0, 0, 0], 1.0, n, depth, tau, compress_tol=ctol, max_rhs=nrhs)
    ref = oracle_lib.Plan(kernel, param, [0, 0, 0], 1.0, depth, tau, compress_tol=ctol)
    plan.set_points(torch.from_numpy(x).cuda())
    one = nrhs == 1
    f = plan.evaluate(torch.from_numpy(sig[0] if one else sig).cuda()).cpu().numpy().reshape(nrhs, n)
    dims = {k: plan.level(k)["d"] for k in range(2, depth + 1)}
    for r in range(nrhs):
        e = rel(f[r], ref.evaluate(x, sig[r]))
        assert e < 1e-10, (kernel, tau, dims, r, e)
    if kernel == "gauss" and depth == 3:
        sig[0, 0] = np.nan
        g = plan.evaluate(torch.from_numpy(sig[0]).cuda()).cpu().numpy()
        assert np.isnan(g).any()
    plan.close()
