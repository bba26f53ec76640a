"""Mixed-precision M2L: every tile height, chunk length and column remainder.

The mixed pass is compared with the oracle's Algorithm 3 in FP64 (the same tables up to
rounding); the tolerance, 1e-6 of the 2-norm, is the one the mixed pass has elsewhere: a
product of FP32 operands over d <= 288 values leaves about sqrt(d) 2^-24 = 1e-6 of its
largest term, a fragment that is lost or out of place 1e-2 or more.
"""
import numpy as np
import pytest

from parity_util import rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch

    from paper_1408_0210_amd import eifmm as E
    from paper_1408_0210_amd import workloads as W
    return torch, E, W


# d or rank of one block to 18: tiles of 2, 3, 4, 5, 6, 8 and 9 blocks, whole and with
# idle blocks, chunks of 3 and of 4 16-k steps, the last one whole and not
@pytest.mark.parametrize("kernel,param,tau,ctol", [
    ("gauss", 1.0, 1e-6, 0.0), ("mq", 1.0, 1e-4, 0.0), ("laplace", 0.0, 1e-1, 0.0),
    ("laplace", 0.0, 1e-2, 0.0), ("laplace", 0.0, 3e-3, 0.0), ("laplace", 0.0, 1e-3, 0.0),
    ("laplace", 0.0, 1e-4, 0.0), ("laplace", 0.0, 1e-4, 6e-4), ("laplace", 0.0, 1e-6, 6e-6),
    ("yukawa", 1.0, 1e-5, 0.0), ("laplace", 0.0, 1e-6, 0.0)])
def test_mixed_m2l_matches_oracle(kernel, param, tau, ctol, gpu, oracle_lib):
    torch, E, W = gpu
    n = 1500
    # most boxes of one corner empty: offsets without a source for whole waves
    x = W.uniform_points(n, 21)
    x[:, ::3] *= 0.3
    sig = np.stack([W.potentials(n, 22 + r) for r in range(3)])
    plan = E.Plan(kernel, param, [0, 0, 0], 1.0, n, 3, tau, compress_tol=ctol, max_rhs=3,
                  precision="mixed")
    ref = oracle_lib.Plan(kernel, param, [0, 0, 0], 1.0, 3, tau, compress_tol=ctol)
    plan.set_points(torch.from_numpy(x).cuda())
    f = plan.evaluate(torch.from_numpy(sig).cuda()).cpu().numpy()
    one = plan.evaluate(torch.from_numpy(sig[1]).cuda()).cpu().numpy()
    for r in range(3):
        want = ref.evaluate(x, sig[r])
        assert rel(f[r], want) < 1e-6, (kernel, tau, r, rel(f[r], want))
    assert rel(one, ref.evaluate(x, sig[1])) < 1e-6, (kernel, tau)
    plan.close()
