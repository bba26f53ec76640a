"""FP64 M2L on the int8 matrix cores: the digits carry the whole FP64 operand.

The far field of the library is compared with the oracle's Algorithm 3 (FP64 loops, the
same tables up to rounding) where a digit can go wrong: sizes at the edges of the 64-element
chunks and of the tiles, sources spread over many binary orders, empty boxes and whole
classes without a source, several right-hand sides, and potentials that are not finite.
The tolerance is the one the pass's parity has elsewhere (1e-10): a lost digit shows as
2^-48 = 4e-15 of the largest term at the least significant end and as 2^-8 at the other.
"""
import numpy as np
import pytest

from parity_util import assert_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch

    from paper_1408_0210_amd import eifmm as E
    from paper_1408_0210_amd import workloads as W
    return torch, E, W


# (kernel, parameter, tau, compression): d or rank below one chunk, just past one, and
# of several chunks; tile heights of 2, 3, 4, 6 and 8 row blocks
@pytest.mark.parametrize("kernel,param,tau,ctol", [
    ("mq", 1.0, 1e-4, 0.0), ("gauss", 1.0, 1e-6, 0.0), ("laplace", 0.0, 1e-3, 0.0),
    ("laplace", 0.0, 1e-4, 6e-4), ("laplace", 0.0, 1e-6, 6e-6), ("cosr", 20.0, 1e-4, 0.0)])
def test_digit_m2l_matches_oracle(kernel, param, tau, ctol, gpu, oracle_lib):
    torch, E, W = gpu
    x, s = W.uniform_points(1500, 11), W.potentials(1500, 12)
    # potentials over 12 decades: boxes of very different magnitude feed one target
    s = s * 10.0 ** (np.arange(1500) % 13 - 6.0)
    plan = E.Plan(kernel, param, [0, 0, 0], 1.0, 1500, 3, tau, compress_tol=ctol)
    ref = oracle_lib.Plan(kernel, param, [0, 0, 0], 1.0, 3, tau, compress_tol=ctol)
    plan.set_points(torch.from_numpy(x).cuda())
    f = plan.evaluate(torch.from_numpy(s).cuda()).cpu().numpy()
    assert_close(f, ref.evaluate(x, s), 1e-10, f"{kernel} tau {tau}")
    plan.close()


def test_digit_m2l_rhs_empty_boxes_and_non_finite(gpu, oracle_lib):
    torch, E, W = gpu
    # two far corners of the domain: most boxes empty, most offsets without a source
    x = np.concatenate([W.uniform_points(300, 1) * 0.2, W.uniform_points(333, 2) * 0.15 + 0.85],
                       axis=1)
    x = np.ascontiguousarray(x)
    n = x.shape[1]
    sig = np.stack([W.potentials(n, q) for q in range(3)])
    sig[1] *= 1e-200
    sig[2] = 0.0
    plan = E.Plan("laplace", 0.0, [0, 0, 0], 1.0, n, 3, 1e-6, max_rhs=3)
    ref = oracle_lib.Plan("laplace", 0.0, [0, 0, 0], 1.0, 3, 1e-6)
    plan.set_points(torch.from_numpy(x).cuda())
    f = plan.evaluate(torch.from_numpy(sig).cuda()).cpu().numpy()
    assert_close(f[0], ref.evaluate(x, sig[0]), 1e-10, "first potential")
    assert_close(f[1] * 1e200, ref.evaluate(x, sig[1] * 1e200), 1e-10, "small potential")
    assert not f[2].any()
    # a potential that is not a number reaches the far targets as such
    bad = sig[0].copy()
    bad[0] = np.nan
    g = plan.evaluate(torch.from_numpy(bad).cuda()).cpu().numpy()
    assert np.isnan(g[300:]).all()
    plan.close()
