"""P2M in segments of a leaf's sources: leaf sizes at the edges of a segment.

The leaf expansion W of a crowded box is compared with its definition, the sum of the
kernel between the check points and the box's sources in numpy; the tolerance is the
rounding of a sum of n terms of one sign pattern (n 2^-53, with a margin of 4).
"""
import numpy as np
import pytest

from parity_util import kernel_matrix

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel,param,tau", [("laplace", 0.0, 1e-4), ("gauss", 1.0, 1e-6),
                                              ("yukawa", 1.0, 1e-6)])
@pytest.mark.parametrize("n", [255, 256, 257, 512, 1500])
def test_segments(n, kernel, param, tau, oracle_lib):
    import torch

    from paper_1408_0210_amd import eifmm as E
    from paper_1408_0210_amd import workloads as W
    depth = 3
    # n sources in box 0, 300 in the last box, and one alone in between
    x = np.concatenate([W.uniform_points(n, 1) / 8.0, 0.875 + W.uniform_points(300, 2) / 8.0,
                        np.full((3, 1), 0.4)], axis=1)
    x = np.ascontiguousarray(x)
    s = W.potentials(x.shape[1], 3)
    plan = E.Plan(kernel, param, [0, 0, 0], 1.0, x.shape[1], depth, tau)
    plan.set_points(torch.from_numpy(x).cuda())
    plan.evaluate(torch.from_numpy(s).cuda())
    got = plan.export_expansion("W", depth)
    X = plan.level(depth)["X"]
    for key, sel, c in ((0, slice(0, n), 1 / 16), (511, slice(n, n + 300), 15 / 16)):
        K = kernel_matrix(oracle_lib, kernel, param, X, np.ascontiguousarray((x[:, sel] - c).T))
        want, size = K @ s[sel], np.abs(K) @ np.abs(s[sel])
        assert (np.abs(got[key] - want) <= 4.0 * K.shape[1] * 2.0 ** -53 * size).all(), key
    plan.close()
