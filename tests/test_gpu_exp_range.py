"""e^(-r^2/h2) with an h2 whose reciprocal overflows: 1 at r = 0, 0 elsewhere."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h2", [1e-310, 5e-324, 1e-300])
def test_gauss_of_denormal_width(h2):
    import torch

    from paper_1408_0210_amd import eifmm as E
    from paper_1408_0210_amd import workloads as W
    n = 300
    x, s = W.uniform_points(n, 81), W.potentials(n, 82)
    x[:, n // 2:] = x[:, :n // 2]  # every point twice
    plan = E.Plan("gauss", h2, [0, 0, 0], 1.0, n, 1, 1e-6)
    plan.set_points(torch.from_numpy(x).cuda())
    f = plan.evaluate(torch.from_numpy(s).cuda()).cpu().numpy()
    pair = s[:n // 2] + s[n // 2:]
    assert np.array_equal(f, np.concatenate([pair, pair]))
    plan.close()
