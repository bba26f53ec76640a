"""Translations and projections of many columns (tall tiles of 5 to 9 row blocks).

9 right-hand sides on the 4096 leaves of a depth-4 tree give the 36,000 columns that take
this form, with a ragged last tile per class.  Row blocks from 5 to 10 (whole tiles, idle
blocks, two row tiles), and a compressed plan for the projections.  One column is compared
with the oracle's Algorithm 3 (1e-10, as the pass elsewhere); the others are that potential
times powers of two and have to be its result times the same power up to the order of the
upward sums (1e-12).
"""
import numpy as np
import pytest

from parity_util import assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tau,ctol", [(2e-3, 0.0), (1e-3, 0.0), (4e-4, 0.0), (2e-4, 0.0),
                                      (1e-4, 6e-4)])
def test_many_columns_match_oracle(tau, ctol, oracle_lib):
    import torch

    from paper_1408_0210_amd import eifmm as E
    from paper_1408_0210_amd import workloads as W
    n, nrhs = 20000, 9
    x = W.uniform_points(n, 71)
    s = W.potentials(n, 72)
    plan = E.Plan("laplace", 0.0, [0, 0, 0], 1.0, n, 4, tau, compress_tol=ctol, max_rhs=nrhs)
    ref = oracle_lib.Plan("laplace", 0.0, [0, 0, 0], 1.0, 4, tau, compress_tol=ctol)
    plan.set_points(torch.from_numpy(x).cuda())
    sig = np.stack([s * 2.0 ** (r - 4) for r in range(nrhs)])
    f = plan.evaluate(torch.from_numpy(sig).cuda()).cpu().numpy()
    d = plan.level(4)["d"]
    assert_close(f[4], ref.evaluate(x, s), 1e-10, f"tau {tau} d {d}")
    for r in range(nrhs):
        assert_close(f[r] * 2.0 ** (4 - r), f[4], 1e-12, f"tau {tau} d {d} column {r}")
    plan.close()
