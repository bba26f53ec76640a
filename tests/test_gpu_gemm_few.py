"""Translations and projections of few columns (one wave per 48 rows of 16 columns).

The pass against the oracle's Algorithm 3 where this form can go wrong: 1 to 10 row blocks
(whole groups of 3 and remainders), one box to a few hundred columns per level, several
right-hand sides, empty children and parents, compressed levels (projections) and the two
sizes of two EIMs.  The tolerance is the pass's elsewhere (1e-10).
"""
import numpy as np
import pytest

from parity_util import assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel,tau,ctol,depth,n,nrhs", [
    ("sqdist", 1e-6, 0.0, 3, 700, 1), ("laplace", 1e-1, 0.0, 4, 300, 1),
    ("laplace", 1e-2, 0.0, 3, 900, 3), ("laplace", 1e-3, 0.0, 4, 4000, 2),
    ("laplace", 1e-4, 6e-4, 4, 2500, 1), ("laplace", 1e-4, 6e-4, 3, 40, 5),
    ("advdiff", 1e-2, 0.0, 3, 1500, 1), ("yukawa", 1e-4, 0.0, 4, 12, 1)])
def test_few_columns_match_oracle(kernel, tau, ctol, depth, n, nrhs, oracle_lib):
    import torch

    from paper_1408_0210_amd import eifmm as E
    from paper_1408_0210_amd import workloads as W
    param = 1.0 if kernel in ("yukawa", "advdiff") else 0.0
    x = W.uniform_points(n, 61)
    x[:, ::3] *= 0.25
    sig = np.stack([W.potentials(n, 62 + r) for r in range(nrhs)])
    plan = E.Plan(kernel, param, [0, 0, 0], 1.0, n, depth, tau, compress_tol=ctol, max_rhs=nrhs)
    ref = oracle_lib.Plan(kernel, param, [0, 0, 0], 1.0, depth, tau, compress_tol=ctol)
    plan.set_points(torch.from_numpy(x).cuda())
    s = torch.from_numpy(sig if nrhs > 1 else sig[0]).cuda()
    f = plan.evaluate(s).cpu().numpy().reshape(nrhs, n)
    for r in range(nrhs):
        assert_close(f[r], ref.evaluate(x, sig[r]), 1e-10, f"{kernel} tau {tau} rhs {r}")
    plan.close()
