"""The triangular solves by four waves per 16 columns, at the edges of their tiles.

A solve is checked by its residual: M What = W and M^T lhat = l are reproduced to the
rounding of the products, whatever the condition of M = K(X, Y) (the bounds that the
other parity tests use).  d runs from one 16-row tile over a tile count that leaves waves
without a row to more rows than a wave loads ahead; the columns from one to several
groups of 16, and past the count up to which this form serves.
"""
import pytest

from parity_util import kernel_matrix, solve_residual

pytestmark = pytest.mark.gpu


# tau -> d: sqdist 5, then 1/r with growing d (about 14, 49, 146, 287, 465)
@pytest.mark.parametrize("kernel,tau,n,depth", [
    ("sqdist", 1e-6, 200, 2), ("laplace", 1e-1, 1, 2), ("laplace", 1e-2, 700, 3),
    ("laplace", 1e-4, 900, 3), ("laplace", 1e-6, 20, 2), ("laplace", 1e-8, 300, 2),
    ("laplace", 1e-3, 60000, 5)])
def test_solve_residuals(kernel, tau, n, depth, oracle_lib):
    import torch

    from paper_1408_0210_amd import eifmm as E
    from paper_1408_0210_amd import workloads as W
    plan = E.Plan(kernel, 0.0, [0, 0, 0], 1.0, n, depth, tau)
    plan.set_points(torch.from_numpy(W.uniform_points(n, 4)).cuda())
    plan.evaluate(torch.from_numpy(W.potentials(n, 5)).cuda())
    for k in range(2, depth + 1):
        lv = plan.level(k)
        M = kernel_matrix(oracle_lib, kernel, 0.0, lv["X"], lv["Y"])
        r2, rb = solve_residual(M, plan.export_expansion("What", k), plan.export_expansion("W", k))
        assert r2 <= 1e-12 and rb <= 1e-11, ("What", k, lv["d"], r2, rb)
    if n > 1:  # (one point has no far field: l = 0)
        r2, rb = solve_residual(M, plan.export_expansion("lhat", depth),
                                plan.export_expansion("l", depth), transpose=True)
        assert r2 <= 1e-12 and rb <= 1e-11, ("lhat", lv["d"], r2, rb)
    plan.close()
