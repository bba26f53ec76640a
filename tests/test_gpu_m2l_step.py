"""FP64 M2L step by itself: g of every box with an interaction list against K^delta What.

What and g are exported from the library, the sums formed in extended precision, box by
box.  Sources fill one corner leaf and separate targets others near and far, so that a
box's sum holds one offset or a few: kernels that decay over the interaction list then
show whether an operator of a far offset keeps its own digits beside the large entries of
the near ones.  The bound per box, over the rows (d terms, ma the largest |entry| of the
operator's row, mb of the source column):
  2^-55 (sqrt(d) ma mb + 8 |g| + (2 + 4 max|ln K|) (sum K^2 What^2)^(1/2)),
the first part for operands of 7 digits rounded at 2^-56 of their scale, the second for the
sums, the third for the rounding of the tables' kernel values.  A lost last digit of 1/r's
operators or sources is 1.8 to 3 times the bound, and one operator scale for all offsets
8 to 3e6 times it where K decays.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def check_step(oracle_lib, kernel, param, tau, nrhs, unit):
    import torch

    from paper_1408_0210_amd import eifmm as E
    from paper_1408_0210_amd import workloads as W
    depth, ns = 3, 40
    # target leaves: within reach of level 3 only, and of level 2 (parents 2 or 3 apart)
    leaves = [(2, 0, 0), (0, 3, 1), (3, 3, 3), (2, 2, 3), (7, 7, 7), (4, 1, 6), (0, 0, 5), (6, 3, 0)]
    src = W.uniform_points(ns, 71) / 8
    tgt = np.concatenate([(W.uniform_points(5, 72 + i) + np.array(c)[:, None]) / 8
                          for i, c in enumerate(leaves)], axis=1)
    src, tgt = np.ascontiguousarray(src), np.ascontiguousarray(tgt)
    sig = np.stack([W.potentials(ns, 90 + r) * 1e3 ** r for r in range(nrhs)])
    plan = E.Plan(kernel, param, [0, 0, 0], 1.0, ns, depth, tau, max_rhs=nrhs,
                  n_targets=tgt.shape[1])
    plan.set_points(torch.from_numpy(src).cuda(), targets=torch.from_numpy(tgt).cuda())
    plan.evaluate(torch.from_numpy(sig[0] if nrhs == 1 else sig).cuda())
    table = oracle_lib.offset_table().astype(np.float64)
    checked = 0
    for k in (2, 3):
        Y = plan.level(k)["Y"]
        X = plan.level(k, second=True)["X"] if kernel == "advdiff" else Y
        il = plan.export_lists(k)
        h = 2.0 ** -k
        for r in range(nrhs):
            what, g = plan.export_expansion("What", k, r), plan.export_expansion("g", k, r)
            for j, box in enumerate(il["active"]):
                ref = np.zeros(len(X), np.longdouble)
                sizes, rounding = np.zeros(len(X)), np.zeros(len(X))
                for q in range(il["il_ptr"][j], il["il_ptr"][j + 1]):
                    b = what[il["il_src"][q]]
                    if not b.any():
                        continue
                    z = X[:, None, :] - (Y[None, :, :] + h * table[il["il_off"][q]])
                    K = oracle_lib.kernel_eval(kernel, param, z.reshape(-1, 3)).reshape(len(X), len(Y))
                    ref += K.astype(np.longdouble) @ b
                    sizes += np.sqrt(len(Y)) * np.abs(K).max(1) * np.abs(b).max()
                    rounding += (2 + 4 * np.abs(np.log(K)).max()) * np.sqrt(K ** 2 @ b ** 2)
                    checked += 1
                tol = unit * (sizes + 8 * np.abs(ref).astype(np.float64) + rounding)
                err = np.abs(g[box] - ref).astype(np.float64)
                e, t = np.sqrt((err ** 2).mean()), np.sqrt((tol ** 2).mean())
                assert e <= t, (kernel, param, k, int(box), r, e / max(t, 1e-300))
    assert checked >= 8 * nrhs
    plan.close()


@pytest.mark.parametrize("nrhs", [1, 3])
@pytest.mark.parametrize("kernel,param,tau", [
    ("laplace", 0.0, 1e-6), ("yukawa", 30.0, 1e-6), ("gauss", 0.03, 1e-6), ("yukawa", 60.0, 1e-4),
    ("advdiff", 20.0, 1e-4)])
def test_m2l_step_far_offsets(kernel, param, tau, nrhs, oracle_lib):
    check_step(oracle_lib, kernel, param, tau, nrhs, 2.0 ** -55)


# one 64-element chunk and two, tiles of 3, 4, 6 and 8 row blocks, 8 digits of a few blocks:
# fewer rows and terms average less, so the bound is the digits' own worst rounding, 2^-54
@pytest.mark.parametrize("kernel,param,tau", [
    ("gauss", 1.0, 1e-6), ("mq", 1.0, 1e-9), ("laplace", 0.0, 1e-3), ("gauss", 0.1, 1e-6)])
def test_m2l_step_small_sizes(kernel, param, tau, oracle_lib):
    check_step(oracle_lib, kernel, param, tau, 3, 2.0 ** -54)
