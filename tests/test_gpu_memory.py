"""Device memory of a plan's sort: histogram bins for the digits that the depth uses.

4e7 points at depth 2 (6 key bits, one pass of 64 bins) against a plan of 1000 points: the
difference is the arrays per point below, rounded up by the allocator's pages.  512 bins, the
most that a digit has, would add 70 MB.
"""
import pytest

pytestmark = pytest.mark.gpu


def test_sort_histogram_follows_the_depth():
    import torch

    from paper_1408_0210_amd import eifmm as E

    def used(n):
        torch.cuda.synchronize()
        free0 = torch.cuda.mem_get_info()[0]
        plan = E.Plan("sqdist", 0.0, [0, 0, 0], 1.0, n, 2, 1e-6)
        free1 = torch.cuda.mem_get_info()[0]
        dpad = plan.stats()["dpad"][2]
        plan.close()
        return free0 - free1, dpad

    used(1000)  # the library's own first allocations
    small, dpad = used(1000)
    n = 40_000_000
    big, _ = used(n)
    # points (3 + 4 doubles), keys and indices twice, sigma, near field; chunks of 32
    # targets, segments of 256 sources and their sums; 64 bins per 1024 keys
    want = n * (7 * 8 + 4 * 4 + 2 * 8) + n // 32 * 4 + n // 256 * (4 + 8 * dpad) + n // 1024 * 64 * 4
    assert big - small <= want + 16 * (2 << 20), (big - small, want)
