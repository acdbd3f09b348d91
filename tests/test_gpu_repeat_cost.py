"""Leaves whose values repeat cost little more than leaves whose values don't
(GPU, times of one process's calls against each other, the least of several
runs on each side)."""
import time

import pytest

from tests.gpu_util import announce, dcs

pytestmark = pytest.mark.gpu


def least_us(call, sync, reps=100, runs=7):
    for _ in range(10):
        call()
    sync()
    best = float("inf")
    for _ in range(runs):
        t0 = time.perf_counter()
        for _ in range(reps):
            call()
        sync()
        best = min(best, (time.perf_counter() - t0) / reps * 1e6)
    return best


@pytest.mark.parametrize("n,repeats", [(4095, 16), (4095, 8), (3000, 19), (2000, 12)])
def test_one_leaf_is_no_slower_than_the_general_launches(n, repeats):
    """A sample of one leaf with a dozen expected repeats or so takes one
    launch; that launch is no slower than the tree and leaf launches that it
    stands for."""
    import torch
    m = dcs()
    N = n * n // (2 * repeats)
    out = torch.empty(n, dtype=torch.int64, device="cuda")
    announce(f"times of one leaf: n={n} N={N}")
    us = {}
    try:
        for mask in (0, -1):
            m.debug_leaf_kernels(mask)
            us[mask] = least_us(lambda: m.sample(n, N, 3, out=out), m.synchronize)
    finally:
        m.debug_leaf_kernels(-1)
    print(f"one leaf n={n} N={N}: {us[-1]:.1f} us, general launches {us[0]:.1f} us")
    assert us[-1] <= us[0], us
