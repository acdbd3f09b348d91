"""Leaves whose values repeat: they cost little more than leaves whose values
don't (times of one process's calls against each other, the least of several
runs on each side), and around the rules that choose how they are sampled they
are the oracle's, bit for bit."""
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


@pytest.mark.parametrize("n,N,n0", [(1 << 20, 17 << 20, 1024), (1 << 16, 17 << 16, 1024)])
def test_small_leaves_of_many_repeats_cost_little_more(n, N, n0):
    """A sample in small leaves of about 20 repeats each takes at most one and
    a half times what the same number of values takes without repeats."""
    import torch
    m = dcs()
    out = torch.empty(n, dtype=torch.int64, device="cuda")
    announce(f"times of small leaves: n={n} N={N} n0={n0}")
    few = least_us(lambda: m.sample(n, 6000 * N + 1, 3, out=out, n0=n0), m.synchronize)
    many = least_us(lambda: m.sample(n, N, 3, out=out, n0=n0), m.synchronize)
    print(f"small leaves n={n} n0={n0}: {few:.1f} us without repeats, {many:.1f} us with")
    assert many <= 1.5 * few, (few, many)


# leaves of one job each: n^2 around 2 N (one repeat expected), and ranges
# around the largest that has a bit per value (37632)
@pytest.mark.parametrize("n,Ns", [(33, [67, 543, 544, 545]), (40, [799, 800, 801]), (273, [37200, 37264, 37300, 40000]),
                                  (274, [37537, 37538, 37539, 37631, 37632, 37633]),
                                  (1000, [2003, 16001, 32767, 32768, 37632, 37633, 40001]),
                                  (1024, [2049, 16385, 37631, 37632, 37633])])
def test_small_leaves_around_the_rules(ref, n, Ns):
    """Small leaves of a batch, each its own job, against the oracle bit for
    bit: on both sides of the rule that chooses marks over the sort, every
    alignment of the output, several rounds of repeats."""
    import numpy as np
    import torch
    from tests.gpu_util import first_mismatch, to_np_u64
    m = dcs()
    specs, wants, off = [], [], 0
    for i in range(48):
        N = Ns[i % len(Ns)]
        specs.append(m.InstanceSpec(n=n, N=N, seed=i, out_offset=off, n0=4096, dense_ratio=2))
        wants.append((off, ref.sample(n, N, i, n0=4096, dense_ratio=2)))
        off += n + (i % 5 == 0)
    out = torch.zeros(off, dtype=torch.int64, device="cuda")
    announce(f"small leaves around the rules: n={n} Ns={Ns}")
    m.Batch(specs).run(out)
    m.synchronize()
    got = to_np_u64(out)
    for (o, want), spec in zip(wants, specs):
        assert np.array_equal(got[o:o + n], want), (spec.N, spec.seed,
                                                    first_mismatch(got[o:o + n], want))


# n^2 = 2 N and one less and more, where one launch changes to the other
@pytest.mark.parametrize("n", [5, 8, 33, 200, 1024, 1025, 3000, 4094, 4095])
def test_one_leaf_around_one_expected_repeat(ref, n):
    import numpy as np
    from tests.gpu_util import first_mismatch, to_np_u64
    m = dcs()
    for N in (n * n // 2 - 1, n * n // 2, n * n // 2 + 1):
        for seed in range(3):
            announce(f"one leaf around one repeat: n={n} N={N} seed={seed}")
            got = to_np_u64(m.sample(n, N, seed, dense_ratio=2))
            m.synchronize()
            want = ref.sample(n, N, seed, dense_ratio=2)
            assert np.array_equal(got, want), first_mismatch(got, want)
