"""Profile kinds of the leaf kernels (GPU): kind 5, the work-group kernel of the
dense leaves over ranges above 2^16, is timed where it is launched and counted
without time where no leaf can need it; small leaves are the one-wave kernel's
(12) and not the work-group kernel's (4)."""
import pytest

from tests.gpu_util import announce, dcs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dense_ratio,launched", [(None, False), (16, False), (64, True)])
def test_time_only_where_launched(dense_ratio, launched):
    m = dcs()
    announce(f"profile kind 5, dense ratio {dense_ratio}")
    n, N = 1 << 16, 40 << 16  # with ratio 64 dense leaves of up to 4095 * 40 elements
    try:
        m.profile_enable(True)
        for _ in range(3):
            m.sample(n, N, 5, dense_ratio=dense_ratio)
        m.synchronize()
        ms, count = m.profile_read(5)
    finally:
        m.profile_enable(False)
    assert count == 3
    assert (ms > 0.0) == launched


def test_small_leaves_are_left_to_the_one_wave_kernel():
    m = dcs()
    n, N = 1 << 23, 3 << 45  # 32768 leaves of about 256 values over ranges that are no powers of two
    announce("profile kinds 4 and 12")
    try:
        m.profile_enable(True)
        m.sample(n, N, 21)
        m.synchronize()
        (sort_ms, sort_n), (small_ms, small_n) = m.profile_read(4), m.profile_read(12)
    finally:
        m.profile_enable(False)
    assert (sort_n, small_n) == (1, 1)
    assert sort_ms < 0.5 * small_ms


@pytest.mark.parametrize("N,launched", [(1 << 20, 0), (1 << 21, 0), ((1 << 21) + 1, 1), (3 << 21, 1)])
def test_one_pass_kernel_is_left_out_of_dense_samples(ref, N, launched):
    """Where the sample is at least twice as dense as the line between dense and
    sparse leaves, no sparse leaf of more than 1024 values can plausibly occur,
    and the one-pass kernel (13) is not launched; the sample is the same."""
    import numpy as np
    from tests.gpu_util import first_mismatch, to_np_u64
    m = dcs()
    n = 1 << 18  # dense_ratio 16: the rule's line is at N = 2^21
    want = ref.sample(n, N, 6)
    for mask in (-1, 0, 7):
        announce(f"one-pass kernel of a dense sample: N={N} mask={mask}")
        m.debug_leaf_kernels(mask)
        try:
            m.profile_enable(True)
            got = to_np_u64(m.sample(n, N, 6))
            m.synchronize()
            count = m.profile_read(13)[1]
        finally:
            m.profile_enable(False)
            m.debug_leaf_kernels(-1)
        assert count == {-1: launched, 0: 1, 7: 0}[mask]
        assert np.array_equal(got, want), first_mismatch(got, want)
