"""Leaves of at most 1024 values sorted by one wave (ranges that are no powers
of two): few and many repeats, words that the range voids, one job per wave and
many, against the oracle bit for bit."""
import numpy as np
import pytest

from tests.gpu_util import announce, dcs, first_mismatch, to_np_u64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("N", [5, 1009, 8009, 16_001, 40_009, 1_000_003, 2_200_000_009])
@pytest.mark.parametrize("n", [34, 300, 1000, 1024])
def test_single_leaves(ref, n, N, variant):
    if variant == 0 and n > N:
        pytest.skip("more values than the range holds")
    m = dcs()
    announce(f"small sort: variant={variant} n={n} N={N}")
    f, g = (m.sample_replacement, ref.replacement) if variant else (m.sample, ref.sample)
    got = to_np_u64(f(n, N, 3, n0=1025))
    m.synchronize()
    want = g(n, N, 3, n0=1025)
    assert np.array_equal(got, want), first_mismatch(got, want)


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("n,N,n0", [(2_000_000, 10**12 + 39, 700), (1_500_000, 50_000_017, 300),
                                    (900_000, 3 * 10**13 + 1, 1025), (700_000, 14_000_029, 1025)])
def test_many_leaves(ref, n, N, n0, variant):
    m = dcs()
    announce(f"small sort: variant={variant} n={n} N={N} n0={n0}")
    f, g = (m.sample_replacement, ref.replacement) if variant else (m.sample, ref.sample)
    got = to_np_u64(f(n, N, 4, n0=n0))
    m.synchronize()
    want = g(n, N, 4, n0=n0)
    assert np.array_equal(got, want), first_mismatch(got, want)


@pytest.mark.parametrize("n,N,n0", [(300, 5003, 4096), (1500, 60_013, 4096), (40, 1009, 4096)])
def test_new_values_at_a_leaf_s_ends(ref, n, N, n0):
    """Repairs of leaves that start at a line of the output, over enough seeds
    for new values below the first and above the last one (each new value is
    either with probability 1/n)."""
    m = dcs()
    announce(f"repairs at a leaf's ends: n={n} N={N}, 300 seeds")
    for seed in range(300):
        got = to_np_u64(m.sample(n, N, seed, n0=n0))
        m.synchronize()
        want = ref.sample(n, N, seed, n0=n0)
        assert np.array_equal(got, want), f"seed {seed}: {first_mismatch(got, want)}"
