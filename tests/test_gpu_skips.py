"""Geometric skips read off the hardware logarithm (with the defined skip where
an integer is near), against the oracle bit for bit: success probabilities at
the ends of the single-precision range and around them, where the skips, and
with them the share of second looks, are largest and smallest."""
import numpy as np
import pytest

from tests.gpu_util import announce, dcs, first_mismatch, to_np_u64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [2.0 ** -10, 0.00101, 0.0123, 0.1, 0.5, 0.75, 0.97, 0.9999,
                               1.0 - 2.0 ** -20])
def test_single_precision_skips(ref, p):
    m = dcs()
    N = min(1 << 31, int(3_000_000 / p))
    announce(f"Bernoulli p={p} N={N}")
    out, cnt = m.sample_bernoulli(p, N, 11)
    m.synchronize()
    want = ref.bernoulli(p, N, 11)
    assert int(cnt.item()) == want.size
    got = to_np_u64(out)[:want.size]
    assert np.array_equal(got, want), first_mismatch(got, want)


@pytest.mark.parametrize("ratio,n0", [(2, 4096), (1.2, 4096), (15, 4096), (60, 2000), (7, 100)])
def test_dense_leaf_skips(ref, ratio, n0):
    m = dcs()
    n = 400_000
    N = int(n * ratio)
    announce(f"dense leaves n={n} N={N} n0={n0}")
    got = to_np_u64(m.sample(n, N, 12, n0=n0, dense_ratio=64))
    m.synchronize()
    want = ref.sample(n, N, 12, n0=n0, dense_ratio=64)
    assert np.array_equal(got, want), first_mismatch(got, want)
