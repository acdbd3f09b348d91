"""The work-group leaf sort at its edges, against the oracle bit for bit:
sizes around its blocks, rows and lines; every alignment of the output; the
bucket sizes at which it takes more rounds or the general sort (a bucket is
the words with equal top 13 bits; the seeds were searched on the CPU for
leaves whose largest bucket has the stated size); and leaves whose values
repeat, few (repaired in place) and many."""
import numpy as np
import pytest

from tests.gpu_util import announce, dcs, first_mismatch, to_np_u64

pytestmark = pytest.mark.gpu


def check(m, ref, variant, n, N, seed, n0=4096, shift=0):
    import torch
    announce(f"leaf sort: variant={variant} n={n} N={N} seed={seed} n0={n0} shift={shift}")
    buf = torch.full((n + 32,), -1, dtype=torch.int64, device="cuda")
    f = m.sample_replacement if variant else m.sample
    f(n, N, seed, out=buf[shift:shift + n], n0=n0)
    m.synchronize()
    got = to_np_u64(buf)
    want = (ref.replacement if variant else ref.sample)(n, N, seed, n0=n0)
    assert np.array_equal(got[shift:shift + n], want), first_mismatch(got[shift:shift + n], want)
    edge = np.uint64(2**64 - 1)
    assert (got[:shift] == edge).all() and (got[shift + n:] == edge).all()


@pytest.mark.parametrize("N", [1 << 32, (1 << 32) - 5, 3_000_000_019])
@pytest.mark.parametrize("n", [33, 111, 113, 255, 257, 1023, 1025, 2047, 2049, 3073, 4095])
def test_leaf_sizes(ref, n, N):
    m = dcs()
    for variant in (0, 1):
        check(m, ref, variant, n, N, n + variant)


@pytest.mark.parametrize("shift", range(16))
def test_output_alignment(ref, shift):
    check(dcs(), ref, 0, 4095 - shift, 1 << 32, 5 + shift, shift=shift)


# n = 4095 of 2^32: largest bucket 5, 6, 7, 9, 10 and 11
@pytest.mark.parametrize("seed", [1, 2, 31, 526884, 1498216, 7211155])
def test_bucket_sizes(ref, seed):
    m = dcs()
    for N in (1 << 32, (1 << 32) - 5):
        check(m, ref, 0, 4095, N, seed)


# values that repeat: a handful per leaf, about as many as are repaired in
# place, and far more (left to the general sort when the one-pass kernel is off)
@pytest.mark.parametrize("N", [1 << 24, 20_000_000, 400_009, 1 << 18, 300_007, 131_101])
def test_repeats(ref, N):
    m = dcs()
    try:
        for mask in (-1, 7):
            m.debug_leaf_kernels(mask)
            for seed in (1, 2, 3):
                check(m, ref, 0, 4090 + seed, N, seed, shift=seed)
                check(m, ref, 1, 4090 + seed, N, seed, shift=seed)
    finally:
        m.debug_leaf_kernels(-1)
