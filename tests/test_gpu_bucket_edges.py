"""The leaf sort's buckets (words with equal leading bits) at its two limits,
against the oracle bit for bit: 8 keys, the most that the row pass takes, at
every place about a row's edge, and 9 and 10, which go to the general sort.  The
seeds were searched on the CPU; the largest bucket of each is counted again
here, from the oracle's stream words."""
import numpy as np
import pytest

from tests.gpu_util import announce, dcs, first_mismatch, to_np_u64

pytestmark = pytest.mark.gpu

ROW = 112  # positions a row writes


def largest_bucket(ref, seed, n, bits):
    """(keys, first position) of the largest bucket of a root leaf's first n
    words."""
    words = np.array([ref.stream_word(seed, 1, ref.P_LEAF, 0, t) for t in range(n)], dtype=np.uint64)
    counts = np.bincount((words >> np.uint64(32 - bits)).astype(np.int64), minlength=1 << bits)
    at = int(counts.argmax())
    return int(counts[at]), int(counts[:at].sum())


@pytest.mark.parametrize("seed,keys", [(1443, 8), (37699, 8), (47581, 8), (51220, 9), (56678, 9),
                                       (526884, 10)])
def test_work_group_sort(ref, seed, keys):
    """One leaf of 4095 values, 13 bits, every alignment of the output."""
    import torch
    m = dcs()
    got_keys, first = largest_bucket(ref, seed, 4095, 13)
    assert got_keys == keys
    straddles = [s for s in range(16) if (first + s) // ROW != (first + s + keys - 1) // ROW]
    assert straddles or seed == 1443 or keys > 8
    for N in (1 << 32, (1 << 32) - 5):
        want = ref.sample(4095, N, seed)
        for shift in range(16):
            announce(f"bucket of {keys}: seed={seed} N={N} shift={shift}")
            buf = torch.zeros(4095 + 16, dtype=torch.int64, device="cuda")
            m.sample(4095, N, seed, out=buf[shift:shift + 4095])
            m.synchronize()
            got = to_np_u64(buf)[shift:shift + 4095]
            assert np.array_equal(got, want), first_mismatch(got, want)


# k_leaf_small: 11 bits, a leaf of a batch over a range that is no power of two
@pytest.mark.parametrize("seed,keys", [(244610, 8), (7139840, 8), (94213, 8), (10277067, 9),
                                       (294218, 10)])
def test_one_wave_sort(ref, seed, keys):
    import torch
    m = dcs()
    N = (1 << 32) - 5  # no word of these leaves is void: the first 1024 are the leaf's
    got_keys, first = largest_bucket(ref, seed, 1024, 11)
    assert got_keys == keys
    assert keys > 8 or first // ROW != (first + keys - 1) // ROW
    want = ref.sample(1024, N, seed)
    specs = [m.InstanceSpec(n=1024, N=N, seed=seed, out_offset=1025 * i) for i in range(16)]
    out = torch.zeros(1025 * 16, dtype=torch.int64, device="cuda")
    announce(f"bucket of {keys}, one wave: seed={seed}")
    m.Batch(specs).run(out)
    m.synchronize()
    got = to_np_u64(out)
    for i in range(16):  # every alignment
        part = got[1025 * i:1025 * i + 1024]
        assert np.array_equal(part, want), (i, first_mismatch(part, want))
