"""Samples of a single leaf, which one kernel takes without a tree: every kind,
the sizes at the rule's edges, against the oracle and, through the library's
hook that keeps the general launches, against those; and replays of a captured
call."""
import numpy as np
import pytest

from tests.gpu_util import announce, dcs, first_mismatch, to_np_u64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant,n,N,n0", [
    (0, 1, 1, 4096), (0, 1, 1 << 32, 4096), (0, 7, (1 << 32) - 1, 4096), (0, 32, 1000, 4096),
    (0, 33, 1 << 20, 4096), (0, 4095, 1 << 32, 4096), (0, 4095, (1 << 32) + 1, 4096),
    (0, 4096, 1 << 32, 4096), (0, 1023, 1 << 31, 1024), (0, 500, 500, 4096), (0, 4000, 8000, 4096),
    (0, 4095, 65_520, 4096), (0, 4000, 65_536, 4096), (0, 4000, 399_999, 4096),
    (0, 4000, 400_001, 4096), (0, 1, 2, 2), (0, 4095, 65_521, 4096), (0, 1794, 60_720, 4096),
    (0, 1000, 16_001, 4096), (0, 700, 11_201, 4096), (0, 1200, 1 << 15, 4096),
    (1, 1, 1, 4096), (1, 4095, 1, 4096), (1, 4096, 1, 4096), (1, 4095, 2, 4096),
    (1, 3000, 1 << 32, 4096), (1, 100, 3_000_000_019, 4096)])
def test_one_leaf(ref, variant, n, N, n0):
    m = dcs()
    f, g = (m.sample_replacement, ref.replacement) if variant else (m.sample, ref.sample)
    want = g(n, N, 21, n0=n0)
    try:
        for mask in (-1, 0, 7):
            m.debug_leaf_kernels(mask)
            announce(f"one leaf: variant={variant} n={n} N={N} n0={n0} mask={mask}")
            got = to_np_u64(f(n, N, 21, n0=n0))
            m.synchronize()
            assert np.array_equal(got, want), first_mismatch(got, want)
    finally:
        m.debug_leaf_kernels(-1)


@pytest.mark.parametrize("n,N", [(100, 230), (90, 201), (1500, 3100), (2000, 90_000)])
def test_one_leaf_of_many_repeats(ref, n, N):
    m = dcs()
    announce(f"one leaf: n={n} N={N} dense_ratio=2")
    got = to_np_u64(m.sample(n, N, 22, dense_ratio=2))
    m.synchronize()
    want = ref.sample(n, N, 22, dense_ratio=2)
    assert np.array_equal(got, want), first_mismatch(got, want)


def test_captured_one_leaf(ref):
    import torch
    m = dcs()
    announce("one leaf: captured and replayed")
    out = torch.zeros(1000, dtype=torch.int64, device="cuda")
    m.sample(1000, 10**9, 5, out=out)  # the call's workspace, outside the capture
    torch.cuda.synchronize()
    want = ref.sample(1000, 10**9, 5)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        m.sample(1000, 10**9, 5, out=out)
    for _ in range(3):
        out.fill_(7)
        graph.replay()
        torch.cuda.synchronize()
        got = to_np_u64(out)
        assert np.array_equal(got, want), first_mismatch(got, want)
