"""Edge pairs written by the leaf kernels that random graphs of ordinary
densities do not reach (GPU): leaves whose values repeat (repaired, marked, in
one pass), dense leaves over ranges above 2^16, and the same as a graph's only
leaf.  Each case states the kind of leaf it is for, which the oracle's tree is
checked to hold; edges against the oracle's, bit for bit."""
import ctypes

import numpy as np
import pytest

from tests.gpu_util import announce, dcs, first_mismatch

pytestmark = pytest.mark.gpu

SMALL, MARKED = 1024, 37632  # k_leaf_small's largest leaf; the largest range with a bit per value


def kind(Nv, nv, dense_ratio):
    if dense_ratio * nv >= Nv:
        return "wide dense" if Nv > 1 << 16 else "dense"
    repeats = nv * nv >= 2 * Nv
    if nv <= SMALL:
        return "marked" if repeats and Nv <= MARKED else "small"
    return "once" if repeats else "sparse"


def leaf_kinds(ref, n, N, seed, n0, dense_ratio):
    """Leaves of more than 32 values by kind."""
    out, todo = {}, [(1, N, n)]
    while todo:
        node, Nv, nv = todo.pop()
        if nv == 0:
            continue
        if nv < n0 and Nv <= 1 << 32:
            if nv > 32:
                k = kind(Nv, nv, dense_ratio)
                out[k] = out.get(k, 0) + 1
            continue
        l = Nv // 2
        L = ref.hyp(nv, l, Nv, seed, node)
        todo += [(2 * node, l, L), (2 * node + 1, Nv - l, nv - L)]
    return out


def pairs(values):
    """(u, v), v < u, of the edge indices values - 1."""
    k = values.astype(np.int64) - 1
    u = ((1.0 + np.sqrt(8.0 * k + 1.0)) / 2).astype(np.int64)
    u -= u * (u - 1) // 2 > k
    u += u * (u + 1) // 2 <= k
    return np.stack([u, k - u * (u - 1) // 2], axis=1).astype(np.uint32)


@pytest.mark.parametrize("want,V,m,n0,dense_ratio", [
    ("once", 4000, 400_000, 4096, 16),       # density 1/20: several repeats in every leaf
    ("once", 9000, 405_000, 4096, 16),       # 1/100
    ("once", 500, 3000, 4096, 16),           # one leaf, 72 repeats: k_leaf_one_pass
    ("sparse", 3000, 2500, 4096, 16),        # one leaf, fewer than one
    ("small", 2000, 1000, 4096, 16),         # one leaf of a quarter repeat
    ("marked", 1500, 60_000, 600, 16),       # small leaves of many repeats
    ("marked", 400, 20_000, 1025, 2),
    ("small", 30_000, 400_000, 500, 16),     # small leaves repaired now and then
    ("wide dense", 4000, 230_000, 4096, 64),
    ("wide dense", 600, 3500, 4096, 64),     # one leaf
    ("dense", 350, 4000, 4096, 64),          # one leaf
])
@pytest.mark.parametrize("seed", [90, 91])
def test_edges(ref, want, V, m, n0, dense_ratio, seed):
    import torch
    mod = dcs()
    N = V * (V - 1) // 2
    kinds = leaf_kinds(ref, m, N, seed, n0, dense_ratio)
    assert kinds.get(want, 0) > 0, kinds
    announce(f"G(n,m) for {want} leaves: n={V} m={m} n0={n0} dense_ratio={dense_ratio}")
    expect = pairs(ref.sample(m, N, seed, n0=n0, dense_ratio=dense_ratio))
    out = torch.zeros((m, 2), dtype=torch.int32, device="cuda")
    for mask in (-1, 0, 7):  # by default; every kernel launched; all in the work-group kernels
        mod.debug_leaf_kernels(mask)
        try:
            out.zero_()
            rc = mod.lib().dcs_sample_edges_gnm(V, m, seed, mod._params(n0, dense_ratio),
                                                ctypes.c_void_p(out.data_ptr()), None)
            assert rc == 0
            mod.synchronize()
        finally:
            mod.debug_leaf_kernels(-1)
        got = out.cpu().numpy().view(np.uint32)
        assert np.array_equal(got, expect), (mask, first_mismatch(got.ravel(), expect.ravel()))
