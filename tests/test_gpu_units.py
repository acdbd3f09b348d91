"""Bernoulli chunks handed out in units of consecutive chunks (four in single,
eight in double precision): chunk counts at and around the edges of a unit and
of a work-group's first units, skips so long that a round's sum passes 2^32,
and edge pairs written by every kernel kind.  Against the oracle bit for bit."""
import numpy as np
import pytest

from tests.gpu_util import announce, dcs, first_mismatch, to_np_u64

pytestmark = pytest.mark.gpu


def check(ref, p, N, seed, n0=None):
    m = dcs()
    kw = {} if n0 is None else {"n0": n0}
    announce(f"Bernoulli p={p!r} N={N} seed={seed} n0={n0}")
    out, cnt = m.sample_bernoulli(p, N, seed, **kw)
    m.synchronize()
    want = ref.bernoulli(p, N, seed, **kw)
    assert int(cnt.item()) == want.size
    got = to_np_u64(out)[:want.size]
    assert np.array_equal(got, want), first_mismatch(got, want)


@pytest.mark.parametrize("chunks", [1, 2, 3, 4, 5, 8, 31, 33, 4100])
@pytest.mark.parametrize("ragged", [0, 77])
def test_single_precision_units(ref, chunks, ragged):
    check(ref, 0.25, chunks * 4096 - ragged, 60 + chunks, n0=64)


@pytest.mark.parametrize("chunks", [1, 2, 7, 8, 9, 16, 65, 2500])
@pytest.mark.parametrize("ragged", [0, 12345])
def test_double_precision_units(ref, chunks, ragged):
    check(ref, 2.0**-24, chunks * 2**32 - ragged, 70 + chunks)


@pytest.mark.parametrize("log2_p,log2_n", [(-27, 44), (-31, 44), (-33, 45), (-41, 52), (-60, 52)])
def test_long_skips(ref, log2_p, log2_n):
    check(ref, 2.0**log2_p, (1 << log2_n) - 99, 80)


@pytest.mark.parametrize("kind", ["sparse", "odd", "dense", "small", "inline", "wide_dense"])
def test_gnm_edges_of_every_leaf_kind(ref, kind):
    nv, m, n0 = {"sparse": (1 << 20, 200_000, None), "odd": (3_001_003, 150_001, 2000),
                 "dense": (1000, 300_000, None), "small": (1 << 18, 30_000, 200),
                 "inline": (1 << 18, 20_000, 24), "wide_dense": (4000, 500_000, 4096)}[kind]
    mod = dcs()
    kw = {} if n0 is None else {"n0": n0}
    announce(f"G(n,m) {kind}: n={nv} m={m} n0={n0}")
    e = mod.sample_edges_gnm(nv, m, 90, **kw)
    mod.synchronize()
    got = e.cpu().numpy().view(np.uint32)[:m]
    want = ref.edges_gnm(nv, m, 90, **kw)
    assert np.array_equal(got, want), first_mismatch(got.ravel(), want.ravel())


@pytest.mark.parametrize("nv,log2_p,words", [(1 << 22, -24, 0), (1 << 16, -12, 0), (1 << 16, -12, 16),
                                             (3000, -3, 0), (700, 0, 0)])
def test_gnp_edges_of_every_chunk_kind(ref, nv, log2_p, words):
    mod = dcs()
    mod.debug_bernoulli_list(words)
    try:
        announce(f"G(n,p) n={nv} p=2^{log2_p} list={words}")
        e, cnt = mod.sample_edges_gnp(nv, 2.0**log2_p, 91)
        mod.synchronize()
    finally:
        mod.debug_bernoulli_list(0)
    want = ref.edges_gnp(nv, 2.0**log2_p, 91)
    assert int(cnt.item()) == len(want)
    got = e.cpu().numpy().view(np.uint32)[:len(want)]
    assert np.array_equal(got, want), first_mismatch(got.ravel(), want.ravel())
