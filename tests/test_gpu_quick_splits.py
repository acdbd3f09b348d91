"""Split deviates whose rejection test is decided by the quick evaluation and
those it leaves to the defined steps, against the oracle bit for bit: means
from just above the inversion's limit (runs of a few terms, far tails) to
2^41 and beyond (where the quick evaluation is off), skewed and even splits,
universes up to 2^62."""
import numpy as np
import pytest

from tests.gpu_util import announce, dcs

pytestmark = pytest.mark.gpu

COUNT = 1 << 17


def device(m, op, p0, p1, p2, seed):
    import torch
    ids = torch.arange(1, COUNT + 1, dtype=torch.int64, device="cuda")
    y = torch.empty_like(ids)
    m.debug_primitive(op, ids, None, y, p0, p1, p2, seed)
    torch.cuda.synchronize()
    return y.cpu().numpy().view(np.uint64)


@pytest.mark.parametrize("n,M,N", [
    (17, 17, 34), (17, 1000, 10**6), (20, 25, 50), (33, 1 << 20, 1 << 21), (64, 64, 10**9),
    (100, 5000, 10**4), (128, 1 << 31, 1 << 32), (500, 1 << 50, (1 << 51) - 3),
    (2000, 3000, 10**5), (4095, 1 << 31, 1 << 32), (4096, 4096, 8192), (5000, 4999, 10001),
    (10**5, 200, 10**7), (10**6, 10**3, 10**8), (1 << 20, 1 << 29, 1 << 30),
    (1 << 30, 1 << 47, 1 << 48), ((1 << 30) + 7, 12345678901, (1 << 40) + 1),
    (1 << 40, 1 << 58, (1 << 59) + 11), (1 << 42, 1 << 57, 1 << 58), (10**6, 1 << 61, 1 << 62),
])
def test_hypergeometric(ref, n, M, N):
    m = dcs()
    announce(f"hypergeometric n={n} M={M} N={N}")
    got = device(m, 6, n, M, N, 77)
    assert np.array_equal(got, ref.hyp_batch(n, M, N, 77, 1, COUNT))


@pytest.mark.parametrize("n,l,Nv", [
    (17, 1, 2), (17, 1, 100), (30, 10, 21), (100, 3, 10**6), (400, 1 << 31, 1 << 32),
    (1000, 499, 1000), (4095, 1 << 20, (1 << 21) + 1), (10**5, 7, 10**6), (1 << 20, 3, 7),
    (1 << 28, 1 << 39, 1 << 40), ((1 << 40) + 3, 1 << 50, (1 << 51) + 1),
    (1 << 43, 1 << 10, 1 << 11), (10**7, 1 << 61, 1 << 62),
])
def test_binomial(ref, n, l, Nv):
    m = dcs()
    announce(f"binomial n={n} l={l} Nv={Nv}")
    got = device(m, 7, n, l, Nv, 78)
    assert np.array_equal(got, ref.binom_batch(n, l, Nv, 78, 1, COUNT))
