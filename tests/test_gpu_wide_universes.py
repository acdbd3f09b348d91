"""Splits of universes from 2^60 to 2^62 (GPU): their deviates are decided by
the quick evaluation like those of narrower ones, at the same cost, and are the
oracle's bit for bit."""
import time

import numpy as np
import pytest

from tests.gpu_util import announce, dcs

pytestmark = pytest.mark.gpu

COUNT = 1 << 17


def deviates(m, op, p0, p1, p2, reps=1):
    """The deviates of nodes 1 .. COUNT and the least time of a launch."""
    import torch
    ids = torch.arange(1, COUNT + 1, dtype=torch.int64, device="cuda")
    y = torch.empty_like(ids)
    best = float("inf")
    for _ in range(reps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        m.debug_primitive(op, ids, None, y, p0, p1, p2, 79)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t0)
    return y.cpu().numpy().view(np.uint64), best


@pytest.mark.parametrize("n,M,N", [
    (40, 1 << 61, 1 << 62), (10**6, 1 << 61, 1 << 62), (5000, (1 << 61) - 7, (1 << 62) - 11),
    (10**9, 1 << 55, 1 << 62), (1 << 40, 1 << 61, 1 << 62), ((1 << 41) - 5, 1 << 61, 1 << 62),
    (10**5, 1 << 59, 1 << 60), (10**5, (1 << 59) - 1, (1 << 60) - 1), (300, 1 << 60, (1 << 62) - 1),
])
def test_hypergeometric(ref, n, M, N):
    announce(f"hypergeometric n={n} M={M} N={N}")
    got, _ = deviates(dcs(), 6, n, M, N)
    assert np.array_equal(got, ref.hyp_batch(n, M, N, 79, 1, COUNT))


@pytest.mark.parametrize("n,l,Nv", [
    (40, 1 << 61, 1 << 62), (10**7, (1 << 61) - 3, (1 << 62) - 5), (1 << 41, 1 << 60, 1 << 62),
    (10**5, 1 << 59, 1 << 60),
])
def test_binomial(ref, n, l, Nv):
    announce(f"binomial n={n} l={l} Nv={Nv}")
    got, _ = deviates(dcs(), 7, n, l, Nv)
    assert np.array_equal(got, ref.binom_batch(n, l, Nv, 79, 1, COUNT))


@pytest.mark.parametrize("op", [6, 7])
def test_cost_does_not_depend_on_the_universe(op):
    m = dcs()
    announce(f"times of splits of 2^58 and 2^62, op {op}")
    us = [deviates(m, op, 10**6, 1 << (b - 1), 1 << b, reps=20)[1] * 1e6 for b in (58, 62)]
    print(f"op {op}: {us[0]:.1f} us at 2^58, {us[1]:.1f} us at 2^62")
    assert us[1] <= 1.25 * us[0], us
