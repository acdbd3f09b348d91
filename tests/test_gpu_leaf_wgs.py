"""leaf_wgs_per_cu of the tuning table reaches the leaf kernels (GPU): a large
sample takes longer with one leaf work-group per compute unit than with as many
as fit, and is the same sample; so does a sample whose leaves are the one-pass
kernel's."""
import pytest

from tests.gpu_util import announce, dcs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,N", [
    (1 << 26, 1 << 44),        # k_leaf_sort
    (1 << 24, (1 << 24) * 50),  # k_leaf_once
])
def test_fewer_work_groups_take_longer(n, N):
    import torch
    m = dcs()
    k = n.bit_length() - 1
    saved = m.tune_get(0, k)
    outs, us = {}, {}
    try:
        for w in (1, 0):
            m.tune_set(0, k, saved[0], w)
            announce(f"leaf work-groups per compute unit {w}: n={n} N={N}")
            outs[w] = torch.empty(n, dtype=torch.int64, device="cuda")
            times = []
            for _ in range(6):
                a, b = torch.cuda.Event(True), torch.cuda.Event(True)
                a.record()
                m.sample(n, N, 11, out=outs[w])
                b.record()
                torch.cuda.synchronize()
                times.append(a.elapsed_time(b) * 1e3)
            us[w] = min(times)
    finally:
        m.tune_set(0, k, *saved)
    print(f"n={n} N={N}: {us}")
    assert torch.equal(outs[0], outs[1])
    assert us[1] >= 1.25 * us[0], us
