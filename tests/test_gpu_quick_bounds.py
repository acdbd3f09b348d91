"""The bounds on which the quick evaluations rest (GPU): the hardware's
single-precision logarithm over all 2^32 words and the skips read off it, the
table logarithm of the double-precision skips, and the quick reciprocal and
root of the split deviates and edges."""
import ctypes
import math
import struct

import numpy as np
import pytest

from tests.gpu_util import announce, dcs

pytestmark = pytest.mark.gpu


def tally(m, op, x, count, p0=0, p1=0):
    """(wrong skips, largest distance of the logarithms)."""
    import torch
    y = torch.zeros(2, dtype=torch.int64, device="cuda")
    rc = m.lib().dcs_debug_primitive(op, ctypes.c_void_p((y if x is None else x).data_ptr()), None,
                                     ctypes.c_void_p(y.data_ptr()), count, p0, p1, 0, 0, None)
    assert rc == 0
    torch.cuda.synchronize()
    wrong, bits = (int(v) for v in y.cpu())
    return wrong, struct.unpack("<d", struct.pack("<q", bits))[0]


# c = 1 / ln(1 - p): the ends of the single-precision range, ordinary
# densities, and p near 1, where every skip is 0 and x' near an integer
@pytest.mark.parametrize("p", [2.0**-10, 0.01, 0.0625, 0.5, 0.999, 1.0 - 2.0**-20])
def test_every_word_gives_the_defined_skip(p):
    m = dcs()
    c = struct.unpack("<I", struct.pack("<f", 1.0 / math.log1p(-p)))[0]
    most = 0.0
    for part in range(8):  # 2^29 words a launch
        announce(f"skips of words {part} 2^29 .. at p={p}")
        wrong, far = tally(m, 10, None, 1 << 27, part << 29, c)
        assert wrong == 0
        most = max(most, far)
    print(f"p={p}: logarithms within {most:.4e} of each other, relative")
    # with c ln 2's, x's and x''s roundings the skips' argument has 4.0e-7 x
    assert most + 3 * 2.0**-24 <= 4.0e-7


def edge_draws():
    """Draws with U at and next to every table interval's ends, for exponents
    over the whole range, next to 1, and the smallest ones."""
    ks = []  # U = (k + 1) 2^-53
    for e in (53, 52, 51, 40, 24, 12, 8):
        for i in range(128):
            at = ((128 + i) << e) >> 7  # m = 1 + i / 128
            ks += [at + d for d in range(-4, 4)]
    ks += list(range(0, 4096)) + [(1 << 53) - 1 - d for d in range(4096)]
    k = np.array([min(max(v, 0), (1 << 53) - 1) for v in ks], dtype=np.uint64)
    k = np.concatenate([k, np.arange(-len(k) % 2, dtype=np.uint64)])
    return k << np.uint64(11)


@pytest.mark.parametrize("log2_p", [-10.5, -16, -24, -31, -41, -60])
def test_double_precision_skips(log2_p):
    import torch
    m = dcs()
    c = struct.unpack("<q", struct.pack("<d", 1.0 / math.log1p(-(2.0**log2_p))))[0] % (1 << 64)
    rng = np.random.default_rng(int(-log2_p * 10))
    for d in (edge_draws(), rng.integers(0, 1 << 64, 1 << 23, dtype=np.uint64),
              rng.integers(0, 1 << 64, 1 << 20, dtype=np.uint64) >> rng.integers(
                  0, 53, 1 << 20, dtype=np.uint64)):
        announce(f"double-precision skips of {d.size} draws at p=2^{log2_p}")
        x = torch.from_numpy(d.view(np.int64)).cuda()
        wrong, far = tally(m, 11, x, d.size // 2, c)
        print(f"p=2^{log2_p}: {d.size} draws, logarithms within 2^{math.log2(far):.2f}")
        assert wrong == 0
        assert far <= 2.0**-45  # each within 2^-46 of ln U


@pytest.mark.parametrize("op,bound", [(12, 2.0**-45), (13, 2.0**-47)])
def test_quick_reciprocal_and_root(op, bound):
    import torch
    m = dcs()
    rng = np.random.default_rng(op)
    x = np.concatenate([
        np.ldexp(1.0 + rng.random(1 << 22), rng.integers(0, 66, 1 << 22).astype(np.int32)),
        np.ldexp(1.0 + np.arange(1 << 16) * 2.0**-52, 4), np.ldexp(2.0 - np.arange(1, 1 << 16) * 2.0**-52, 7),
        np.arange(1, 1 << 20, dtype=np.float64), 8.0 * np.arange(0, 1 << 20, dtype=np.float64) + 1.0])
    y = torch.empty(x.size, dtype=torch.float64, device="cuda")
    announce(f"quick {'1/x' if op == 12 else 'sqrt(x)'} of {x.size} values")
    m.debug_primitive(op, torch.from_numpy(x).cuda(), None, y)
    torch.cuda.synchronize()
    wide = x.astype(np.longdouble)
    want = 1 / wide if op == 12 else np.sqrt(wide)
    far = float(np.max(np.abs((y.cpu().numpy().astype(np.longdouble) - want) / want)))
    print(f"op {op}: within 2^{math.log2(far):.2f}")
    assert far <= bound
