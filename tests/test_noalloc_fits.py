"""Workspaces of calls that have to fit the allocation-free entry point's static
scratch under the committed tuning table (CPU): a deeper cut means more stacks,
which a tuned geometry must not let outgrow it; and the tuner's rule for that."""
import os

import pytest

import paper_1610_05141_amd as dcs
from paper_1610_05141_amd import autotune


@pytest.fixture
def committed():
    if not os.path.exists(dcs.LIB_PATH):
        pytest.skip("library not built")
    dcs.lib()
    saved = [(v, c, *dcs.tune_get(v, c)) for v in (0, 1) for c in range(autotune.N_CLASSES)]
    autotune.apply_table()
    yield
    for row in saved:
        dcs.tune_set(*row)


@pytest.mark.parametrize("variant,n,N,n0", [
    (0, 4095, 1 << 62, 4096), (0, 8192, 1 << 46, 8), (0, 8192, 1 << 62, 4096),
    (0, 16384, 1 << 62, 4096), (0, 24576, 1 << 62, 256), (0, 32767, 1 << 56, 1024),
    (0, 1 << 21, 1 << 46, 64), (0, 1 << 22, 1 << 47, 4096), (0, 12582912, 1 << 36, 100),
    (0, 12582912, 1 << 47, 4096), (0, 16777215, 1 << 47, 4096), (1, 4096, 1 << 62, 4096),
    (1, 30000, 1 << 60, 4096),
])
def test_fits_the_scratch(committed, variant, n, N, n0):
    assert dcs.workspace_size(variant, n, N, n0=n0) <= dcs.NOALLOC_SCRATCH_BYTES


def test_tuner_leaves_out_biases_that_outgrow_it(committed):
    table = autotune.load_table()
    allowed = autotune.allowed_biases(autotune.GEOMETRY_CLASSES, table)
    assert 2 not in allowed[0, 13] and 2 not in allowed[0, 22]
    assert allowed[0, 19] == list(autotune.CUT_BIASES)  # its calls outgrow it anyway
    for e in table["geometry"]:
        assert e["cut_bias"] in allowed[e["variant"], e["log2_n"]]
