"""Registers of the built tree and segment kernels (CPU: read from the library's
own code object).  Their work is a chain of splits, hidden only by other waves,
so what they need beyond 128 vector registers, a wave per SIMD, is time: the
320,000 top paths of 300,000 segments took 556 us at three waves per SIMD and
453 at four."""
import glob
import os
import re
import shutil
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def vgprs(tmp_path_factory):
    import paper_1610_05141_amd as m
    if not os.path.exists(os.path.join(LLVM, "llvm-objdump")):
        pytest.skip("no LLVM tools")
    d = tmp_path_factory.mktemp("objects")
    shutil.copy(m.LIB_PATH, d / "libdcs.so")
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", "libdcs.so"], cwd=d,
                   check=True, capture_output=True)
    counts = {}
    for f in glob.glob(str(d / "*gfx950*")):
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", f], check=True,
                               capture_output=True, text=True).stdout
        for block in re.split(r"\n\s+- (?=\.agpr_count|\.args)", notes):
            name = re.search(r"\.name:\s+(_Z\S+)", block)
            count = re.search(r"\.vgpr_count:\s+(\d+)", block)
            if name and count:
                counts[name.group(1)] = int(count.group(1))
    return counts


@pytest.mark.parametrize("kernel", ["k_tree_top", "k_segments", "k_part_roots"])
def test_four_waves_per_simd(vgprs, kernel):
    got = [v for k, v in vgprs.items() if re.search(r"\d" + kernel + "E", k)]
    assert len(got) == 1, sorted(vgprs)
    assert got[0] <= 128
