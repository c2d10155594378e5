"""Registers of the adjoint kernels in the built device code: the largest two-sided shape that the default and the even
spread of groups choose (six ring pairs per lane, one wave) keeps its slots in registers.  The counts are those the
compiler left in the kernels' metadata."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2606_06175_amd", "libakra.so")
BIN = "/opt/rocm/llvm/bin/"


def test_six_two_sided_slots(tmp_path):
    if not os.path.exists(BIN + "llvm-readelf"):
        pytest.skip("no llvm-readelf")
    assert os.path.exists(LIB), "build libakra.so first"
    shutil.copy(LIB, tmp_path / "lib.so")
    subprocess.run([BIN + "llvm-objdump", "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    spill = {}
    for f in os.listdir(tmp_path):
        if f.endswith("gfx950"):
            notes = subprocess.run([BIN + "llvm-readelf", "--notes", f], cwd=tmp_path, check=True, capture_output=True,
                                   text=True).stdout
            for m in re.finditer(r"\.name:\s+(\S*k_leg_adjI\S+)\n(?:.*\n)*?\s+\.vgpr_spill_count:\s+(\d+)", notes):
                spill[m.group(1)] = int(m.group(2))
    # k_leg_adj<S, 6, 1, 8, GCLS_BOTH>
    six = {n: v for n, v in spill.items() if re.search(r"k_leg_adjI[fd]Li6ELi1ELi8ELi0E", n)}
    assert len(six) == 2, sorted(spill)[:4]
    assert max(six.values()) <= 24, six
