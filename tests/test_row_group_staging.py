"""HM_OPT_LDS_SPLIT = 1 (whole complex values through LDS) holds for the row pass by groups of shifts too: every group
kernel is built with both stagings."""
import os
import re
import shutil
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"


@pytest.mark.skipif(not shutil.which(f"{LLVM}/llvm-objdump"), reason="no llvm-objdump")
def test_groups_are_built_with_both_stagings(tmp_path):
    import paper_2601_07824_amd as hm
    so = os.path.join(os.path.dirname(os.path.abspath(hm.__file__)), "libhmag.so")
    os.symlink(so, tmp_path / "lib.so")  # the code objects are written beside it
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    built = {"0": set(), "1": set()}
    for obj in (f for f in os.listdir(tmp_path) if f.endswith("gfx950")):
        syms = subprocess.run([f"{LLVM}/llvm-readelf", "--symbols", "--wide", obj], cwd=tmp_path, check=True,
                              capture_output=True, text=True).stdout
        for t, nt, rb, nl, split in re.findall(r"k_sre_rowgroupI([fd])Li(\d+)ELi(\d+)ELi(\d+)ELb([01])E", syms):
            built[split].add((t, nt, rb, nl))
    assert len(built["1"]) >= 17 and built["0"] == built["1"], built
