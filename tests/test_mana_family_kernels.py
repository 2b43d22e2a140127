"""The family kernels of two-pass mana are built for the rows that a plan can take by families, and for no others:
complex64 n = 9 .. 13 (rows of 3^5 .. 3^7), complex128 n = 8 .. 12 (rows of 3^4 .. 3^6)."""
import os
import re
import shutil
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"


@pytest.mark.skipif(not shutil.which(f"{LLVM}/llvm-objdump"), reason="no llvm-objdump")
def test_built_rows(tmp_path):
    import paper_2601_07824_amd as hm
    so = os.path.join(os.path.dirname(os.path.abspath(hm.__file__)), "libhmag.so")
    os.symlink(so, tmp_path / "lib.so")  # the code objects are written beside it
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    built = set()
    for obj in (f for f in os.listdir(tmp_path) if f.endswith("gfx950")):
        syms = subprocess.run([f"{LLVM}/llvm-readelf", "--symbols", "--wide", obj], cwd=tmp_path, check=True,
                              capture_output=True, text=True).stdout
        built |= set(re.findall(r"k_mana_rowfamiliesI([fd])Li\d+ELi\d+ELi(\d+)EE", syms))
    assert built == {("f", "5"), ("f", "6"), ("f", "7"), ("d", "4"), ("d", "5"), ("d", "6")}
