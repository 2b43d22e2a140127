"""The backward-row kernels of the gradient loop over tiles (shifts) with no barrier between the iterations, which
is sound only while every re-layout stays inside a wave (rows of at most 2^(6 + RB) values).  Longer rows have to be
refused by the compiler: with S0 > 6 a wave would write into the LDS that another one still reads."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_07824_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
@pytest.mark.parametrize("kernel,args,nl_ok,nl_bad", [
    ("k_sre_rowback", "RowPassArgs A", 10, 11), ("k_grad_rowback_accum", "FusedArgs A", 10, 11)])
def test_rows_beyond_a_wave_do_not_compile(tmp_path, kernel, args, nl_ok, nl_bad):
    def compiles(nl):
        shape = f"float, 256, 4, {nl}, true" if kernel == "k_sre_rowback" else f"float, 256, 4, 4, {nl}, true"
        src = tmp_path / f"{kernel}{nl}.hip"
        src.write_text(f'#include "hm_grad2_kern.h"\nnamespace hm {{\nnamespace {{\ntemplate __global__ void {kernel}<{shape}>({args});\n}}\n}}\n')
        p = subprocess.run([HIPCC, "-std=c++17", "--offload-arch=gfx950", "--cuda-device-only", "-fsyntax-only", "-I", CSRC,
                            str(src)], capture_output=True, text=True)
        return p.returncode == 0, p.stderr
    ok, err = compiles(nl_ok)
    assert ok, err
    ok, err = compiles(nl_bad)
    assert not ok and "inside a wave" in err, err
