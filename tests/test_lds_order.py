"""Order of the LDS traffic in the compiled gradient kernels, read from the gfx950 code of libhmag.so.

The fused backward-row + accumulation kernel zeroes its partner-side slices with all threads of a workgroup, and
every wave then adds into its own row tasks' slices, which other waves zeroed.  The re-layouts between the two do
not order the waves (moves inside a wave have no barrier), so the kernel needs a workgroup barrier of its own:
without it a late wave can zero what another one has added, and no run shows that reliably."""
import os
import re
import shutil
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"


def _disassemble(tmp, kernel):
    """{mangled name: [instruction, ...] in address order} of every instantiation of `kernel`."""
    import paper_2601_07824_amd as hm
    so = os.path.join(os.path.dirname(os.path.abspath(hm.__file__)), "libhmag.so")
    if not os.path.exists(so):
        import __graft_entry__
        __graft_entry__.build()
    os.symlink(so, os.path.join(tmp, "lib.so"))  # the code objects are written beside it
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", "lib.so"], cwd=tmp, check=True, capture_output=True)
    found = {}
    for obj in sorted(f for f in os.listdir(tmp) if f.endswith("gfx950")):
        with open(os.path.join(tmp, obj), "rb") as f:
            if kernel.encode() not in f.read():
                continue
        syms = subprocess.run([f"{LLVM}/llvm-readelf", "--symbols", "--wide", obj], cwd=tmp, check=True,
                              capture_output=True, text=True).stdout
        names = sorted({w for line in syms.splitlines() if " FUNC " in line for w in line.split()[-1:] if kernel in w})
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", "--no-leading-addr",
                               "--disassemble-symbols=" + ",".join(names), obj], cwd=tmp, check=True,
                              capture_output=True, text=True).stdout
        name = None
        for line in text.splitlines():
            m = re.match(r"<(\S+)>:$", line.strip()) or re.match(r"[0-9a-f]+ <(\S+)>:$", line.strip())
            if m:
                name = m.group(1)
                found.setdefault(name, [])
            elif name and line.strip():
                found[name].append(line.split()[0])
    return found


@pytest.mark.skipif(not shutil.which(f"{LLVM}/llvm-objdump"), reason="no llvm-objdump")
def test_slices_are_zeroed_before_any_wave_adds(tmp_path):
    kernels = _disassemble(str(tmp_path), "k_grad_rowback_accum")
    assert len(kernels) >= 10, sorted(kernels)
    for name, ops in kernels.items():
        reads = [i for i, op in enumerate(ops) if op.startswith("ds_read")]
        barriers = [i for i, op in enumerate(ops) if op.startswith("s_barrier")]
        assert reads and barriers, name
        # the first reads are the re-layouts' and the slices' in the shift loop, the zeroing is before them
        assert any(op.startswith("ds_write") for op in ops[:barriers[0]]), name
        assert barriers[0] < reads[0], f"{name}: no barrier between zeroing the slices and the shift loop"
