"""The fp16 attention kernels keep their accumulators in accumulation registers
that inline assembly names outright; the compiler must put nothing there.  The
kernels are compiled as the library is, and every use of an accumulation
register outside the inline assembly fails."""
import os
import re
import subprocess

import pytest

from paper_2606_07878_amd import build


def _uses_outside_inline_assembly(asm: str):
    inside, kernel, found = False, "", []
    for line in asm.splitlines():
        m = re.match(r"^(_Z\w+):", line)
        if m:
            kernel = m.group(1)
        if "#ASMSTART" in line:
            inside = True
        elif "#ASMEND" in line:
            inside = False
        elif not inside and line.startswith("\t") and not line.startswith(("\t.", "\t;")):
            if re.search(r"accvgpr|\ba\[?\d", line.split(";")[0]) and "xattn_f16" in kernel:
                found.append(f"{kernel}: {line.strip()}")
    return found


def test_checker_sees_a_use():
    asm = "_Zxattn_f16_k:\n\tv_add_f32 v0, v1, v2\n\t;;#ASMSTART\n\tv_accvgpr_read_b32 v0, a[5]\n\t;;#ASMEND\n"
    assert not _uses_outside_inline_assembly(asm)
    assert _uses_outside_inline_assembly(asm + "\tv_accvgpr_write_b32 a7, v1\n")
    assert _uses_outside_inline_assembly(asm + "\tglobal_load_dwordx4 a[0:3], v[0:1], off\n")


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc")
def test_accumulation_registers_are_left_alone(tmp_path):
    out = tmp_path / "xattn.s"
    src = os.path.join(build.CSRC, "xattn.hip")
    r = subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", "-o", str(out), src],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    asm = out.read_text()
    assert asm.count("v_mfma_f32_32x32x16_f16") > 1000   # the kernels are there
    found = _uses_outside_inline_assembly(asm)
    assert not found, found[:5]
