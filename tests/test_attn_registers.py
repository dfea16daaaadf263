"""The fp16 attention kernels keep their accumulators in accumulation registers
that inline assembly names outright; the compiler must put nothing there.  The
kernels are compiled as the library is, and every use of an accumulation
register outside the inline assembly fails, as does more scratch memory than
the present kernels take."""
import os
import re
import subprocess

import pytest

from paper_2606_07878_amd import build


def test_checker_sees_a_use():
    asm = "_Zxattn_f16_k:\n\tv_add_f32 v0, v1, v2\n\t;;#ASMSTART\n\tv_accvgpr_read_b32 v0, a[5]\n\t;;#ASMEND\n"
    assert not build.accumulation_register_uses(asm)
    assert build.accumulation_register_uses(asm + "\tv_accvgpr_write_b32 a7, v1\n")
    assert build.accumulation_register_uses(asm + "\tglobal_load_dwordx4 a[0:3], v[0:1], off\n")


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc")
def test_accumulation_registers_are_left_alone(tmp_path):
    out = tmp_path / "xattn.s"
    src = os.path.join(build.CSRC, "xattn.hip")
    r = subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", "-o", str(out), src],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    asm = out.read_text()
    assert asm.count("v_mfma_f32_32x32x16_f16") > 1000   # the kernels are there
    found = build.accumulation_register_uses(asm)
    assert not found, found[:5]
    # scratch bytes per lane: <latents, value features, candidates, key tiles per wave>
    spilled = {(128, 256, 1, 4): 80, (128, 256, 0, 4): 48, (128, 512, 1, 2): 16}
    sizes = build.scratch_bytes(asm)
    assert len(sizes) == 12
    for name, size in sizes.items():
        key = tuple(map(int, re.search(r"ILi(\d+)ELi(\d+)ELb(\d)ELi(\d)E", name).groups()))
        assert size <= spilled.get(key, 0), f"{name}: {size} bytes of scratch"
