"""The hand-written blocks read scalar registers that the compiler may have written with a VALU instruction right before the
block, which it does not look into: the two wait states gfx950 wants must stand inside the block."""
import os
import re
import subprocess

import pytest

from paper_2605_14292_amd import build


def _blocks(source, tmp_path):
    out = tmp_path / "out.s"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *build.FLAGS, "-S", "--cuda-device-only",
                    os.path.join(build.CSRC, source), "-o", str(out)], check=True, stderr=subprocess.DEVNULL)
    return re.findall(r"#ASMSTART\n(.*?)#ASMEND", out.read_text(), re.S)


def _states(instructions):
    """Wait states of the s_nop and of the scalar moves to m0 among them."""
    return sum(1 + int(n or 0) for _, n in re.findall(r"^\s+(s_nop|s_mov_b32)\s+(?:m0.*|(\d+))$", instructions, re.M))


@pytest.mark.parametrize("source", ["kvr_retain_dense16.hip", "kvr_select_dense_f32.hip"])
def test_the_race_waits_before_its_first_scalar_operand(source, tmp_path):
    races = lanes = 0
    for block in _blocks(source, tmp_path):
        if "v_writelane_b32" in block and "v_fma_f32" in block:
            races += 1
            before = block[: block.index("v_fma_f32")]
            assert _states(before) >= 3 and "s_nop" in before   # two, and the scalar move that stands there anyway
        elif "v_writelane_b32" in block:                        # the lists of the chain without a penalty
            lanes += 1
            assert _states(block[: block.index("v_writelane_b32")]) >= 2
    assert races > 0 and lanes > 0
