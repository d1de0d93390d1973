"""The hand-written blocks read scalar registers that the compiler may have written with a VALU instruction right before the
block, which it does not look into: the two wait states gfx950 wants must stand inside the block."""
import os
import re
import subprocess

import pytest

from paper_2605_14292_amd import build


def _blocks(source, tmp_path):
    out = tmp_path / "out.s"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *build.FLAGS, "-I", build.CSRC, "-S", "--cuda-device-only",
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


def test_the_mask_blocks_wait_at_either_end(tmp_path):
    """x of masks_ge / masks_eq may come from a v_readfirstlane right before the block, a mask may go to a vector instruction
    right after it."""
    src = tmp_path / "masks.hip"
    src.write_text("""#include "kvr_dense_common.hpp"
template <int S> __global__ void masks(const uint32_t* u, const float* f, unsigned long long* out, uint32_t x, float y) {
  uint32_t v[S]; float g[S]; unsigned long long m[3][S];
  for (int k = 0; k < S; ++k) { v[k] = u[64 * k + threadIdx.x]; g[k] = f[64 * k + threadIdx.x]; }
  kvr::masks_ge<S>(v, x, m[0]); kvr::masks_ge<S>(g, y, m[1]); kvr::masks_eq<S>(g, y, m[2]);
  for (int q = 0; q < 3; ++q) for (int k = 0; k < S; ++k) out[q * S + k] = m[q][k];
}
""" + "".join("template __global__ void masks<%d>(const uint32_t*, const float*, unsigned long long*, uint32_t, float);\n" % n
              for n in (2, 3, 4, 8, 16)))
    blocks = [re.findall(r"^\s+([a-z]\S+)\s*(.*)$", b, re.M) for b in _blocks(str(src), tmp_path) if "v_cmp" in b]
    assert len(blocks) == 3 * (4 + 2)                           # sixteen slots are two blocks
    for b in blocks:
        assert b[0] == ("s_nop", "1") and b[-1] == ("s_nop", "1")
        assert all(op in ("v_cmp_le_u32", "v_cmp_le_f32", "v_cmp_eq_f32") for op, _ in b[1:-1]) and len(b) > 3
        written = [args.split(",")[0] for _, args in b[1:-1]]
        assert len(set(written)) == len(written)
