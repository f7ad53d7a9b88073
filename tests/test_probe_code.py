"""The matrix-instruction probes of the benchmark (csrc/probe.hip) measure the
instruction's rate only if their loops hold nothing else: the loop of each, as
compiled with the library's flags, has its 8 matrix instructions and no register
move.
"""
import os
import re
import subprocess

import pytest

from paper_2211_07715_amd import build as b


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    out = tmp_path_factory.mktemp("probe") / "probe.asm"
    subprocess.run([b.HIPCC, f"--offload-arch={b.ARCH}", "-std=c++17", "-O3", *b.DEVICE_FLAGS, "--cuda-device-only",
                    "-S", os.path.join(b.CSRC, "probe.hip"), "-o", str(out)],
                   check=True, stderr=subprocess.DEVNULL)
    return out.read_text()


@pytest.mark.parametrize("op,instr", [(0, "v_mfma_i32_16x16x64_i8"), (1, "v_mfma_i32_32x32x32_i8"),
                                      (2, "v_smfmac_i32_16x16x128_i8")])
def test_loop_has_only_matrix_instructions(asm, op, instr):
    body = asm[asm.index(f"_Z17probe_mfma_kernelILi{op}EEviPi:"):]
    body = body[:body.index(".Lfunc_end")]
    blocks = re.split(r"^\.LBB\w+:", body, flags=re.M)
    loops = [blk[:blk.index("s_cbranch")] for blk in blocks if instr in blk and "s_cbranch" in blk]
    loops = [blk for blk in loops if instr in blk]
    assert len(loops) == 1
    ops = re.findall(r"^\s+(v_\w+)", loops[0], flags=re.M)
    assert ops == [instr] * 8, ops
