"""Generated-code check for the kernels that stream a matrix straight to registers (deer_stream.hpp).  Their loads are asm
statements whose data arrives later, which the compiler does not know: were such a register copied, spilled or lent out
meanwhile, the copy would be of old data and the data would land in whatever the register holds then (an address: a wild
access).  So from the first of these loads to the last product, nothing but the loads and the products may name one of their
registers, and nothing may be spilled.  (A form with four row tiles and two blocks per wave, which needs more than 256 registers,
had its loads' registers copied to accumulation registers at once and used again as addresses.)"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2512_15176_amd import build

SOURCE = """
#include "deer_stream.hpp"
namespace deer {
#define MOE(M, S) template __global__ void k_gemm_moe<M, S>(const MoeArgs, int); template __global__ void k_moe_block<M, S>(const MoeArgs, int);
MOE(MOE_GATEUP, true) MOE(MOE_GATEUP, false) MOE(MOE_DOWN, true) MOE(MOE_DOWN, false)
#define LM(MT, S, WPE) template __global__ void k_lm_head<4, MT, 2, S, WPE>(const GemmArgs, int);
LM(1, true, 3) LM(1, false, 3) LM(2, true, 2) LM(2, false, 2)
}
"""


def registers(operand):
    m = re.match(r"([va])(?:\[(\d+):(\d+)\]|(\d+))$", operand)
    return {(m[1], i) for i in range(int(m[2] or m[4]), int(m[3] or m[4]) + 1)} if m else set()


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")
def test_registers_of_streamed_loads_are_left_alone(tmp_path):
    src, out = tmp_path / "stream.hip", tmp_path / "stream.s"
    src.write_text(SOURCE)
    cmd = [build.hipcc_path(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I", os.path.join(build.ROOT, "include"), "-I", os.path.join(build.PKG_DIR, "csrc"), "--cuda-device-only", "-S", "-o", str(out), str(src)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    text = out.read_text()
    api = open(build.SOURCES[0]).read()   # the forms above are those that the host launches
    assert set(re.findall(r"k_lm_head<4, (\d), 2, (\w+), (\d)>", api)) == set(re.findall(r"LM\((\d), (\w+), (\d)\)", SOURCE))
    kernels = 0
    for name, body in re.findall(r"^(_ZN4deer\w*(?:k_gemm_moe|k_moe_block|k_lm_head|k_gemm_gateup)\w*):(.*?)^\.Lfunc_end", text, re.S | re.M):
        ops, asm, inside = [], [], False   # asm: ops from asm statements
        for line in body.split("\n"):
            inside = "#ASMSTART" in line or inside and "#ASMEND" not in line
            code = line.split(";")[0].strip()
            if code and not code.startswith("."):
                if inside:
                    asm.append(len(ops))
                ops.append(re.split(r"[ ,]+", code))
        loads = [i for i in asm if ops[i][0] == "global_load_dwordx4"]
        products = [i for i, o in enumerate(ops) if o[0].startswith("v_mfma")]
        loads = [i for i in loads if "sc1" not in ops[i]]   # (partial sums: waited for where they are requested)
        held = set().union(*(registers(ops[i][1]) for i in loads))
        assert len(loads) >= 16 and len(held) >= 64, name
        for i in range(loads[0], products[-1] + 1):
            touched = set().union(*(registers(x) for x in ops[i][1:])) & held
            assert not touched or i in loads or (i in products and not registers(ops[i][1]) & held), (name, ops[i])
        assert not any(o[0].startswith(("scratch_", "v_accvgpr")) for o in ops), name
        kernels += 1
    assert kernels == 13
