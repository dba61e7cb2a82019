"""Generated-code check for the kernels that stream a matrix straight to registers (deer_stream.hpp), on the assembly of the library
itself.  Their loads are asm statements whose data arrives later, which the compiler does not know: were such a register copied,
spilled or lent out meanwhile, the copy would be of old data and the data would land in whatever the register holds then (an
address: a wild access).  So from the first of these loads to the last product, nothing but the loads and the products may name one
of their registers; the same holds for the row index that k_gemm_moe requests, up to the wait for it; and no vector register may
be spilled.  (A form with four row tiles and two blocks per wave, which needs more than 256 registers, had its loads' registers copied
to accumulation registers at once and used again as addresses.)

Scalar registers may be kept in the lanes of a vector register.  But a vector instruction that writes a scalar register
(v_readlane_b32 brings one back) must stand five wait states before a load that takes it as its base; the compiler sees to
that for its own loads, not for those inside an asm statement."""
import os
import re
import shutil

import pytest

from paper_2512_15176_amd import build

WAIT_STATES = 5


def registers(operand):
    m = re.match(r"([vas])(?:\[(\d+):(\d+)\]|(\d+))$", operand)
    return {(m[1], i) for i in range(int(m[2] or m[4]), int(m[3] or m[4]) + 1)} if m else set()


def scalars(operand):
    return {r for r in registers(operand) if r[0] == "s"}


def parse(body):
    """Instructions as lists of mnemonic and operands, the indices of those from asm statements, labels -> index."""
    ops, asm, labels, inside = [], set(), {}, False
    for line in body.split("\n"):
        inside = "#ASMSTART" in line or inside and "#ASMEND" not in line
        code = line.split(";")[0].strip()
        if m := re.match(r"(\.LBB\w+):", code):
            labels[m[1]] = len(ops)
        elif code and not code.startswith("."):
            if inside:
                asm.add(len(ops))
            ops.append(re.split(r"[ ,]+", code))
    return ops, asm, labels


def scalar_written_just_before(ops, labels, at, base):
    """An instruction within WAIT_STATES before ops[at], on any path, that is a vector instruction and writes a register of base."""
    sources = {}
    for i, o in enumerate(ops):
        if o[0].startswith(("s_branch", "s_cbranch")):
            sources.setdefault(labels[o[1]], []).append(i)
    todo, seen = [(at, 0)], set()
    while todo:
        i, waited = todo.pop()   # what can stand before instruction i, `waited` wait states before the load
        if waited >= WAIT_STATES or (i, waited) in seen:
            continue
        seen.add((i, waited))
        for j in ([i - 1] if i and not ops[i - 1][0].startswith(("s_branch", "s_endpgm")) else []) + sources.get(i, []):
            o = ops[j]
            if o[0].startswith("v_") and any(scalars(x) & base for x in o[1:3 if "_co_" in o[0] or "div_scale" in o[0] else 2]):
                return o
            todo.append((j, waited + (int(o[1]) + 1 if o[0] == "s_nop" else 1)))
    return None


def test_the_search_for_scalar_writes():
    near, far = "v_readlane_b32 s4, v1, 0\n s_nop 3\n", "v_readlane_b32 s4, v1, 0\n s_nop 4\n"
    load = "global_load_dwordx4 v[0:3], v9, s[4:5]"
    for body, found in ((near + load, True), (far + load, False), ("v_readlane_b32 s6, v1, 0\n" + load, False), ("v_cmp_lt_i32_e64 s[4:5], v1, v2\n" + load, True),
                        ("v_add_co_u32 v2, s[4:5], v1, v2\n" + load, True), ("v_readfirstlane_b32 s5, v1\n s_cbranch_scc0 .LBB0_1\n s_nop 7\n.LBB0_1:\n" + load, True),
                        ("v_readlane_b32 s4, v1, 0\n s_branch .LBB0_2\n.LBB0_1:\n" + load + "\n.LBB0_2:\n s_nop 4\n s_branch .LBB0_1", False)):
        ops, _, labels = parse(body)
        at = next(i for i, o in enumerate(ops) if o[0].startswith("global"))
        assert (scalar_written_just_before(ops, labels, at, scalars(ops[at][3])) is not None) == found, body


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")
def test_registers_of_streamed_loads_are_left_alone(tmp_path):
    text = open(build.device_assembly(str(tmp_path / "deer_device.s"))).read()
    kernels, row_indices, partials = 0, 0, 0
    for name, body in re.findall(r"^(_ZN4deer\w*(?:k_gemm_moe|k_moe_block|k_lm_head|k_gemm_gateup)\w*):(.*?)^\.Lfunc_end", text, re.S | re.M):
        ops, asm, labels = parse(body)
        products = [i for i, o in enumerate(ops) if o[0].startswith("v_mfma")]
        loads = [i for i in sorted(asm) if ops[i][0] == "global_load_dwordx4" and "sc1" not in ops[i]]   # (sc1: partial sums, behind the products)
        held = set().union(*(registers(ops[i][1]) for i in loads))
        assert len(loads) >= 16 and len(held) >= 64, name
        for i in range(loads[0], products[-1] + 1):
            touched = set().union(*(registers(x) for x in ops[i][1:])) & held
            assert not touched or i in loads or (i in products and not registers(ops[i][1]) & held), (name, ops[i])
        for i in loads:
            assert scalars(ops[i][3]), (name, ops[i])
            assert scalar_written_just_before(ops, labels, i, scalars(ops[i][3])) is None, (name, i, ops[i])
        for i in (i for i in asm if ops[i][0] == "global_load_dword" or "sc1" in ops[i] and ops[i][0] == "global_load_dwordx4"):
            wait = next(j for j in range(i, len(ops)) if j in asm and ops[j][0] == "s_waitcnt" and "vmcnt" in ops[j][1])
            assert not any(o[0].startswith(("s_branch", "s_cbranch")) for o in ops[i:wait]), (name, ops[i], "the wait for it")
            assert not any(registers(x) & registers(ops[i][1]) for o in ops[i + 1 : wait] for x in o[1:]), (name, ops[i])
            if ops[i][0] == "global_load_dword":
                assert i < loads[0] < wait, name
                row_indices += 1
            else:
                assert "vmcnt(0)" in ops[wait][1], (name, ops[wait])
                partials += 1
        assert not any(o[0].startswith(("scratch_", "v_accvgpr")) for o in ops), name
        kernels += 1
    # two projections in two ways to fold, for few and for many rows; LM heads of one and two row tiles in two ways to fold; gate/up of two row tiles
    assert kernels == 4 + 4 + 4 + 1 and row_indices == 2 and partials >= 16
