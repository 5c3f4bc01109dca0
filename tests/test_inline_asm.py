"""The library's inline assembly, looked at in the assembler listing that the compiler writes for it.

A scalar register written by the vector unit (v_readfirstlane, v_readlane) may be read as an address by a vector memory
instruction no earlier than five wait states later.  The compiler sees to that for instructions of its own, not for those
inside an inline assembly block, whose load then takes a stale base."""
import os
import re
import subprocess

import pytest

from paper_2410_13344_amd import build

WAIT_STATES = 5
MEMORY = re.compile(r"(global|buffer|flat|scratch)_")


def scalar_registers(operand):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.fullmatch(r"s(\d+)", operand)
    return {int(m[1])} if m else set()


def instructions(listing):
    """(operation, operands, number of the inline assembly block or 0) of every instruction."""
    block, blocks = 0, 0
    for line in listing.splitlines():
        if "ASMSTART" in line:
            blocks += 1
            block = blocks
        if "ASMEND" in line:
            block = 0
        text = line.split(";")[0].strip()
        if not text or text.startswith(".") or text.endswith(":"):
            continue
        op, _, rest = text.partition(" " if " " in text else "\t")
        yield op.strip(), [o for o in re.split(r"[\s,]+", rest) if o], block


def stale_bases(listing):
    """Memory instructions that read a scalar register too soon after a vector instruction wrote it."""
    out, since = [], {}
    for op, operands, _ in instructions(listing):
        if MEMORY.match(op):
            out += [(op, operands) for o in operands for r in scalar_registers(o) if since.get(r, WAIT_STATES) < WAIT_STATES]
        states = int(operands[0], 0) + 1 if op == "s_nop" else 1
        since = {r: n + states for r, n in since.items() if n + states < WAIT_STATES}
        if operands and op.startswith(("v_", "s_")):
            for r in scalar_registers(operands[0]):
                since.pop(r, None)
                if op.startswith("v_"):
                    since[r] = 0
    return out


def unguarded_blocks(listing):
    """Inline assembly blocks that read a scalar base and do not begin with the wait."""
    blocks = {}
    for op, operands, block in instructions(listing):
        if block:
            blocks.setdefault(block, []).append((op, operands))
    bad = []
    for body in blocks.values():
        if any(MEMORY.match(op) and any(scalar_registers(o) for o in operands) for op, operands in body):
            op, operands = body[0]
            if op != "s_nop" or int(operands[0], 0) + 1 < WAIT_STATES:
                bad.append(body)
    return bad


def test_the_scan_sees_a_stale_base():
    late = "v_readfirstlane_b32 s4, v0\n;;#ASMSTART\nglobal_load_dwordx4 v[0:3], v8, s[4:5]\n;;#ASMEND\n"
    assert len(stale_bases(late)) == 1 and len(unguarded_blocks(late)) == 1
    waited = late.replace("global_load", "s_nop 4\nglobal_load")
    assert not stale_bases(waited) and not unguarded_blocks(waited)
    assert stale_bases(late.replace("global_load", "s_nop 3\nglobal_load"))
    assert not stale_bases("v_readfirstlane_b32 s4, v0\ns_add_u32 s4, s4, s8\n" + late.split("\n", 1)[1])


@pytest.mark.parametrize("source", ["gemm_team.hip", "gemm_tile_gate_up.hip", "gemm_tile_planes.hip", "attention.hip"])
def test_inline_loads_wait_for_their_scalar_base(source):
    cmd = [build.hipcc(), *build.FLAGS, "-S", "--offload-device-only", os.path.join(build.CSRC, source), "-o", "-"]
    listing = subprocess.run(cmd, capture_output=True, text=True, check=True).stdout
    assert listing.count("ASMSTART") > 0
    assert not stale_bases(listing)
    assert not unguarded_blocks(listing)
