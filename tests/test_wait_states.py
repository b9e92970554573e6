"""Wait states around the lane permutations of the Hadamard kernels, read from the assembly that the library's own sources
compile to (no GPU).  gfx950 needs two between a vector write of a register and a permuted (DPP) read or a lane-register swap
of it; the compiler inserts them for its own instructions, but it does not see writes made inside inline assembly."""
import os
import re
import subprocess

import pytest

from paper_2512_23367_amd import build

NEEDED = 2


def _registers(operand):
    m = re.fullmatch(r"v\[(\d+):(\d+)\]", operand)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.fullmatch(r"[-|]*v(\d+)\|?", operand)
    return {int(m[1])} if m else set()


def violations(assembly):
    """(kernel, instruction, operand registers, wait states found) of every hazard in a listing, and how many instructions
    were looked at.  Along the listing, labels ignored: a write that falls through into the next block counts."""
    found, looked_at, kernel = [], 0, ""
    states = []                                        # registers written in each of the last wait states, newest last
    for line in assembly.splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            kernel, states = m[1], []
        text = line.split(";")[0].strip()
        if not re.match(r"[a-z]+_\w+", text):
            continue
        op, _, rest = text.partition(" ")
        operands = [o.split()[0] for o in rest.split(",") if o.strip()]
        reads = set()
        if "permlane" in op and "swap" in op:
            reads = _registers(operands[0]) | _registers(operands[1])
        elif op.endswith("_dpp"):
            reads = _registers(operands[1])            # the permuted operand
        if reads:
            looked_at += 1
            for distance, written in enumerate(reversed(states)):
                if written & reads:
                    found.append((kernel, text, written & reads, distance))
                    break
        if op == "s_nop":
            states += [set()] * (int(rest, 0) + 1)
        else:
            w = set()
            if op.startswith("v_") and not op.startswith("v_cmp") and operands:
                w = _registers(operands[0])
                if "swap" in op:
                    w |= _registers(operands[1])
            states.append(w)
        states = states[-NEEDED:]
    return found, looked_at


def test_the_reader_sees_a_missing_wait():
    short = "_Zk:\n\tv_fmac_f32_dpp v2, v2, v9 row_ror:8\n\ts_nop 0\n\tv_permlane16_swap_b32_e32 v7, v2\n"
    assert [v[3] for v in violations(short)[0]] == [1]
    assert violations(short.replace("s_nop 0", "s_nop 1"))[0] == []
    assert violations("_Zk:\n\tv_add_f32_e32 v2, v3, v4\n\tv_mov_b32_dpp v5, v2 row_half_mirror\n")[0][0][3] == 0


def test_lane_permutations_have_their_wait_states(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no compiler here")
    out = tmp_path / "transform.s"
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "transform.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    found, looked_at = violations(out.read_text())
    assert looked_at > 1000                            # the lane stages and swaps of every block size
    assert not found, "\n".join(map(str, found[:20]))
