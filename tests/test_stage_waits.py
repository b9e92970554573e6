"""Counted waits of the prefill kernels of four-wavefront workgroups, read from the assembly that the library's own sources compile to
(no GPU).  Their stages of tokens are loaded into LDS three ahead, each wavefront a share, and a wavefront's own waits in front of a
barrier are all that says its share of the next stage is there.  The waits count loads, so they hold only for the loads, and the
order of them, that the compiler leaves in a kernel."""
import os
import re
import subprocess

import pytest

from paper_2512_23367_amd import build

STAGES = 3


def walk(lines, passes=3, second_tile=False):
    """The instructions of one kernel in the order a wavefront meets them: forward conditional branches not taken (partial work, absent
    parts), a backward one taken `passes` times (the stage loop).  second_tile: the first one is taken (a kernel of two tile forms)."""
    labels = {m[1]: i for i, l in enumerate(lines) if (m := re.match(r"(\.LBB\w+):", l))}
    taken, i = {}, 0
    while i < len(lines):
        text = lines[i].split(";")[0].strip()
        m = re.match(r"s_(c?)branch\w*\s+(\.LBB\w+)", text)
        if m and (labels[m[2]] <= i or not m[1] or second_tile):
            second_tile = False
            taken[i] = taken.get(i, 0) + 1
            if taken[i] <= passes:
                i = labels[m[2]]
                continue
        yield text
        if text.startswith("s_endpgm"):
            return
        i += 1


def late_stages(lines, second_tile=False):
    """(barrier, loads into LDS in flight there, how many may be) of every barrier of the stage loop where a share of the next stage may
    still be on its way, and the number of barriers looked at."""
    flying, issued, barriers, share, found = [], 0, 0, 0, []
    for text in walk(lines, second_tile=second_tile):
        if re.match(r"(buffer|global)_load", text):
            flying.append(text.endswith("lds"))
            issued += flying[-1]
        elif m := re.search(r"vmcnt\((\d+)\)", text):
            flying = flying[len(flying) - int(m[1]):] if len(flying) > int(m[1]) else flying
        elif text.startswith("s_barrier"):
            if not share:
                share = issued // STAGES                    # of one stage; the loop's start has asked for all three
                assert share and issued == share * STAGES
            if barriers and not flying:                     # behind the loop: all is drained
                break
            allowed = share * (STAGES - 1 if barriers == 0 else STAGES - 2)
            if sum(flying) > allowed:
                found.append((barriers, sum(flying), allowed))
            barriers += 1
    return found, barriers


def kernels(assembly):
    for m in re.finditer(r"^(_Z\w+):\s.*?^\.Lfunc_end", assembly, re.S | re.M):
        if " lds" in m[0]:
            yield m[1], m[0].splitlines()[1:]


def test_the_reader_sees_a_missing_wait():
    load, token = "buffer_load_dwordx4 v[0:3], v4, s[0:3], 0 offen", "buffer_load_dwordx4 v9, s[0:3], 0 offen lds"
    loop = [".LBB0_1:", "s_waitcnt vmcnt(2)", load, "s_barrier", token, "s_cbranch_scc1 .LBB0_1", "s_waitcnt vmcnt(0)", "s_endpgm"]
    good = [token, token, load, load, token, "s_waitcnt vmcnt(2)", "s_barrier"] + loop
    assert late_stages(good) == ([], 5)                       # the loop's start and four passes
    assert late_stages([l.replace("vmcnt(2)", "vmcnt(4)") for l in good])[0]
    assert late_stages(good[:7] + [".LBB0_1:", "s_waitcnt vmcnt(3)"] + loop[2:])[0]


@pytest.mark.parametrize("source", ["gemm_prefill_w4.hip", "gemm_prefill_w8.hip"])
def test_the_next_stage_has_landed_at_every_barrier(tmp_path, source):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no compiler here")
    out = tmp_path / "kernels.s"
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", str(out)], check=True, capture_output=True)
    late, looked_at = {}, 0
    for name, lines in kernels(out.read_text()):
        for second_tile in (False, True) if "tail" in name else (False,):
            found, barriers = late_stages(lines, second_tile)
            assert barriers >= 4, name
            looked_at += 1
            if found:
                late[name, second_tile] = found
    assert looked_at >= 10
    assert not late, late
