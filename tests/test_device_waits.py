"""The histogram kernel's ticket (no GPU; the assembly that the library's own
flags give): the last block reads the bins that every wave of every block added
to, and a barrier alone does not wait for memory operations, so each wave's
additions must be complete when it reaches the barrier in front of the ticket.
The scan follows every branch and keeps the additions without a wait since."""
import os
import re
import shutil
import subprocess

import pytest

PKG = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2608_13255_amd")


def kernels(asm, name):
    for m in re.finditer(r"^(_ZN2gc\S+):.*?^\.Lfunc_end", asm, re.S | re.M):
        if name in m.group(1):
            yield m.group(1), [line.split(";")[0].strip() for line in m.group(0).splitlines()]


def open_at_barriers(lines, op):
    """(barriers met, those that some path reaches with an `op` not waited for)."""
    label = {line[:-1]: i for i, line in enumerate(lines) if re.match(r"\.LBB\S+:$", line)}
    todo, done, met, bad = [(0, False)], set(), set(), set()
    while todo:
        i, pending = todo.pop()
        if i >= len(lines) or (i, pending) in done:
            continue
        done.add((i, pending))
        line = lines[i]
        if line.startswith("s_barrier"):
            met.add(i)
            if pending:
                bad.add(i)
        if line.split(" ")[0].split("\t")[0] == op:
            pending = True
        if re.match(r"s_waitcnt\b.*vmcnt\(0\)", line):
            pending = False
        branch = re.match(r"s_c?branch\w*\s+(\.LBB\S+)", line)
        if branch:
            todo.append((label[branch.group(1)], pending))
        if not re.match(r"s_(branch|endpgm)\b", line):
            todo.append((i + 1, pending))
    return met, bad


def test_scan_sees_a_missing_wait():
    body = [".LBB0_1:", "global_atomic_add_x2 v[0:1], v[2:3], off", "s_cbranch_execnz .LBB0_1", "s_barrier", "s_endpgm"]
    assert open_at_barriers(body, "global_atomic_add_x2") == ({3}, {3})
    assert open_at_barriers(body[:3] + ["s_waitcnt vmcnt(0)"] + body[3:], "global_atomic_add_x2") == ({4}, set())


@pytest.mark.skipif(shutil.which("make") is None or not os.path.exists("/opt/rocm/bin/hipcc"), reason="no hipcc")
def test_bins_are_added_before_the_ticket(tmp_path):
    out = tmp_path / "gc_coverage.hip.s"
    subprocess.run(["make", "-s", "-C", PKG, f"BUILD={tmp_path}", str(out)], check=True, capture_output=True, timeout=300)
    asm = out.read_text()
    found = 0
    for name, lines in kernels(asm, "k_cov_hist"):
        assert sum("global_atomic_add_x2" in line for line in lines) >= 1, name
        met, bad = open_at_barriers(lines, "global_atomic_add_x2")
        assert met and not bad, name
        found += 1
    assert found == 4   # selection and scores, each with and without the staleness step
