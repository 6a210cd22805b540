"""CPU check of the LDS-direct kernels' stage reuse, on the assembly of this build.

These kernels move operands from global memory straight into LDS, three stages in turn: the
barrier of step t lets the loads of step t + 2 overwrite the stage that step t - 1 read.  A
wave must therefore have no LDS read in flight when it reaches a barrier.  That is timing
dependent on a GPU and shows in no result reliably, so it is checked where it is decided: in
the instructions that the compiler emitted.  A forward data flow over every kernel's blocks
counts the LDS instructions issued since the last wait that covers them (they complete in
order), the largest count over all ways into a block.
"""
import os
import re
import subprocess

import pytest

from paper_2207_04636_amd import build as B


def _kernels(asm):
    """(name, instruction and label lines) of every function of an assembly text."""
    name, body = None, []
    for line in asm.splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            name, body = m.group(1), []
        elif name and line.startswith(".Lfunc_end"):
            yield name, body
            name = None
        elif name:
            s = line.split(";")[0].strip()
            if s and (s.startswith(".LBB") or not s.startswith(".")):
                body.append(s)


def _reads_at_barriers(body):
    """Most LDS instructions in flight at each s_barrier of a kernel."""
    blocks, label = [[]], {}
    for s in body:
        if s.startswith(".LBB"):
            blocks.append([])
            label[s.rstrip(":")] = len(blocks) - 1
            continue
        blocks[-1].append(s)
        if re.match(r"s_c?branch|s_endpgm", s):
            blocks.append([])

    def run(block, n, out=None):
        for s in block:
            if s.startswith("ds_"):
                n += 1
            elif s.startswith("s_waitcnt"):
                m = re.search(r"lgkmcnt\((\d+)\)", s)
                n = min(n, int(m.group(1))) if m else n
            elif s == "s_barrier" and out is not None:
                out.append(n)
        return min(n, 64)

    entry, todo = {0: 0}, [0]
    while todo:
        i = todo.pop()
        n = run(blocks[i], entry[i])
        last = blocks[i][-1] if blocks[i] else ""
        m = re.match(r"s_(c?)branch\w*\s+(\.LBB\w+)", last)
        after = [label[m.group(2)]] if m else []
        if not (m and not m.group(1)) and not last.startswith("s_endpgm") and i + 1 < len(blocks):
            after.append(i + 1)
        for j in after:
            if entry.get(j, -1) < n:
                entry[j] = n
                todo.append(j)
    out = []
    for i in sorted(entry):
        run(blocks[i], entry[i], out)
    return out


def test_counts_reads_over_a_loop():
    """The counting itself: reads left in flight at the barrier, across a back edge too."""
    loop = [".LBB0_1:", "s_barrier", "ds_read_b64 v[0:1], v2", "ds_read_b64 v[4:5], v2", "{wait}",
            "s_cbranch_scc1 .LBB0_1", "s_endpgm"]
    assert _reads_at_barriers([s.format(wait="s_nop 0") for s in loop])[0] > 2
    assert _reads_at_barriers([s.format(wait="s_waitcnt vmcnt(0)") for s in loop])[0] > 2
    assert _reads_at_barriers([s.format(wait="s_waitcnt lgkmcnt(1)") for s in loop]) == [1]
    assert _reads_at_barriers([s.format(wait="s_waitcnt vmcnt(3) lgkmcnt(0)") for s in loop]) == [0]


def _sources():
    return sorted(f for f in os.listdir(B.CSRC) if f.endswith(".hip")
                  and "global_load_lds" in open(os.path.join(B.CSRC, f)).read())


@pytest.mark.parametrize("src", _sources())
def test_no_lds_read_in_flight_at_a_barrier(src, tmp_path):
    out = str(tmp_path / "k.s")
    cmd = [B._hipcc(), *B.COMMON, *B.DEVICE, "--cuda-device-only", "-S", os.path.join(B.CSRC, src), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    direct, bad = 0, {}
    for name, body in _kernels(open(out).read()):
        n = _reads_at_barriers(body)
        direct += any(re.match(r"(global|buffer)_load\w*lds|buffer_load.*\blds\b", s) for s in body)
        if any(n):
            bad[name] = n
    assert direct > 0, "no kernel of this source loads into LDS: the check has nothing to look at"
    assert not bad, bad
