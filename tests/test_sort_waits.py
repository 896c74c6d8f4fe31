"""Ordering in the sort's kernels that no run can show reliably, read off the
assembly that the build's own flags give for gfx950: every path through a
kernel is followed (loops included), block by block.

sort_count: the last group to finish reads every group's counts, so no atomic of
a wave may be on its way when the wave passes the barrier before the group's
ticket.  sort_arrange: the last group clears the request that every wave
reads on entry, so each path to the ticket passes a barrier, also that of a
group whose segments are all empty."""
import os
import re
import subprocess

import pytest

from paper_1909_09613_amd import build as B


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "sort.s"
    subprocess.run([B.HIPCC] + B.FLAGS + ["-x", "hip", "--cuda-device-only", "-S", os.path.join(B.CSRC, "sort.hip"),
                                          "-o", str(out)], check=True, stderr=subprocess.DEVNULL)
    found, name = {}, None
    for line in out.read_text().splitlines():
        line = line.split(";")[0].strip()
        m = re.match(r"(_Z\w*sort_(?:count|arrange)\w*):$", line)
        if m:
            name = m.group(1)
            found[name] = []
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name and line and (not line.startswith(".") or line.startswith(".LBB")):
            found[name].append(line)
    return found


def _follow(lines, state, step):
    """Every state step() can leave an instruction in, over all paths."""
    where = {ln[:-1]: i for i, ln in enumerate(lines) if ln.endswith(":")}
    todo, seen = [(0, state)], set()
    while todo:
        i, s = todo.pop()
        if (i, s) in seen or i >= len(lines):
            continue
        seen.add((i, s))
        ln = lines[i]
        op = ln.split()[0]
        assert not op.startswith(("s_setpc", "s_swappc", "s_call")), ln
        if op.startswith("s_endpgm"):
            continue
        if op.startswith(("s_branch", "s_cbranch")):
            todo.append((where[ln.split()[-1]], s))
            if op.startswith("s_branch"):
                continue
        todo.append((i + 1, s if ln.endswith(":") else step(ln, s)))


def _ticket(ln):
    return ln.startswith("global_atomic_add ") and ln.endswith("sc0")


def _of(kernels, which):
    got = [k for k in kernels if which in k]
    assert len(got) >= 4   # both precisions, 2D and 3D
    return got


def test_counts_have_landed_before_the_ticket(kernels):
    for name in _of(kernels, "sort_count"):
        bad = []

        def step(ln, on_the_way):
            if ln.startswith("global_atomic_") and not ln.endswith("sc0"):
                return True
            if ln.startswith("s_waitcnt") and "vmcnt(0)" in ln:
                return False
            if ln.startswith("s_barrier") and on_the_way:
                bad.append(ln)
            return on_the_way

        assert any(map(_ticket, kernels[name]))
        _follow(kernels[name], False, step)
        assert not bad, name


def test_every_wave_has_read_the_request_before_the_ticket(kernels):
    for name in _of(kernels, "sort_arrange"):
        bad = []

        def step(ln, passed):
            if ln.startswith("s_barrier"):
                return True
            if _ticket(ln) and not passed:
                bad.append(ln)
            return passed

        assert any(map(_ticket, kernels[name]))
        _follow(kernels[name], False, step)
        assert not bad, name
