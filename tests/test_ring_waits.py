"""The waits of the ring tiles (csrc/ring_k.h) in the code the compiler made of them: at every barrier of every path, the activations that
the step behind it reads have arrived.

A wait allows a number of outstanding loads, so it is right only while the loads it counts on are really issued: the compiler leaves
out a load whose result no path uses, while a load to LDS stays.  So what is checked is the AMD assembly, with the queue of outstanding
vector memory accesses followed through all branches."""
import os
import re
import subprocess

import pytest

from paper_2512_09277_amd import build

ACCESS = re.compile(r"(buffer|global|flat|scratch)_(load|store|atomic)")
BRANCH = re.compile(r"s_c?branch\w*\s+(\S+)")


def assembly(source, path):
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.check_call(["hipcc", *flags, "--cuda-device-only", "-S", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                           os.path.join(build.CSRC, source), "-o", path])
    with open(path) as f:
        return f.read()


def functions(text):
    """{name: [line]} of the instructions, the labels and the rings' marks of every function."""
    out, name = {}, None
    for raw in text.splitlines():
        line = raw.strip()
        if not line.startswith("; ring"):
            line = line.split(";")[0].strip()
        m = re.match(r"(_Z\w+):$", line)
        if m:
            name = m.group(1)
            out[name] = []
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name and line and (not line.startswith(".") or line.endswith(":")):
            out[name].append(line)
    return out


def weak_waits(lines):
    """[(line number, loads to LDS in flight, allowed)] where too many are; {(stages, loads of a stage)} of the rings passed."""
    label = {line[:-1]: i for i, line in enumerate(lines) if line.endswith(":")}
    weak, rings, seen = set(), set(), set()
    # next line; outstanding accesses from the oldest load to LDS on (True for those); the ring, and whether a barrier of it was passed
    todo = [(0, (), None, False)]
    while todo:
        at, queue, ring, begun = todo.pop()
        while at < len(lines):
            line = lines[at]
            at += 1
            if ACCESS.match(line):
                lds = re.search(r"\blds\b", line) is not None
                if lds or queue:
                    queue += (lds,)
            elif line.startswith("s_waitcnt"):
                m = re.search(r"vmcnt\((\d+)\)", line)
                if m:
                    queue = queue[max(len(queue) - int(m.group(1)), 0):]
                    while queue and not queue[0]:
                        queue = queue[1:]
            elif line.startswith("; ring of"):
                ring, begun = tuple(int(n) for n in re.findall(r"\d+", line)), False
                rings.add(ring)
            elif line == "; ring done":
                if queue:
                    weak.add((at, sum(queue), 0))
                ring = None
            elif line == "s_barrier" and ring:
                stages, loads = ring
                # of the stages that are being filled, the oldest is read behind the barrier
                allowed = (stages - 2 if begun else stages - 1) * loads
                begun = True
                if sum(queue) > allowed:
                    weak.add((at, sum(queue), allowed))
            elif line.startswith("s_endpgm") or line.startswith("s_setpc"):
                break
            elif BRANCH.match(line):
                state = (label[BRANCH.match(line).group(1)], queue, ring, begun)
                if state not in seen:
                    seen.add(state)
                    todo.append(state)
                if line.startswith("s_branch"):
                    break
            elif line.endswith(":"):
                state = (at - 1, queue, ring, begun)
                if (at, state) in seen:
                    break
                seen.add((at, state))
    return sorted(weak), rings


@pytest.mark.parametrize("source,tiles", [("gate.hip", {(3, 4), (4, 2)}), ("ffn.hip", {(4, 1), (4, 2), (3, 3), (3, 4)})])
def test_needed_activations_have_arrived(tmp_path, source, tiles):
    found = set()
    for name, lines in functions(assembly(source, str(tmp_path / "kernels.s"))).items():
        weak, rings = weak_waits(lines)
        assert not weak, (name, weak)
        found |= rings
    assert found == tiles


RING = """
; ring of 4 stages, 1 loads each
buffer_load_dwordx4 v1, s[0:3], s4 offen lds
global_load_dwordx4 v[2:5], v[6:7], off
buffer_load_dwordx4 v1, s[0:3], s4 offen lds
buffer_load_dwordx4 v1, s[0:3], s4 offen lds
buffer_load_dwordx4 v1, s[0:3], s4 offen lds
s_waitcnt vmcnt(3)
s_barrier
.LOOP:
buffer_load_dwordx4 v1, s[0:3], s4 offen lds
s_cbranch_scc1 .SKIP
global_load_dwordx4 v[2:5], v[6:7], off
.SKIP:
s_waitcnt vmcnt({n}) lgkmcnt(0)
s_barrier
s_cbranch_scc1 .LOOP
s_waitcnt vmcnt(0)
; ring done
s_endpgm
"""


@pytest.mark.parametrize("n,right", [(1, True), (2, True), (3, False)])
def test_the_walk_itself(n, right):
    """Four stages of one load: two may be in flight where a step ends, also on the path that leaves the weights out."""
    weak, rings = weak_waits(RING.format(n=n).split("\n"))
    assert rings == {(4, 1)} and (not weak) == right
