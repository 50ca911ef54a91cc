"""Build-time guard for the stage of group_fwd_kernel (no GPU needed): a wave refills its own stage with loads that go straight to LDS, which
nothing but a wait keeps behind the reads of the stage's last contents.  On every path from a read to a refill the generated code has to
hold the wait that the source asks for (an inline-assembly s_waitcnt lgkmcnt(0)); that the compiler happens to wait there is not enough."""
import os
import re
import subprocess

from paper_2210_03858_amd import build
from test_isa_guards import ROOT


def _unguarded(body):
    """(reads, refills, refills that some path reaches from a read without the wait)"""
    blocks, name = {"": []}, ""  # label -> instructions; a wait that the source asks for as "guard"
    asked = False
    for line in (l.strip() for l in body.split("\n")):
        if line.startswith(";;#ASM"):
            asked = line.endswith("START")
        elif re.match(r"\.LBB\w+:", line):
            blocks[line.split(":")[0]] = [("next", name)]  # (of the block before, replaced below)
            name = line.split(":")[0]
        elif line and line[0] not in ";.":
            guard = asked and line.startswith("s_waitcnt") and "lgkmcnt(0)" in line
            kind = "guard" if guard else "read" if line.startswith("ds_read") else "refill" if re.match(r"buffer_load.*\blds\b", line) else line
            blocks[name].append((kind, line))
    names, into = list(blocks), {n: {} for n in blocks}  # into: block -> {predecessor: position of the jump}
    for i, n in enumerate(names):
        blocks[n] = [x for x in blocks[n] if x[0] != "next"]
        ends = False
        for at, (kind, line) in enumerate(blocks[n]):
            jump = re.match(r"s_c?branch\w*\s+(\.LBB\w+)", line)
            if jump:
                into[jump.group(1)].setdefault(n, set()).add(at)
            ends = line.startswith("s_branch ") or line.startswith("s_endpgm")
        if not ends and i + 1 < len(names):
            into[names[i + 1]].setdefault(n, set()).add(len(blocks[n]))

    def state_at(n, at, start):
        for kind, _ in blocks[n][:at]:
            start = True if kind == "guard" else False if kind == "read" else start
        return start
    safe = {n: True for n in blocks}
    while True:  # a block starts safe if all jumps to it are
        new = {n: all(state_at(p, at, safe[p]) for p, places in into[n].items() for at in places) for n in blocks}
        if new == safe:
            break
        safe = new
    reads = sum(kind == "read" for b in blocks.values() for kind, _ in b)
    refills = [(n, at, line) for n, b in blocks.items() for at, (kind, line) in enumerate(b) if kind == "refill"]
    return reads, len(refills), [line for n, at, line in refills if not state_at(n, at, safe[n])]


def test_a_path_without_the_wait_is_seen():
    wait = [";;#ASMSTART", "s_waitcnt lgkmcnt(0)", ";;#ASMEND"]
    first, loop = ["buffer_load_dwordx4 v1, s[0:3], s4 offen lds"], [".LBB0_1:", "ds_read_b128 v[2:5], v6"]
    refill = ["buffer_load_dwordx4 v7, s[0:3], s4 offen lds", "s_cbranch_scc1 .LBB0_1", "s_endpgm"]
    assert _unguarded("\n".join(first + loop + wait + refill)) == (1, 2, [])
    assert _unguarded("\n".join(first + loop + ["s_waitcnt lgkmcnt(0)"] + refill)) == (1, 2, refill[:1])  # the compiler's own
    around = ["s_cbranch_scc0 .LBB0_2"] + wait + [".LBB0_2:"]
    assert _unguarded("\n".join(first + loop + around + refill)) == (1, 2, refill[:1])
    back = [".LBB0_3:"] + refill[:1] + ["s_endpgm"] + loop + ["s_branch .LBB0_3"]  # the refill stands before the read
    assert _unguarded("\n".join(first + ["s_branch .LBB0_1"] + back))[2] == refill[:1]


def test_every_refill_waits_for_the_reads_of_its_stage(tmp_path):
    src, out = os.path.join(ROOT, "paper_2210_03858_amd", "csrc", "bcq_fused.hip"), str(tmp_path / "bcq_fused.s")
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-fPIC", "-Wall", "-Wno-unused-function")]
    r = subprocess.run([build._hipcc()] + flags + ["-S", "--cuda-device-only", src, "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    bodies = re.findall(r"^(_ZN3bcq16group_fwd_kernelILi\dELi\dELi\dEE\w*):[^\n]*\n(.*?)\.Lfunc_end", open(out).read(), re.S | re.M)
    assert len(bodies) == 20  # one to four planes, one and two words to a lane with one and two tiles of tokens, four words with one
    for name, body in bodies:
        reads, refills, bad = _unguarded(body)
        assert reads >= 4 and refills >= 2 and not bad, (name, reads, refills, bad[:3])
