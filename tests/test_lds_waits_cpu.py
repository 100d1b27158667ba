"""The eight-wave kernels read LDS with instructions written in inline assembly
and wait for them by hand (s_waitcnt lgkmcnt), so the compiler does not know
when their registers are written.  This test compiles the kernels for gfx950
and follows every path through their assembly, branches and back edges
included: no instruction may touch a register that an LDS read still in flight
is going to write, and no read from inline assembly may be in flight at a
branch, where the compiler places the moves of values that change registers.

LDS operations complete in order, so a wait for a count of n leaves the n
newest; scalar loads share the counter and may complete in any order, so while
some are in flight a count only vouches for what it must.
"""
import os
import re
import subprocess

import pytest

from paper_2408_11743_amd import build as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2408_11743_amd", "csrc")
SMEM = "smem"


class AsmRead(frozenset):
    """Registers of an LDS read that the compiler does not know as one."""


def registers(text):
    out = set()
    for kind, lo, hi, one in re.findall(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        out |= {kind + str(i) for i in (range(int(lo), int(hi) + 1) if lo else (int(one),))}
    return out


class Line:
    def __init__(self, text, in_asm):
        self.text, self.asm = text, in_asm
        self.op, _, rest = text.partition(" ")
        self.regs = registers(rest)
        self.dest = frozenset(registers(rest.split(",")[0])) if self.op.startswith("ds_read") else frozenset()
        m = re.search(r"lgkmcnt\((\d+)\)", text) if self.op == "s_waitcnt" else None
        self.wait = int(m.group(1)) if m else None
        self.target = rest.strip() if self.op.startswith(("s_cbranch", "s_branch")) else None


def parse(body):
    """Instructions of one kernel, and the index each label stands at."""
    lines, labels, in_asm = [], {}, False
    for raw in body.splitlines():
        t = raw.strip()
        if t.startswith(";;#ASMSTART"):
            in_asm = True
        elif t.startswith(";;#ASMEND"):
            in_asm = False
        t = t.split(";")[0].strip()
        m = re.match(r"^(\.?\w+):", t)
        if m:
            labels[m.group(1)] = len(lines)
        elif t and not t.startswith("."):
            lines.append(Line(" ".join(t.split()), in_asm))
    return lines, labels


def completed(flight, n):
    """What may be in flight after a wait for a count of n."""
    scalar = flight.count(SMEM)
    drop = max(0, len(flight) - n - (scalar if n else 0))
    kept = []
    for f in flight:
        if drop and (f != SMEM or n == 0):
            drop -= 1
        else:
            kept.append(f)
    return tuple(kept)


def walk(lines, labels):
    """Follow every path; flight: the registers of each LDS read in flight, oldest first."""
    bad, seen, todo = [], set(), [(0, ())]
    leaders = set(labels.values())
    while todo:
        at, flight = todo.pop()
        while at < len(lines):
            if at in leaders:
                if (at, flight) in seen:
                    break
                seen.add((at, flight))
            line = lines[at]
            if line.wait is not None:
                flight = completed(flight, line.wait)
            for f in flight:
                if f != SMEM and f & line.regs:
                    bad.append("line %d: %s while %s is in flight" % (at, line.text, sorted(f)))
            if line.op.startswith("s_load") or line.op.startswith("s_buffer_load"):
                flight += (SMEM,)
            elif line.op.startswith("ds_"):
                flight += (AsmRead(line.dest) if line.asm else line.dest,)
            assert len(seen) < 200000
            if len(flight) > 64:
                bad.append("line %d: %s is one of 65 operations nobody waits for" % (at, line.text))
                break
            if line.target:
                pending = sum(isinstance(f, AsmRead) for f in flight)
                if pending:
                    bad.append("line %d: %s with %d reads in flight" % (at, line.text, pending))
                todo.append((labels[line.target], flight))
                if line.op == "s_branch":
                    break
            if line.op == "s_endpgm":
                break
            at += 1
    return sorted(set(bad))


def kernels(src, tmp_path):
    out = str(tmp_path / "k.s")
    flags = B.SOURCE_FLAGS.get(src, B.DEVICE_FLAGS)
    subprocess.run([B.hipcc(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                    "-I", CSRC, *flags, "--cuda-device-only", "-S", "-o", out, os.path.join(CSRC, src)], check=True,
                   capture_output=True)
    text = open(out).read()
    for m in re.finditer(r"^(_Z\S*w4a16_\w+_kernel\S*):", text, re.M):
        yield m.group(1), *parse(text[m.end():text.index(".Lfunc_end", m.end())])


@pytest.mark.parametrize("src,count", [("pair.hip", 2), ("tile8.hip", 4), ("wide.hip", 2)])
def test_no_register_is_used_before_its_read_has_landed(tmp_path, src, count):
    n = 0
    for name, lines, labels in kernels(src, tmp_path):
        n += 1
        assert sum(l.asm and l.op.startswith("ds_read") for l in lines) > 20, name
        bad = walk(lines, labels)
        assert not bad, "%s: %d\n%s" % (name, len(bad), "\n".join(bad[:8]))
    assert n == count


def test_the_walk_finds_a_missing_wait():
    def run(text):
        return walk(*parse(text))
    ok = "ds_read_b128 v[0:3], v9\nds_read_b64 v[4:5], v9\ns_waitcnt lgkmcnt(1)\nv_add_f32 v8, v0, v3\n" \
         "s_waitcnt lgkmcnt(0)\nv_mov_b32_e32 v8, v5\ns_endpgm\n"
    assert not run(ok)
    assert len(run(ok.replace("lgkmcnt(1)", "lgkmcnt(2)"))) == 1
    assert len(run(ok.replace("lgkmcnt(0)", "vmcnt(0)"))) == 1
    assert len(run(ok.replace("ds_read_b64 v[4:5], v9", "s_load_dword s0, s[2:3], 0x0"))) == 1  # which of the two is done?
    mine = ";;#ASMSTART\nds_read_b32 v0, v9\n;;#ASMEND\ns_cbranch_scc1 .LBB0_1\n.LBB0_1:\ns_waitcnt lgkmcnt(0)\ns_endpgm\n"
    assert run(mine) and not run(mine.replace(";;#ASMEND", ";;#ASMEND\ns_waitcnt lgkmcnt(0)"))
    loop = ".LBB0_1:\ns_waitcnt lgkmcnt(0)\nv_mov_b32_e32 v1, v0\nds_read_b32 v0, v9\nv_mov_b32_e32 v2, v3\n" \
           "s_cbranch_scc1 .LBB0_1\ns_waitcnt lgkmcnt(0)\ns_endpgm\n"
    assert not run(loop)
    assert run(loop.replace("v2, v3", "v2, v0")) and run(loop.replace(".LBB0_1:\ns_waitcnt lgkmcnt(0)", ".LBB0_1:"))
