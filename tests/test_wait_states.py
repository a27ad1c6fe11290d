"""The compiler puts no wait states in front of inline asm.  On gfx950 a vector memory instruction may read an SGPR that
a vector instruction wrote five wait states earlier or before; the library's loads to LDS are inline asm, so their
distance is counted here in the built code: every instruction is one wait state, s_nop N is N + 1, along the listing and
across each branch."""
from __future__ import annotations

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2603_12707_amd", "libhs.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
NEED = 5


def _sgprs(text):
    regs = {int(r) for r in re.findall(r"\bs(\d+)\b", text)}
    for lo, hi in re.findall(r"\bs\[(\d+):(\d+)\]", text):
        regs |= set(range(int(lo), int(hi) + 1))
    return regs


def _functions(listing):
    """Instructions (offset, text, branch target offset or None) of each function of an llvm-objdump listing."""
    fn, start = [], 0
    for line in listing.splitlines():
        head = re.match(r"([0-9a-f]+) <(.+)>:", line)
        if head:
            if fn:
                yield fn
            fn, start = [], int(head.group(1), 16)
            continue
        ins = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+):", line)
        if ins:
            target = re.search(r"<[^>+]+(?:\+0x([0-9a-f]+))?>\s*$", line) if ins.group(1).startswith("s_") else None
            to = int(target.group(1) or "0", 16) if target and "branch" in ins.group(1) else None
            fn.append((int(ins.group(2), 16) - start, ins.group(1), to))
    if fn:
        yield fn


def _hazards(fn):
    at = {off: i for i, (off, _, _) in enumerate(fn)}

    def reads(i, left, regs, found, src):
        """regs: SGPRs written `NEED - left` wait states before instruction i"""
        while left > 0 and regs and i < len(fn):
            off, text, to = fn[i]
            op = text.split()[0]
            if re.match(r"(buffer|global|flat|scratch)_", op) and regs & _sgprs(text):
                found.append((src, text))
                return
            if op.startswith("s_"):  # a scalar write takes the register's place
                dst = text[len(op):].split(",")[0]
                if not re.match(r"s_(nop|waitcnt|barrier|cmp|bitcmp|cbranch|branch|endpgm)", op):
                    regs = regs - _sgprs(dst)
            left -= int(text.split()[1], 0) + 1 if op == "s_nop" else 1
            if to is not None and to in at:
                reads(at[to], left, regs, found, src)
                if op == "s_branch":
                    return
            i += 1

    found = []
    for i, (_, text, _) in enumerate(fn):
        op = text.split()[0]
        if op.startswith("v_"):
            dst = _sgprs(text[len(op):].split(",")[0])
            if dst:
                reads(i + 1, NEED, dst, found, text)
    return found


def test_scanner():
    def listing(*ins):
        return "0000000000001000 <k>:\n" + "".join("\t%s // %012X: 00000000%s\n" % (t.split("@")[0], 0x1000 + 4 * i,
                                                   " <k+0x%s>" % t.split("@")[1] if "@" in t else "")
                                                   for i, t in enumerate(ins))
    load = "buffer_load_dwordx4 v3, s[40:43], s6 offen lds"

    def count(*ins):
        return [len(_hazards(f)) for f in _functions(listing(*ins))]
    assert count("v_readfirstlane_b32 s41, v2", "s_mov_b32 m0, s23", "s_nop 0", load) == [1]
    assert count("v_readfirstlane_b32 s41, v2", "s_nop 2", "s_mov_b32 m0, s23", "s_nop 0", load) == [0]
    assert count("v_readfirstlane_b32 s6, v2", "s_mov_b32 s6, s23", "s_nop 0", load) == [0]
    assert count("s_nop 0", load, "v_readfirstlane_b32 s6, v2", "s_branch 65532@0") == [1]


@pytest.mark.skipif(not os.path.exists(LIB) or not os.path.exists(OBJDUMP), reason="no built library or llvm-objdump")
def test_loads_to_lds_read_settled_sgprs(tmp_path):
    lib = shutil.copy(LIB, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True)
    loads = 0
    for name in sorted(os.listdir(tmp_path)):
        if not name.endswith("gfx950"):
            continue
        text = subprocess.run([OBJDUMP, "-d", os.path.join(tmp_path, name)], check=True, capture_output=True,
                              text=True).stdout
        loads += len(re.findall(r"buffer_load_dwordx4 .* lds", text))
        for fn in _functions(text):
            assert not _hazards(fn), _hazards(fn)[:3]
    assert loads > 100
