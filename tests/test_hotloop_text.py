"""The hot loop's assembly, read as text: on every path through it a register
is written before it is read.  What the block finds in a register it did not
write is whatever the compiler left there; results may not show it (the order
in which groups run, for one, does not change them)."""
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1907_08467_amd", "csrc")


def block():
    """The block's instructions and labels, and the registers it is handed."""
    src = open(os.path.join(CSRC, "hotloop.h")).read().replace("#pragma once", "")
    out = subprocess.run(["g++", "-E", "-P", "-x", "c++", "-"], input=src, capture_output=True, text=True, check=True).stdout
    out = out[out.index("asm volatile("):]
    text, pos = "", len("asm volatile(")
    lit = re.compile(r'\s*"((?:[^"\\]|\\.)*)"')
    while m := lit.match(out, pos):
        text += m.group(1)
        pos = m.end()
    text = text.replace("\\n", "\n").replace("%=", "")
    operands = out[pos:out.index(";", pos)].split('"memory"')[0]     # outputs and inputs; clobbers follow
    pinned = {r for c in re.findall(r'"[+=]?\{([^}]*)\}"', operands) for r in regs(c)}
    return [l.strip() for l in text.split("\n") if l.strip()], pinned


def regs(arg):
    """Registers of one operand: s12, v[100:101], vcc, exec, m0, %[name]."""
    arg = arg.strip()
    m = re.fullmatch(r"([sv])\[(\d+):(\d+)\]", arg)
    if m:
        return [f"{m.group(1)}{k}" for k in range(int(m.group(2)), int(m.group(3)) + 1)]
    if re.fullmatch(r"[sv]\d+", arg) or arg in ("vcc", "m0"):
        return [arg]
    return []


def reads_and_writes(op, args):
    dst = 1
    if op.startswith(("s_cmp", "s_bitcmp", "s_cbranch", "s_branch", "s_waitcnt", "s_nop", "s_setpc", "ds_write",
                      "global_store")):
        dst = 0
    writes = [r for a in args[:dst] for r in regs(a)]
    reads = [r for a in args[dst:] for r in regs(a)]
    if op in ("s_bitset0_b64", "s_bitset1_b64", "v_writelane_b32"):
        reads += writes
    if "vccnz" in op or "vccz" in op:
        reads.append("vcc")
    if op.startswith("s_cselect") or op in ("s_cbranch_scc0", "s_cbranch_scc1"):
        reads.append("scc")
    if op.startswith(("s_add", "s_sub_", "s_cmp", "s_bitcmp", "s_and", "s_or_", "s_xor", "s_lshl", "s_lshr", "s_bfe",
                      "s_min", "s_max")):
        writes.append("scc")
    return reads, writes


def unwritten(lines, pinned):
    """(register, instruction) pairs read on some path before any write to them."""
    ins, labels, entries = [], {}, {}
    for l in lines:
        if l.endswith(":"):
            labels[l[:-1]] = len(ins)
        elif l.startswith(".org"):
            m = re.match(r"\.org \S+ \+ 128\*(\d+)", l)
            entries.setdefault(int(m.group(1)), []).append(len(ins))
        elif not l.startswith("."):
            op, _, rest = l.partition(" ")
            args = [re.sub(r"\s*(offset\d?|bitop3):.*| off$", "", a.strip()) for a in rest.split(",")]
            ins.append((op, args, l))
    header = open(os.path.join(CSRC, "hotloop.h")).read()
    m = re.search(r"kHotWork = (\d+)", header)
    work = int(m.group(1)) if m else 1 << 30
    # slots that no word names (opcode 0) are only branched to
    ops = re.findall(r"0x(..)", re.search(r"kHotSlotOp\[kHotSlots\] = \{(.*?)\}", header, re.S).group(1))
    handlers = [i for s, v in entries.items() if s == 0 or s < work and ops[s] != "00" for i in v] + [labels[".Lline"]]
    works = [i for s, v in entries.items() if s >= work for i in v]

    def successors(i):
        op, args, _ = ins[i]
        if op == "s_branch":
            return [labels[args[0]]]
        if op.startswith("s_cbranch"):
            return [labels[args[0]], i + 1]
        if op.startswith("s_setpc"):
            return {"s[74:75]": handlers, "s[90:91]": works, "s[96:97]": []}[args[0]]
        if op.startswith("s_swappc"):                # the call, and (with what it may write left out) the return
            return [labels[".Lsnap"], i + 1]
        return [i + 1]

    # the table of waiting groups is written and read lane by lane, m0 is saved and restored
    written = {0: frozenset(pinned | {f"v{k}" for k in range(102, 109)} | {"m0"})}
    todo, bad = [0], set()
    while todo:
        i = todo.pop()
        if i >= len(ins):
            continue
        reads, writes = reads_and_writes(ins[i][0], ins[i][1])
        have = written[i]
        bad |= {(r, i) for r in reads if r not in have}      # (`have` only shrinks)
        after = have | set(writes)
        for j in successors(i):
            meet = after & written[j] if j in written else after
            if written.get(j) != meet:
                written[j] = meet
                todo.append(j)
    return sorted({(r, ins[i][2]) for r, i in bad})


def test_registers_are_written_before_they_are_read():
    assert unwritten(*block()) == []


@pytest.mark.parametrize("line,reg", [("s_mov_b64 s[54:55], 0", "s54"), ("s_movk_i32 s68, 1696", "s68"),
                                      ("v_mov_b32 %[obase], v111", None)])
def test_the_check_sees_a_missing_write(line, reg):
    lines, pinned = block()
    assert line in lines
    found = unwritten([l for l in lines if l != line], pinned)
    assert any(r == reg for r, _ in found) == (reg is not None)


def test_labels_differ_in_every_copy():
    """The compiler appends a number to each label of a copy of the block: a label
    that ends in a digit could become another one's (.Lsync2 of copy 0, .Lsync of 20)."""
    src = open(os.path.join(CSRC, "hotloop.h")).read()
    labels = set(re.findall(r"(\.L\w*)%=", src))
    assert len(labels) > 20 and not [l for l in labels if l[-1].isdigit()]
    assert not re.search(r'(?:#?\b(?:id|tk|code|k|slot)) "%=', src)     # a macro's argument at the end
