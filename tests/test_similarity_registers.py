"""The fragment reads of the similarity kernel are loads in inline assembly, whose registers the compiler takes as written at
once.  From the assembly of the kernel as it is built: between such a read and the wait for it, on every path, no instruction
may touch its registers."""
import os
import re
import subprocess

import pytest

from paper_2601_03067_amd import build as kbuild

REG = re.compile(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+)\b)")


def _regs(text):
    out = set()
    for kind, lo, hi, one in REG.findall(text):
        out |= {(kind, i) for i in (range(int(lo), int(hi) + 1) if lo else (int(one),))}
    return out


def _blocks(lines):
    """-> ([(label, instructions)], successors): basic blocks in text order."""
    blocks = [("entry", [])]
    for line in lines:
        label = re.match(r"^(\.LBB\w+):", line)
        if label:
            blocks.append((label.group(1), []))
            continue
        t = line.split(";")[0].strip()
        if not t or t.startswith(".") or t.endswith(":"):
            continue
        blocks[-1][1].append(t)
        if t.startswith(("s_cbranch", "s_branch", "s_endpgm")):
            blocks.append(("", []))
    at = {name: i for i, (name, _) in enumerate(blocks) if name}
    succ = []
    for i, (_, ins) in enumerate(blocks):
        last = ins[-1] if ins else ""
        nxt = [at[last.split()[1]]] if last.startswith(("s_cbranch", "s_branch")) else []
        if not last.startswith(("s_branch", "s_endpgm")) and i + 1 < len(blocks):
            nxt.append(i + 1)
        succ.append(nxt)
    return blocks, succ


def _touched_in_flight(lines):
    blocks, succ = _blocks(lines)
    entry = [frozenset()] * len(blocks)

    def walk(i, found=None):
        flight = set(entry[i])
        for t in blocks[i][1]:
            if "lgkmcnt(0)" in t:
                flight.clear()
                continue
            if found is not None and _regs(t) & flight:
                found.append(t)
            if t.startswith("ds_read_b128"):
                flight |= _regs(t.split(None, 1)[1].split(",")[0])
        return frozenset(flight)

    todo = list(range(len(blocks)))
    while todo:
        i = todo.pop()
        out = walk(i)
        for s in succ[i]:
            if not out <= entry[s]:
                entry[s] = entry[s] | out
                todo.append(s)
    found = []
    for i in range(len(blocks)):
        walk(i, found)
    return found


def test_no_register_is_touched_while_its_read_is_in_flight(tmp_path):
    try:
        hipcc = kbuild._hipcc()
    except RuntimeError:
        pytest.skip("no hipcc here")
    asm = tmp_path / "similarity.s"
    subprocess.check_call([hipcc, *kbuild.FLAGS, "--offload-device-only", "-S", os.path.join(kbuild.CSRC, "similarity.hip"), "-o", str(asm)],
                          stderr=subprocess.DEVNULL)
    kernels, name = {}, None
    for line in asm.read_text().split("\n"):
        start = re.match(r"^(_Z\w*similarity_ring_kernel\w*):", line)
        if start:
            name = start.group(1)
            kernels[name] = []
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name:
            kernels[name].append(line)
    assert len(kernels) >= 20
    bad = {k: v[:3] for k, v in ((k, _touched_in_flight(v)) for k, v in kernels.items()) if v}
    assert not bad, bad
