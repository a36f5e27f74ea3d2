"""The inline-assembly LDS reads of the attention kernels across basic blocks.
A read issued in one block may be waited for in another; until then no
instruction on any path may touch its destination registers (vector or
accumulation), whether the compiler placed a copy, a spill or another value
there. Data flow over each kernel's control-flow graph: the LDS operations in
flight at a block's entry are the union over its predecessors, aligned from
the most recent one, since they complete in order (CPU only)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2607_03333_amd import build

ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
HIPCC = os.path.join(ROCM, "bin", "hipcc")


def _regs(text):
    out = set()
    for m in re.finditer(r"\b([va])\[(\d+):(\d+)\]|\b([va])(\d+)\b", text):
        if m.group(5) is not None:
            out.add((m.group(4), int(m.group(5))))
        else:
            out.update((m.group(1), i) for i in range(int(m.group(2)), int(m.group(3)) + 1))
    return out


def _blocks(lines):
    """[(label, [instruction or asm marker])] of a kernel and its successors by block index."""
    bbs = [("entry", [])]
    for t in lines:
        m = re.match(r"^(\.LBB\S+?):", t)
        if m:
            bbs.append((m.group(1), []))
        elif re.match(r"^; %bb\.", t):
            bbs.append(("", []))
        else:
            bbs[-1][1].append(t)
    index = {label: i for i, (label, _) in enumerate(bbs) if label}
    succ = []
    for i, (_, body) in enumerate(bbs):
        to, falls = set(), True
        for t in body:
            m = re.match(r"s_(c?)branch\S*\s+(\.LBB\S+)", t)
            if m:
                to.add(index[m.group(2)])
                falls = falls and m.group(1) == "c"
            if t.startswith("s_endpgm"):
                falls = False
        if falls and i + 1 < len(bbs):
            to.add(i + 1)
        succ.append(to)
    return [b for _, b in bbs], succ


def _flow(body, pending, report=None):
    pending, in_asm = [set(p) for p in pending], False
    for t in body:
        if t.startswith(";;#ASMSTART") or t.startswith(";;#ASMEND"):
            in_asm = t.startswith(";;#ASMSTART")
            continue
        if not t or t[0] in ";.":
            continue
        op, _, args = t.replace("\t", " ").partition(" ")
        args = args.split(";")[0]
        if op == "s_waitcnt":
            m = re.search(r"lgkmcnt\((\d+)\)", t)
            if m:
                keep = int(m.group(1))
                pending = [] if keep == 0 else pending[-keep:]
            continue
        read = op.startswith("ds_read") and in_asm
        touched = _regs(args.split(",")[0] if read else args)
        if report is not None and any(p & touched for p in pending):
            report.append(t)
        if op.startswith("ds_") or op.startswith("s_load"):
            pending.append(_regs(args.split(",")[0]) if read else set())
    return pending[-64:]


def pending_read_uses(lines):
    """Instructions that touch the destination of an LDS read in flight."""
    bodies, succ = _blocks(lines)
    entry, work = {0: []}, [0]
    while work:
        i = work.pop()
        out = _flow(bodies[i], entry[i])
        for s in succ[i]:
            old = entry.get(s)
            n = max(len(out), len(old or []))
            new = [(out[-q] if q <= len(out) else set()) | (old[-q] if old and q <= len(old) else set())
                   for q in range(n, 0, -1)]
            if old is None or new != old:
                entry[s] = new
                work.append(s)
    report = []
    for i in sorted(entry):
        _flow(bodies[i], entry[i], report)
    return report


def test_the_flow_sees_a_spill_in_another_block():
    bad = """;;#ASMSTART
ds_read_b32 v5, v2
;;#ASMEND
s_cbranch_vccnz .LBB0_2
; %bb.1:
scratch_store_dword off, v5, off
.LBB0_2:
s_waitcnt lgkmcnt(0)
v_readfirstlane_b32 s26, v5
s_endpgm""".splitlines()
    assert pending_read_uses(bad) == ["scratch_store_dword off, v5, off"]
    good = [t for t in bad if not t.startswith("scratch")]
    assert pending_read_uses(good) == []


@pytest.mark.skipif(shutil.which(HIPCC) is None and not os.path.exists(HIPCC), reason="hipcc not installed")
def test_attention_kernels_leave_reads_in_flight_alone(tmp_path):
    out = tmp_path / "attention.s"
    cmd = [HIPCC, *build.DEVICE_FLAGS, f"-I{build.INCLUDE}", f"-I{build.CSRC}", "--cuda-device-only", "-S",
           "-o", str(out), os.path.join(build.CSRC, "attention.hip")]
    subprocess.run(cmd, check=True, capture_output=True, timeout=600)
    kernels, name = {}, None
    for line in out.read_text().splitlines():
        t = line.strip()
        m = re.match(r"^(_Z\S*attn_bf16\S*):", t)
        if m:
            name = m.group(1)
            kernels[name] = []
        elif t.startswith(".Lfunc_end"):
            name = None
        elif name:
            kernels[name].append(t)
    assert len(kernels) == 10  # narrow (4 and 8 waves, one and two row tiles per wave) and wide, 16- and 32-token blocks
    for name, lines in kernels.items():
        assert pending_read_uses(lines) == [], name
