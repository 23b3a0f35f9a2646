"""Asynchronous global -> LDS copies against the LDS reads and address registers
around them, in the compiled kernels.

A copy lands in LDS whenever its data arrives, and the compiler neither counts
it nor orders it: it only sees the asm block.  So no LDS read may be outstanding
where a copy is issued (the copy may be into the slot that the read is from), and
no vector instruction may write a scalar register that a copy in an asm block
reads less than five wait states later (the compiler's own hazard handling does
not look into asm blocks).  Both are checked on the machine code of the packed
linear's small-batch kernels, over every path through them."""
import os
import re
import subprocess

import pytest

from paper_2308_13137_amd import build

WIDE = [(2, 2), (6, 1), (7, 2)]  # BITS, RT of the kernel for many rows
INSTANCES = [  # BITS, TT, RT, SUB, 16-byte copies
    (4, 4, 1, 1, True), (2, 4, 2, 2, True), (3, 4, 1, 4, False), (7, 4, 1, 4, True), (4, 16, 2, 1, True), (6, 8, 1, 2, True),
    (3, 24, 1, 1, True), (5, 16, 1, 2, False), (4, 32, 1, 2, True),
]

SOURCE = """
#include "packed_linear.h"
namespace oq {
hipError_t all(const LinArgs& a, const uint16_t* X, void* Y) {
  hipError_t e = hipSuccess;
%s
  return e;
}
}
"""


def blocks_of(lines):
    """Basic blocks of one kernel's assembly: {label: (instructions, successors)}."""
    blocks, order, name = {}, [], "entry"
    blocks[name] = []
    order.append(name)
    fresh = 0
    for line in lines:
        line = line.split(";")[0].strip() if not line.strip().startswith(";") else ""
        if not line or (line.startswith(".") and not line.endswith(":")):
            continue
        if line.endswith(":"):
            name = line[:-1]
            blocks[name] = []
            order.append(name)
            continue
        blocks[name].append(line)
        if line.startswith(("s_branch", "s_cbranch", "s_endpgm")):
            fresh += 1
            name = f"fall{fresh}"
            blocks[name] = []
            order.append(name)
    succ = {}
    for i, b in enumerate(order):
        last = blocks[b][-1] if blocks[b] else ""
        nxt = [order[i + 1]] if i + 1 < len(order) else []
        if last.startswith("s_endpgm"):
            succ[b] = []
        elif last.startswith("s_branch"):
            succ[b] = [last.split()[1]]
        elif last.startswith("s_cbranch"):
            succ[b] = [last.split()[1]] + nxt
        else:
            succ[b] = nxt
    return blocks, succ


def flow(blocks, succ, start, step, join):
    """Forward data flow to a fixed point; step(state, instruction) -> state."""
    state, work = {"entry": start}, ["entry"]
    while work:
        b = work.pop()
        s = state[b]
        for ins in blocks[b]:
            s = step(s, ins)
        for t in succ[b]:
            new = s if t not in state else join(state[t], s)
            if t not in state or new != state[t]:
                state[t] = new
                work.append(t)
    return state


def outstanding_reads(s, ins):
    """At most this many LDS reads may be outstanding (they return in order)."""
    if re.match(r"ds_(read|load)", ins):
        return min(s + 1, 64)
    if ins.startswith("s_waitcnt"):
        m = re.search(r"lgkmcnt\((\d+)\)", ins)
        return min(s, int(m.group(1))) if m else s
    return s


def vector_written(s, ins):
    """{scalar register: wait states since a vector instruction wrote it}, up to 5."""
    if ins.startswith("s_nop"):
        return {r: n + int(ins.split()[1], 0) + 1 for r, n in s.items() if n + int(ins.split()[1], 0) + 1 < 5}
    out = {r: n + 1 for r, n in s.items() if n + 1 < 5}
    if ins.startswith("v_"):
        # destinations that are scalar: readlane's, a compare's, a carry's
        for op in ins.split(None, 1)[1].split(",")[:2]:
            op = op.strip()
            m = re.fullmatch(r"s(\d+)", op)
            if m and (op == ins.split(None, 1)[1].split(",")[0].strip()):
                out[int(m.group(1))] = 0
            m = re.fullmatch(r"s\[(\d+):(\d+)\]", op)
            if m:
                out.update({r: 0 for r in range(int(m.group(1)), int(m.group(2)) + 1)})
    return out


def least(a, b):
    return {r: min(a.get(r, 9), b.get(r, 9)) for r in a.keys() | b.keys()}


def findings(lines):
    """(copies, copies with an LDS read outstanding, copies too soon after a vector write)."""
    blocks, succ = blocks_of(lines)
    copy = re.compile(r"(global_load_lds|buffer_load\w* .*\blds\b)")
    n, unordered, hazards = 0, [], []
    reads = flow(blocks, succ, 0, outstanding_reads, max)
    regs = flow(blocks, succ, {}, vector_written, least)
    for b in reads:
        r, w = reads[b], regs[b]
        for ins in blocks[b]:
            if copy.match(ins):
                n += 1
                if r:
                    unordered.append((b, ins, r))
                for m in re.finditer(r"s\[(\d+):(\d+)\]", ins):
                    if any(k in w for k in range(int(m.group(1)), int(m.group(2)) + 1)):
                        hazards.append((b, ins))
            r, w = outstanding_reads(r, ins), vector_written(w, ins)
    return n, unordered, hazards


def kernels(asm):
    """{symbol: lines} of the kernels in an assembly listing."""
    out, name = {}, None
    for line in asm.splitlines():
        m = re.match(r"(_Z\w+):", line)
        if m:
            name = m.group(1)
            out[name] = []
        elif name and line.startswith(".Lfunc_end"):
            name = None
        elif name:
            out[name].append(line)
    return out


def test_the_scan_finds_what_it_looks_for():
    loop = ["ds_read_b32 v1, v0", "s_waitcnt lgkmcnt(1)", ".LBB0_1:", "global_load_lds_dwordx4 v2, s[4:5]",
            "ds_read_b32 v1, v0", "s_cbranch_scc1 .LBB0_1", "s_endpgm"]
    assert len(findings(loop)[1]) == 1
    waited = loop[:1] + ["s_waitcnt lgkmcnt(0)"] + loop[2:5] + ["s_waitcnt vmcnt(0) lgkmcnt(0)"] + loop[5:]
    assert findings(waited) == (1, [], [])
    assert len(findings(loop[:2] + loop[2:5] + ["s_waitcnt lgkmcnt(0)"] + loop[5:])[1]) == 1   # the first pass
    soon = ["v_readfirstlane_b32 s5, v0", "s_nop 2", "global_load_lds_dword v2, s[4:5]", "s_endpgm"]
    assert len(findings(soon)[2]) == 1
    assert findings([soon[0], "s_nop 4"] + soon[2:])[2] == []


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
def test_refills_of_the_packed_linears_rings_follow_the_slots_reads(tmp_path):
    src = tmp_path / "instances.hip"
    calls = [f"  e = launch_mfma<{b}, {tt}, {rt}, {sub}, 2, {str(a16).lower()}>(a, X, {min(tt, 4)}, Y);"
             for b, tt, rt, sub, a16 in INSTANCES]
    calls += [f"  e = launch_wide<{b}, {rt}>(a, X, 32, Y);" for b, rt in WIDE]
    src.write_text(SOURCE % "\n".join(calls))
    asm = tmp_path / "instances.s"
    subprocess.run([build.HIPCC, *build.FLAGS, "-Wno-everything", "--cuda-device-only", "-S", str(src), "-o", str(asm)],
                   check=True, timeout=600)
    found = {k: findings(v) for k, v in kernels(asm.read_text()).items() if "packed_mfma_kernel" in k or "packed_wide_kernel" in k}
    assert len(found) == len(INSTANCES) + len(WIDE)
    for name, (copies, unordered, hazards) in found.items():
        assert copies > 0, name
        assert not unordered, (name, unordered[:3], len(unordered))
        assert not hazards, (name, hazards[:3])
