"""Static check of a contract the compiler cannot see (csrc/gemm_bf16.h, register-fed row block of the wide tile).

The block's activation fragments are fetched by plain global loads written as inline assembly, so that they ride the
pipeline's hand-kept `s_waitcnt vmcnt` accounting.  Their destination registers are written by the hardware some time
after the statement, behind the compiler's back: from the request to the wait that retires them (another assembly
statement, `s_waitcnt vmcnt(n)`, which names the registers) no instruction may read or write those registers.  The
source is arranged so that the compiler has no reason to (the window lies inside one loop trip and ends in the naming
wait), but nothing in the language enforces it; this module checks the generated code.

A second contract: no wave passes a barrier with LDS writes of its own under way (barrier_violations).  The language has it
for __syncthreads, but the compiler has been seen to lose the wait of a barrier at the head of a loop where the writes are
outstanding only along the way back: waves then read tables that others were still filling.  Barriers placed by hand
(__builtin_amdgcn_s_barrier) never had one.  Reads may be under way at those: the GEMM pipelines do so by design.

A third: a condition that is the same for the whole wave, tested inside a loop that lanes leave one by one and again behind it, is not
carried out of the loop as a lane mask (stale_lane_masks).  The compiler did that to the copy of two rows at a time: lanes that had
left the loop a pass earlier stored the tail of a second row where there was none.

    python -m paper_2605_23764_amd.asm_check        # compiles the device code to assembly and checks it
"""
from __future__ import annotations

import functools
import os
import re
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))

_RANGE = re.compile(r"\bv\[(\d+):(\d+)\]")
_SINGLE = re.compile(r"\bv(\d+)\b")


def _vregs(text: str) -> set:
    regs = set()
    for lo, hi in _RANGE.findall(text):
        regs.update(range(int(lo), int(hi) + 1))
    regs.update(int(r) for r in _SINGLE.findall(_RANGE.sub(" ", text)))
    return regs


@functools.lru_cache(maxsize=None)
def device_assembly() -> str:
    """Device-only assembly of csrc/moe_ffn.hip with the library's own flags."""
    from .build import HIPCC_FLAGS, SOURCES
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = [f for f in HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "device.s")
        res = subprocess.run([hipcc, *flags, "--cuda-device-only", "-S", *SOURCES, "-o", out], capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)
        with open(out) as f:
            return f.read()


def check_register_fed_loads(asm: str):
    """Returns (number of assembly loads with register destinations, list of violations).  A violation is
    (line number, instruction, registers) for an instruction between such a load and the next assembly
    `s_waitcnt vmcnt` that touches the load's destination registers."""
    pending = {}          # register -> line of the load that will write it
    n_loads, bad = 0, []
    in_asm = False
    for no, raw in enumerate(asm.splitlines(), 1):
        line = raw.split(";")[0].strip() if not raw.lstrip().startswith(";;#") else raw.strip()
        if line.startswith(";;#ASMSTART"):
            in_asm = True
            continue
        if line.startswith(";;#ASMEND"):
            in_asm = False
            continue
        if not line or line.startswith(".") or line.endswith(":"):
            if line.startswith(".end_amdhsa_kernel") or line.startswith(".amdhsa_kernel"):
                pending.clear()
            continue
        if in_asm:
            m = re.match(r"global_load_dwordx4\s+v\[(\d+):(\d+)\]\s*,\s*(.*)", line)
            if m:
                n_loads += 1
                touched = _vregs(m.group(3)) & set(pending)
                if touched:
                    bad.append((no, line, sorted(touched)))
                for r in range(int(m.group(1)), int(m.group(2)) + 1):
                    pending[r] = no
                continue
            if line.startswith("s_waitcnt") and "vmcnt" in line:
                pending.clear()       # the naming wait: everything requested before it is retired
                continue
        if pending:
            touched = _vregs(line) & set(pending)
            if touched:
                bad.append((no, line, sorted(touched)))
    return n_loads, bad


def loads_ahead_of_first_branch(asm: str, kernel: str):
    """Scalar loads (base, offset) of the kernel ahead of its first branch, in the groups that one wait covers."""
    start = asm.index(f"\n{kernel}:")
    groups = [[]]
    for raw in asm[start + 1:].splitlines()[1:]:
        line = raw.split(";")[0].strip()
        if line.startswith("s_cbranch") or line.startswith("s_branch"):
            break
        m = re.match(r"s_load_dword\w*\s+[^,]+,\s*(s\[\d+:\d+\])\s*,\s*(\w+)", line)
        if m:
            groups[-1].append((m.group(1), int(m.group(2), 0)))
        elif line.startswith("s_waitcnt") and "lgkmcnt" in line:
            groups.append([])
    return groups


def innermost_loops(asm: str, kernel: str):
    """Instructions of each of the kernel's loops that contains no other loop."""
    start = asm.index(f"\n{kernel}:")
    lines = [raw.split(";")[0].strip() for raw in asm[start:asm.index(".Lfunc_end", start)].splitlines()]
    labels, loops = {}, []
    for i, line in enumerate(lines):
        m = re.match(r"(\.LBB\w+):", line)
        if m:
            labels[m.group(1)] = i
        m = re.match(r"s_c?branch\w*\s+(\.LBB\w+)", line)
        if m and m.group(1) in labels:
            loops.append((labels[m.group(1)], i))
    inner = [(a, b) for a, b in loops if not any((a, b) != (c, d) and a <= c and d <= b for c, d in loops)]
    return [[line for line in lines[a:b + 1] if line and not line.startswith(".")] for a, b in inner]


def _control_flow(asm: str):
    """Per kernel: its name, blocks of instructions [(line, text)], and the blocks that may follow each."""
    lines = [raw.split(";")[0].strip() for raw in asm.splitlines()]
    kernels = set(re.findall(r"\.amdhsa_kernel\s+(\w+)", asm))
    i = 0
    while i < len(lines):
        if not (lines[i].endswith(":") and lines[i][:-1] in kernels):
            i += 1
            continue
        name, first = lines[i][:-1], i + 1
        while not lines[i].startswith((".Lfunc_end", ".amdhsa_kernel")):
            i += 1
        blocks, labels, jumps, target = [[]], {}, {}, None
        for no in range(first, i):
            line = lines[no]
            m = re.match(r"(\.LBB\w+):", line)
            if m:
                if blocks[-1]:
                    blocks.append([])
                labels[m.group(1)] = len(blocks) - 1
            if not line or line.startswith(".") or line.endswith(":"):
                continue
            blocks[-1].append((no + 1, line))
            m = re.search(r"\((\.LBB\w+)-\.Lpost_getpc", line)      # a long branch: the address is added up, then s_setpc_b64
            target = m.group(1) if m else target
            op = line.split()
            if op[0].startswith(("s_cbranch", "s_branch", "s_setpc", "s_endpgm")):
                jumps[len(blocks) - 1] = ([target] if op[0].startswith("s_setpc") else op[1:2], op[0].startswith("s_cbranch"))
                blocks.append([])
        follow = []
        for n in range(len(blocks)):
            to, falls = jumps.get(n, ([], True))
            follow.append([labels[t] for t in to] + ([n + 1] if falls and n + 1 < len(blocks) else []))
        yield name, blocks, follow


_DS_WRITE = re.compile(r"ds_(write|or|and|xor|add|sub|inc|dec|min|max|cmpst|wrxchg|mskor|append|consume)")


def barrier_violations(asm: str):
    """Returns (number of barriers, list of (kernel, line of the barrier, line of an LDS write or atomic that a wave may pass it
    with)), over every path of the control flow.  A wave's LDS operations complete in order, so a write is complete once
    `s_waitcnt lgkmcnt(n)` has been passed with n or more LDS operations issued behind it."""
    n_barriers, bad = 0, []
    for name, blocks, follow in _control_flow(asm):

        def flow(b, behind, report=None):
            # behind: None, nothing under way; else (LDS operations issued behind the youngest such write, its line)
            for no, line in blocks[b]:
                if _DS_WRITE.match(line):
                    behind = (0, no)
                elif line.startswith("ds_") and behind:
                    behind = (behind[0] + 1, behind[1])
                elif line.startswith("s_waitcnt"):
                    m = re.search(r"lgkmcnt\((\d+)\)", line)
                    if m and behind and behind[0] >= int(m.group(1)):
                        behind = None
                elif line.startswith("s_barrier") and report is not None:
                    report.append((no, behind))
            return behind

        entry, seen, work = {0: None}, {0}, [0]
        while work:
            b = work.pop()
            out = flow(b, entry[b])
            for s in follow[b]:
                old = entry.get(s)
                new = out if old is None or (out is not None and out[0] < old[0]) else old
                if s not in seen or new != old:
                    seen.add(s)
                    entry[s] = new
                    work.append(s)
        for b in sorted(seen):
            found = []
            flow(b, entry[b], found)
            n_barriers += len(found)
            bad += [(name, no, behind[1]) for no, behind in found if behind]
    return n_barriers, bad


def _sgprs(token: str) -> set:
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", token)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.fullmatch(r"s(\d+)", token)
    return {int(m.group(1))} if m else set()


def stale_lane_masks(asm: str):
    """Branches behind a loop that lanes leave one by one, decided for the whole wave by a lane mask of a compare inside the loop: the mask
    has zeros for the lanes that were no longer in it.  Returns (number of such loops, list of (kernel, line of the use, line of the
    compare))."""
    n_loops, bad = 0, []
    for name, blocks, follow in _control_flow(asm):
        before = [[] for _ in blocks]
        for b, f in enumerate(follow):
            for s in f:
                before[s].append(b)
        for latch, block in enumerate(blocks):
            if not any(line.startswith("s_andn2_b64 exec, exec") for _, line in block):
                continue
            # the smallest loop that this block closes
            body = None
            for head in follow[latch]:
                loop, work = {head, latch}, [latch]
                while work:
                    b = work.pop()
                    if b != head:
                        new = [q for q in before[b] if q not in loop]
                        loop.update(new)
                        work += new
                if (0 not in loop or head == 0) and (body is None or len(loop) < len(body)):
                    body = loop
            if body is None:
                continue
            n_loops += 1
            masks, other = {}, set()
            for b in body:
                for no, line in blocks[b]:
                    op = line.replace(",", " ").split()
                    if len(op) < 2:
                        continue
                    if op[0].startswith("v_cmp") and op[1].startswith("s["):
                        masks[op[1]] = no
                    else:
                        other |= _sgprs(op[1]) if not op[0].startswith("s_c") else set()
            masks = {m: no for m, no in masks.items() if not _sgprs(m) & other}
            # from the loop's ends on, until the mask is written again
            seen = set()
            work = [(s, frozenset(masks)) for b in body for s in follow[b] if s not in body] if masks else []
            while work:
                b, live = work.pop()
                if b in body or (b, live) in seen:
                    continue
                seen.add((b, live))
                for i, (no, line) in enumerate(blocks[b]):
                    op = line.replace(",", " ").split()
                    if op[0] in ("s_and_b64", "s_andn2_b64") and op[1] == "vcc" and "exec" in op[2:4]:
                        if any(o[1].startswith("s_cbranch_vcc") for o in blocks[b][i + 1:]):
                            bad += [(name, no, masks[m]) for m in op[2:4] if m in live]
                    if len(op) > 1 and not op[0].startswith("s_cmp"):
                        live = frozenset(m for m in live if not _sgprs(m) & _sgprs(op[1]))
                if live:
                    work += [(s, live) for s in follow[b]]
    return n_loops, sorted(set(bad))


def main():
    n, bad = check_register_fed_loads(device_assembly())
    print(f"{n} assembly loads with register destinations, {len(bad)} instructions inside a request-to-retire window touch them")
    for no, line, regs in bad[:20]:
        print(f"  line {no}: {line}   (v{regs})")
    n_barriers, late = barrier_violations(device_assembly())
    print(f"{n_barriers} barriers, {len(late)} passed with LDS writes under way")
    for kernel, no, write in late[:20]:
        print(f"  {kernel}: barrier in line {no}, write in line {write}")
    n_loops, stale = stale_lane_masks(device_assembly())
    print(f"{n_loops} loops that lanes leave one by one, {len(stale)} uses of their lane masks for the whole wave behind them")
    for kernel, no, compare in stale[:20]:
        print(f"  {kernel}: use in line {no}, compare in line {compare}")
    sys.exit(1 if bad or late or stale or n == 0 else 0)


if __name__ == "__main__":
    main()
