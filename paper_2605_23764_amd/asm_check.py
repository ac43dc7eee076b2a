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


_DS_WRITE = re.compile(r"ds_(write|or|and|xor|add|sub|inc|dec|min|max|cmpst|wrxchg|mskor|append|consume)")


def barrier_violations(asm: str):
    """Returns (number of barriers, list of (kernel, line of the barrier, line of an LDS write or atomic that a wave may pass it
    with)), over every path of the control flow.  A wave's LDS operations complete in order, so a write is complete once
    `s_waitcnt lgkmcnt(n)` has been passed with n or more LDS operations issued behind it."""
    lines = [raw.split(";")[0].strip() for raw in asm.splitlines()]
    kernels = set(re.findall(r"\.amdhsa_kernel\s+(\w+)", asm))
    n_barriers, bad, i = 0, [], 0
    while i < len(lines):
        if not (lines[i].endswith(":") and lines[i][:-1] in kernels):
            i += 1
            continue
        name, first = lines[i][:-1], i + 1
        while not lines[i].startswith((".Lfunc_end", ".amdhsa_kernel")):
            i += 1
        # blocks of instructions (line, text); labels; where each may go on
        blocks, labels, target = [[]], {}, None
        jumps = {}
        for no in range(first, i):
            line = lines[no]
            m = re.match(r"(\.LBB\w+):", line)
            if m:
                blocks.append([])
                labels[m.group(1)] = len(blocks) - 1
            if not line or line.startswith(".") or line.endswith(":"):
                continue
            blocks[-1].append((no + 1, line))
            m = re.search(r"\((\.LBB\w+)-\.Lpost_getpc", line)      # a long branch: the address is added up, then s_setpc_b64
            target = m.group(1) if m else target
            op = line.split()
            if op[0].startswith(("s_cbranch", "s_branch", "s_setpc", "s_endpgm")):
                to = [target] if op[0].startswith("s_setpc") else op[1:2]
                jumps[len(blocks) - 1] = (to, op[0].startswith("s_cbranch"))
                blocks.append([])

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
            to, falls = jumps.get(b, ([], True))
            for s in [labels[t] for t in to] + ([b + 1] if falls and b + 1 < len(blocks) else []):
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


def main():
    n, bad = check_register_fed_loads(device_assembly())
    print(f"{n} assembly loads with register destinations, {len(bad)} instructions inside a request-to-retire window touch them")
    for no, line, regs in bad[:20]:
        print(f"  line {no}: {line}   (v{regs})")
    n_barriers, late = barrier_violations(device_assembly())
    print(f"{n_barriers} barriers, {len(late)} passed with LDS writes under way")
    for kernel, no, write in late[:20]:
        print(f"  {kernel}: barrier in line {no}, write in line {write}")
    sys.exit(1 if bad or late or n == 0 else 0)


if __name__ == "__main__":
    main()
