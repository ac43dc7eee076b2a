"""Order of the copies into the LDS in the grouped bf16 GEMM kernel, on the CPU: csrc/gemm_bf16.h itself is compiled for the
host with its assembly statements recorded instead of executed (tests/lds_copy_order.cpp), the kernel's loop over its work
items is run for the four waves of a workgroup, and no two waves may write the same 1 KB of LDS, or a wave's epilogue region,
without a wait and a barrier between them.  Tiles of every shape follow each other in one workgroup: wide (two wave rows),
wide with the register-fed row block, tall, and the halved last round."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2605_23764_amd", "csrc")
CLANG = next((c for c in ("/opt/rocm/llvm/bin/clang++", shutil.which("clang++")) if c and os.path.exists(c)), None)

NN, NT, STORE, SWIGLU, SWIGLU_GRAD = 0, 1, 0, 1, 2


def _balanced(src, start):
    """Index behind the parenthesis that closes the one at src[start]."""
    depth, i, quoted = 0, start, False
    while True:
        c = src[i]
        if c == '"' and src[i - 1] != "\\":
            quoted = not quoted
        elif not quoted:
            depth += (c == "(") - (c == ")")
            if depth == 0:
                return i + 1
        i += 1


def _split(text, sep):
    """text at `sep`, outside of quotes and parentheses."""
    parts, depth, quoted, cur = [], 0, False, ""
    for i, c in enumerate(text):
        if c == '"' and text[i - 1] != "\\":
            quoted = not quoted
        if not quoted:
            depth += (c in "([") - (c in ")]")
        if c == sep and depth == 0 and not quoted:
            parts.append(cur)
            cur = ""
        else:
            cur += c
    return parts + [cur]


def recorded(src):
    """The source with `asm volatile(text : outputs : inputs : clobbers)` as `sim_asm(text, inputs...)`."""
    out, at = "", 0
    for m in re.finditer(r"asm volatile\s*\(", src):
        end = _balanced(src, m.end() - 1)
        text, _, ins = (_split(src[m.end():end - 1], ":") + ["", ""])[:3]
        args = [a[a.index("(") + 1:a.rindex(")")] for a in _split(ins, ",") if a.strip()]
        out += src[at:m.start()] + "sim_asm(" + ", ".join([text.strip()] + args) + ")"
        at = end
    return out + src[at:]


def test_assembly_statements_become_calls():
    src = 'f(); asm volatile("a %0, %1" "\\n\\tb" : "=v"(d) : "v"(x[i]), "n"(KS * 32) : "memory"); asm volatile("" : "+v"(l)); asm volatile("s_nop 1" ::: "memory");'
    assert recorded(src) == 'f(); sim_asm("a %0, %1" "\\n\\tb", x[i], KS * 32); sim_asm(""); sim_asm("s_nop 1");'


@pytest.fixture(scope="module")
def sim(tmp_path_factory):
    if CLANG is None:
        pytest.skip("needs clang++")
    d = tmp_path_factory.mktemp("lds_order")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text("#pragma once\n")
    for name in ("common.h", "gemm_bf16.h", "stream_rule.h"):
        with open(os.path.join(CSRC, name)) as f:
            (d / name).write_text(recorded(f.read()))
    exe = str(d / "lds_copy_order")
    res = subprocess.run([CLANG, "-x", "c++", "-std=c++17", "-O1", "-w", "-I", str(d), os.path.join(HERE, "lds_copy_order.cpp"), "-o", exe],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]

    def run(lay, epi, steps, keep_h1, workers, rows):
        res = subprocess.run([exe, *map(str, (lay, epi, 64 * steps, keep_h1, workers, *rows))], capture_output=True, text=True, timeout=60)
        assert res.returncode == 0, res.stdout + res.stderr
        return res.stdout

    return run


# rows of four M tiles of one XCD (two pair slots); a tall tile has a slot of its own
ROWS = [(256, 225, 384, 0), (384, 0, 256, 200), (320, 300, 330, 0), (330, 0, 289, 0), (384, 0, 336, 0), (130, 70, 350, 0), (256, 250, 256, 0)]


@pytest.mark.parametrize("steps", [1, 2, 3, 4, 5, 6, 7, 8, 22])
@pytest.mark.parametrize("lay,epi", [(NN, SWIGLU), (NN, STORE), (NT, SWIGLU_GRAD), (NT, STORE)])
def test_no_two_waves_meet_in_the_lds(sim, lay, epi, steps):
    for rows in ROWS:
        for workers in (1, 2, 3, 5):      # one workgroup takes all items in turn; others end on a halved round
            out = sim(lay, epi, steps, workers & 1, workers, rows)
            assert [line for line in out.splitlines() if line.startswith("races")] == ["races 0"] * workers, (rows, workers, out)
