"""CPU test of the built device code: no register copy or reload sits under a mask that is not its
own.  Where an inner `if` ends with the outer one, the compiler narrows the mask without saving it
(s_and_b64 exec, exec, ...) and restores both at once (s_or_b64 exec, ...).  A copy that the
register allocator places between the inner block and that restore runs for the inner block's
lanes only, though every lane needs it: the PCG loop once lost entries of S that way.  Such a copy
is told from the block's own by what reads it: nothing in the block does."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2309_08079_amd", "libmpcpcg.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"

NARROW = re.compile(r"s_and_b64 exec, exec, ")
ENDS = re.compile(r"(s_or_b64|s_mov_b64|s_and_b64|s_andn2_b64|s_xor_b64) exec|s_\w*saveexec|s_endpgm|s_branch|s_setpc")
COPY = re.compile(r"(v_mov_b32\S*|v_mov_b64\S*|v_accvgpr_read\S*) (\S+), [va][\[\d]|(scratch_load_\S+) (\S+),")


def registers(text):
    out = set()
    for a, b, c in re.findall(r"\bv(?:\[(\d+):(\d+)\]|(\d+))", text):
        out |= set(range(int(a), int(b) + 1)) if a else {int(c)}
    return out


def stray_copies(code):
    """(kernel, instruction) of copies under a narrowed mask that nothing under it reads"""
    found, kernel, n = [], "", len(code)
    for i, line in enumerate(code):
        m = re.match(r"(?:[0-9a-f]+ <)?(_Z\w+)>?:", line)
        if m:
            kernel = m.group(1)
        if not NARROW.match(line):
            continue
        end = i + 1
        while end < n and not ENDS.match(code[end]):
            end += 1
        if end == n or not code[end].startswith("s_or_b64 exec"):
            continue  # (another block begins inside)
        body = code[i + 1:end]
        for k, ins in enumerate(body):
            m = COPY.match(ins)
            if not m:
                continue
            dst = registers(m.group(2) or m.group(4))
            reads = set()
            for later in body[k + 1:]:
                ops = later.split(" ", 1)[1] if " " in later else ""
                first, _, rest = ops.partition(",")
                stores = re.match(r"(ds_write|ds_add|global_store|buffer_store|scratch_store|flat_store|v_cmp|global_atomic)", later)
                reads |= registers(ops if stores or "fmac" in later else rest)
            if not dst & reads:
                found.append((kernel, ins))
    return found


def lines(text):
    return [s for s in (l.split("//")[0].split(";")[0].strip() for l in text.splitlines()) if s]


def test_the_pattern_is_recognised():
    bad = """
        s_and_saveexec_b64 s[30:31], s[10:11]
        ds_write_b32 v56, v0
        s_or_b64 exec, exec, s[30:31]
        s_and_b64 exec, exec, s[12:13]
        ds_write_b32 v56, v0 offset:1088
        s_setprio 0
        v_mov_b64_e32 v[72:73], v[90:91]
        s_or_b64 exec, exec, s[28:29]
    """
    good = bad.replace("        s_setprio 0\n        v_mov_b64_e32 v[72:73], v[90:91]\n", "").replace(
        "ds_write_b32 v56, v0 offset:1088", "v_mov_b32_e32 v1, v0\n        ds_write_b32 v56, v1 offset:1088")
    assert stray_copies(lines(bad)) == [("", "v_mov_b64_e32 v[72:73], v[90:91]")]
    assert stray_copies(lines(good)) == []


@pytest.mark.skipif(not os.path.exists(LIB), reason="libmpcpcg.so not built")
@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="llvm-objdump not available")
def test_no_copy_under_another_blocks_mask(tmp_path):
    lib = str(tmp_path / "lib.so")
    shutil.copy(LIB, lib)  # (the code objects are written beside it)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True)
    objs = [f for f in os.listdir(tmp_path) if "gfx950" in f]
    assert objs
    kernels = 0
    for f in objs:
        code = lines(subprocess.run([OBJDUMP, "-d", str(tmp_path / f)], check=True, capture_output=True, text=True).stdout)
        kernels += sum("pcg_kernel" in l and l.endswith(">:") for l in code)
        assert stray_copies(code) == []
    assert kernels > 20
