"""The built code of the 6-bit float GEMM, as the compiler lists it: distances between instructions that it cannot see to itself
because one of them stands in inline assembly.  CPU only (hipcc cross-compiles)."""
import os
import re
import subprocess

import pytest

from paper_2511_22316_amd import build

CSRC = os.path.join(os.path.dirname(build.__file__), "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def listing(source, tmp_path):
    out = str(tmp_path / "listing.s")
    flags = [f for f in build.FLAGS if f not in ("-shared",)]
    subprocess.run([HIPCC, *flags, "-I", os.path.join(CSRC, "..", "..", "include"), "-I", CSRC, "--cuda-device-only", "-S",
                    "-x", "hip", os.path.join(CSRC, source), "-o", out], check=True, capture_output=True)
    with open(out) as f:
        return f.read().splitlines()


def instructions(lines):
    """(text, whether it stands in inline assembly) of every instruction, in order."""
    inside = False
    for line in (l.strip() for l in lines):
        if line.startswith(";;#ASMSTART"):
            inside = True
        elif line.startswith(";;#ASMEND"):
            inside = False
        text = line.split(";")[0].strip()
        if text and not text.startswith((".", "/")) and not text.endswith(":"):
            yield text, inside


def registers(operand):
    m = re.match(r"([va])\[(\d+):(\d+)\]", operand)
    if m:
        return {m[1] + str(k) for k in range(int(m[2]), int(m[3]) + 1)}
    return {operand} if re.match(r"[va]\d+$", operand) else set()


def too_close(lines):
    """Lane swaps and matrix instructions that read what inline assembly wrote less than two wait states before."""
    seen, found, readers = list(instructions(lines)), [], 0
    for k, (text, _) in enumerate(seen):
        name = text.split()[0]
        swap, matrix = "permlane" in name, "mfma" in name
        if not (swap or matrix):
            continue
        readers += 1
        operands = [o.split()[0] for o in text.split(None, 1)[1].split(", ")]
        read = set().union(*[registers(o) for o in (operands if swap else operands[1:])])
        states, b = 0, k - 1
        while states < 2 and b >= 0:
            before, inside = seen[b]
            if before.startswith("s_nop"):
                states += int(before.split()[1], 0)
            elif inside and before.startswith("v_") and "mfma" not in before and registers(before.split(None, 1)[1].split(",")[0]) & read:
                found.append((before, text))
            states, b = states + 1, b - 1
    return found, readers


def loads_behind_m0(lines):
    """Global -> LDS loads directly behind the scalar instruction that sets M0, which they read one wait state later at the earliest."""
    seen = [text for text, _ in instructions(lines)]
    loads = [k for k, text in enumerate(seen) if "_load_lds_" in text]
    return [(seen[k - 1], seen[k]) for k in loads if re.match(r"s_\w+ m0,", seen[k - 1])], len(loads)


def test_scan_sees_a_write_that_is_too_close():
    asm = [";;#ASMSTART", "v_fma_mixhi_f16 v7, v66, v25, 0", ";;#ASMEND"]
    swap = ["v_permlane32_swap_b32_e32 v5, v7"]
    assert too_close(asm + swap)[0] and too_close(asm + ["v_mov_b32_e32 v1, v2"] + swap)[0]
    assert too_close(asm + ["s_nop 0"] + swap)[0]
    assert not too_close(asm + ["s_nop 1"] + swap)[0]
    assert not too_close(asm + ["s_nop 0", "v_mov_b32_e32 v1, v2"] + swap)[0]
    assert too_close(asm + ["v_mfma_f32_32x32x16_f16 a[0:15], v[4:7], v[8:11], a[0:15]"])[0]
    load = "global_load_lds_dwordx4 v1, s[2:3]"
    assert loads_behind_m0(["s_add_u32 m0, m0, 0x1000", ";;#ASMEND", ";;#ASMSTART", load])[0]
    assert not loads_behind_m0(["s_mov_b32 m0, s1", "s_nop 0", load])[0]


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_six_bit_float_kernel_keeps_its_distances(tmp_path):
    lines = listing("sq_w4a4_fp6.hip", tmp_path)
    found, readers = too_close(lines)
    assert readers > 1000, "the kernels are in the listing"
    assert not found, found[:4]
    found, loads = loads_behind_m0(lines)
    assert loads > 100 and not found, found[:4]
