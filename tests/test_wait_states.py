"""Idle cycles between lane swaps written in asm and the matrix instructions that read their results: a matrix instruction
reads a vector register two cycles after a vector instruction wrote it at the earliest.  The compiler sees to that for its own
instructions and not for asm, so the listing of the search's kernels is read here (nothing runs)."""
import os
import re
import subprocess

import pytest

from paper_2505_18231_amd import build

REG = re.compile(r"\bv(\d+)\b|\bv\[(\d+):(\d+)\]")


def _registers(text):
    out = set()
    for one, lo, hi in REG.findall(text):
        out |= {int(one)} if one else set(range(int(lo), int(hi) + 1))
    return out


def _short_waits(listing):
    """(instruction, register, idle cycles) of every matrix instruction that comes too early, instruction by instruction."""
    found, swapped, now, in_asm = [], {}, 0, False
    for line in listing:
        in_asm = (in_asm or "#ASMSTART" in line) and "#ASMEND" not in line
        text = line.split(";")[0].strip()
        if line.startswith("_Z"):
            swapped = {}
        if not text or text.startswith(".") or text.endswith(":"):
            continue
        op, _, args = text.partition(" ")
        if op.startswith("v_mfma"):
            dst, _, src = args.partition(",")
            found += [(text, r, now - swapped[r] - 1) for r in _registers(src) if r in swapped and now - swapped[r] < 3]
            for r in _registers(dst):
                swapped.pop(r, None)
        elif op.startswith(("v_", "ds_read", "global_load", "scratch_load")):
            written = _registers(args if "permlane" in op else args.split(",")[0])
            for r in written:
                swapped.pop(r, None)
                if in_asm:
                    swapped[r] = now
        now += int(args) + 1 if op == "s_nop" else 1
    return found


def test_the_reader_of_listings_sees_a_short_wait():
    code = "_Zk:\n;;#ASMSTART\nv_permlane32_swap_b32 v1, v9\n;;#ASMEND\n{}v_mfma_f32_32x32x16_f16 v[16:31], v[4:7], v[0:3], 0\n"
    assert [w[1:] for w in _short_waits(code.format("").splitlines())] == [(1, 0)]
    assert [w[1:] for w in _short_waits(code.format("s_nop 0\n").splitlines())] == [(1, 1)]
    assert _short_waits(code.format("s_nop 1\n").splitlines()) == []


@pytest.mark.parametrize("source", ["nsn_codebook.hip", "nsn_encode.hip"])
def test_matrix_instructions_wait_for_swapped_operands(source, tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    out = tmp_path / "kernels.s"
    flags = [f for f in build.HIPCC_FLAGS if f != "-shared"]
    subprocess.run([hipcc, *flags, "--cuda-device-only", "-S", "-I", os.path.join(build.HERE, "..", "include"),
                    os.path.join(build.CSRC, source), "-o", str(out)], check=True, capture_output=True)
    listing = out.read_text().splitlines()
    assert sum("v_permlane32_swap_b32" in l for l in listing) > 100 and sum("v_mfma" in l for l in listing) > 100
    found = _short_waits(listing)
    assert not found, f"{len(found)} matrix instructions read a swapped register too early, e.g. {found[:3]}"
