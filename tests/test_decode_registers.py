"""What the compiler makes of the decode kernel's loops, read from its listing (nothing runs): registers that spill to
memory, and waits that drain the loads which a loop asks for ahead of their use."""
import os
import re
import subprocess

import pytest

from paper_2505_18231_amd import build

# sub_dim, waves, powers of two, paged, persistent, 4-bit side information, sign + index, rotary
ONE_SPLIT = ["8,8,true,false,false,false", "4,8,true,false,false,false", "4,8,false,false,false,true"]
SIGN_4BIT = ["8,8,false,false,false,true,true,false", "8,8,false,true,false,true,true,false"]


def _listing(instances, where):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    source, out = where / "instances.hip", where / "instances.s"
    kernels = "".join(f"(const void*)dec_tile_kernel<{i}>, " for i in instances)
    source.write_text(f'#include "nsn_decode_tile.h"\nnamespace nsn {{ namespace tile {{ const void* all[] = {{{kernels}}}; }} }}\n')
    flags = [f for f in build.HIPCC_FLAGS if f != "-shared"]
    subprocess.run([hipcc, *flags, "--cuda-device-only", "-S", "-I", os.path.join(build.HERE, "..", "include"),
                    "-I", build.CSRC, str(source), "-o", str(out)], check=True, capture_output=True)
    return out.read_text()


def test_sign_codes_with_4bit_side_information_spill_no_vector_registers(tmp_path):
    text = _listing(SIGN_4BIT, tmp_path)
    spilled = [int(n) for n in re.findall(r"\.vgpr_spill_count:\s+(\d+)", text)]
    assert spilled == [0] * len(SIGN_4BIT), spilled


def test_rotary_instances_spill_what_their_comment_says(tmp_path):
    """(The other 26 instances of the legacy layout spill none: too many to build here.)"""
    paged = ["8,8,false,true,true,true,true,true", "4,8,false,true,true,true,false,true", "8,8,false,true,true,false,true,true"]
    text = _listing(paged + ["8,8,false,false,true,true,true,true", "8,8,false,false,false,true,true,true"], tmp_path)
    spilled = [int(n) for n in re.findall(r"\.vgpr_spill_count:\s+(\d+)", text)]
    assert len(spilled) == 5 and sorted(spilled)[:2] == [0, 0] and max(spilled) <= 9, spilled


def _loop_loads(kernel):
    """Targets of the main loop's loads of four bytes and less (Shift vectors, read only where the Shift group changes, and 4-bit
    side information) with the number of vector and LDS instructions of the loop that write the same register."""
    code = [line.split(";")[0].strip() for line in kernel]
    code = [line for line in code if line]
    first = next(i for i, line in enumerate(code) if line.startswith("v_mfma_f32_16x16x32"))
    last = max(i for i, line in enumerate(code) if line.startswith("v_mfma_f32_4x4x4"))
    targets = {line.split()[1].rstrip(",") for line in code[first:last] if re.match(r"(global|buffer)_load_(dword|ushort|ubyte) ", line)}
    writes = dict.fromkeys(targets, 0)
    for line in code[first:last]:
        if line.startswith(("v_", "ds_read")):
            args = [a.strip() for a in line.split(None, 1)[1].split(",")]
            for reg in args[:2] if "swap" in line else args[:1]:
                if reg in writes:
                    writes[reg] += 1
    return writes


def test_load_targets_of_the_main_loop_hold_nothing_else(tmp_path):
    """A load's target that is a temporary too makes the loop wait for that load, and with it for every load asked for ahead.
    (Ten writes: the code where the Shift group changes takes the value from its register and may reuse it there.)"""
    kernels = re.split(r"^_Z\S*dec_tile_kernel\S*:", _listing(ONE_SPLIT, tmp_path), flags=re.M)[1:]
    assert len(kernels) == len(ONE_SPLIT)
    for kernel in kernels:
        writes = _loop_loads(kernel.split(".Lfunc_end")[0].splitlines())
        assert len(writes) >= 6 and max(writes.values()) <= 10, writes


def test_up_to_four_query_heads_pay_nothing_for_two_units(tmp_path):
    """The arithmetic of two units per kv head (five to eight query heads) is in the instances of such calls only."""
    flags = "8,true,true,true,false,false,false"
    for sub in (4, 8):
        kernels = re.split(r"^_Z\S*dec_tile_kernel\S*:", _listing([f"{sub},{flags},false", f"{sub},{flags},true"], tmp_path),
                           flags=re.M)[1:]
        few, many = (len(re.findall(r"^\s+s_(?!nop|waitcnt|barrier|branch)", k.split(".Lfunc_end")[0], flags=re.M)) for k in kernels)
        assert few < many, (few, many)


def test_the_codebook_row_is_requested_ahead_of_the_other_loads(tmp_path):
    """The table fill waits for the codebook row, so its load goes out first, and not just in front of the bulk loads that
    fill the memory pipeline (one workgroup per split)."""
    for kernel in re.split(r"^_Z\S*dec_tile_kernel\S*:", _listing(ONE_SPLIT[:2], tmp_path), flags=re.M)[1:]:
        code = [line.split(";")[0].strip() for line in kernel.splitlines()]
        code = [line for line in code if line and not line.startswith(".")]
        first, second = [i for i, line in enumerate(code) if line.startswith(("global_load", "buffer_load"))][:2]
        assert second - first >= 20, (first, second)


def test_the_arguments_come_in_one_trip(tmp_path):
    """Scalar loads are waited for all together, and no cache holds the arguments at the start of a launch: every 64-byte line of
    them that is read ahead of the first vector load is asked for ahead of the first wait (one workgroup per split)."""
    for kernel in re.split(r"^_Z\S*dec_tile_kernel\S*:", _listing(ONE_SPLIT, tmp_path), flags=re.M)[1:]:
        code = [line.split(";")[0].strip() for line in kernel.splitlines()]
        vector = next(i for i, line in enumerate(code) if line.startswith(("global_load", "buffer_load")))
        wait = next(i for i, line in enumerate(code) if line.startswith("s_waitcnt"))
        lines = {True: set(), False: set()}  # asked for ahead of the wait, behind it
        for i, line in enumerate(code[:vector]):
            m = re.match(r"s_load_dword(?:x(\d+))? \S+ s\[0:1\], (\w+)", line)
            if m:
                at, n = int(m.group(2), 0), 4 * int(m.group(1) or 1)
                lines[i < wait] |= {at // 64, (at + n - 1) // 64}
        assert lines[True] >= {0, 1, 2} | lines[False], lines
