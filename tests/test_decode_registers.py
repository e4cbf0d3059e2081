"""What the compiler makes of the decode kernel's loops, read from its listing (nothing runs): registers that spill to
memory, and waits that drain the loads which a loop asks for ahead of their use."""
import os
import re
import subprocess

import pytest

from paper_2505_18231_amd import build

# sub_dim, waves, powers of two, paged, persistent, 4-bit side information, sign + index, rotary
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
