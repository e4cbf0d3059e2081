"""Groups are asked for ahead of their use, past the end of a sequence too: their first tokens near the largest cache (2^31 - 64
tokens), worked out with the decode kernel's own functions on the CPU.  As signed sums they wrap, and a clamp by the smaller one
then takes the wrapped one: a Shift vector 4 GiB in front of the first."""
import os
import subprocess

import pytest

from paper_2505_18231_amd import build

PROGRAM = r"""
#include "nsn_host.h"
#include <cstdio>
int main() {
  long bad = 0;
  const int64_t most = ((int64_t)1 << 31) - 64, far = 24 + 7;  // three groups ahead of eight waves, the last wave
  for (int64_t end : {most, most - 64, most - 31 * 64, most - 4096, (int64_t)1 << 30, (int64_t)64})
    for (int64_t t0 : {(int64_t)0, end / 128 * 64, end > 2048 ? end - 2048 : 0, end - 64}) {
      const int64_t groups = (end - t0) / 64;
      for (int64_t n = groups > 40 ? groups - 40 : 0; n <= groups + far; ++n) {
        const int64_t want = t0 + 64 * n, last = end - 64;
        const uint32_t at = nsn::token_of_group((int)t0, (int)n);
        if ((int64_t)at != want) ++bad;
        if (nsn::token_up_to(at, (int)last) != (want < last ? want : last)) ++bad;
      }
    }
  printf("%ld\n", bad);
}
"""


def test_groups_past_the_end_of_the_largest_cache(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    source, program = tmp_path / "ahead.cpp", tmp_path / "ahead"
    source.write_text(PROGRAM)
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-I", build.CSRC, str(source), "-o", str(program)],
                   check=True, capture_output=True)
    assert subprocess.run([str(program)], check=True, capture_output=True, text=True).stdout.strip() == "0"
