"""Token sums of the decode kernels near the largest cache (2^31 - 64 tokens), worked out with their own functions on the CPU.

Groups are asked for ahead of their use, past the end of a sequence too; as signed sums their first tokens wrap, and a clamp
by the smaller one then takes the wrapped one: a Shift vector 4 GiB away.  The end of a sequence's last split, counted from its start by
the splits' length, may lie beyond 2^31; wrapped, the split has no tokens."""
import os
import subprocess

import pytest

from paper_2505_18231_amd import build

AHEAD = r"""
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
SPLITS = r"""
#include "nsn_host.h"
#include <cstdio>
int main() {
  long bad = 0;
  for (int len : {0, 1, 64, 65, 4096, 100000, (1 << 25) + 1, 2147483584 - 4096, 2147483584 - 17, 2147483584})
    for (int n = 1; n <= 64; ++n) {
      const int per = (((len + n - 1) / n) + 63) & ~63;
      int64_t tokens = 0;
      for (int s = 0; s < n; ++s) {
        const int t0 = s * per, t1 = nsn::split_end(t0, per, len);
        const int64_t want = (int64_t)t0 + per < len ? (int64_t)t0 + per : len;
        if (t1 != want) ++bad;
        tokens += t1 > t0 ? t1 - t0 : 0;
      }
      if (tokens != len) ++bad;
    }
  printf("%ld\n", bad);
}
"""


@pytest.mark.parametrize("program", [AHEAD, SPLITS], ids=["groups past the end", "ends of splits"])
def test_tokens_near_the_largest_cache(tmp_path, program):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    source, binary = tmp_path / "tokens.cpp", tmp_path / "tokens"
    source.write_text(program)
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-I", build.CSRC, str(source), "-o", str(binary)],
                   check=True, capture_output=True)
    assert subprocess.run([str(binary)], check=True, capture_output=True, text=True).stdout.strip() == "0"
