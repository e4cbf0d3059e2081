"""Reciprocals that stand in for divisions of token indices by group and page sizes: against the division, on the CPU."""
import os
import subprocess

import pytest

from paper_2505_18231_amd import build

PROGRAM = r"""
#include "nsn_host.h"
#include <cstdio>
int main() {
  long bad = 0;
  uint64_t state = 1;
  auto rnd = [&](uint32_t n) { state = state * 6364136223846793005ull + 1442695040888963407ull; return (uint32_t)((state >> 33) % n); };
  const int64_t most = ((int64_t)1 << 31) - 64;  // the largest multiple of 64
  auto check = [&](int64_t tokens) {
    const nsn::Geometry::Div v = nsn::tokens_divisor((int)tokens);
    auto at = [&](int64_t t) { if (t >= 0 && t <= most && nsn::tokens_div((int)t, v) != (int)(t / tokens)) ++bad; };
    for (int64_t m : {(int64_t)0, (int64_t)1, (int64_t)2, most / tokens / 2, most / tokens}) at(m * tokens), at(m * tokens - 64), at(m * tokens + 64);
    at(most);
    for (int i = 0; i < 50; ++i) at(64 * (int64_t)rnd(1u << 25));
  };
  for (int64_t d = 1; d <= 5000; ++d) check(64 * d);
  for (int k = 0; k < 25; ++k)
    for (int64_t d : {((int64_t)1 << k) - 1, (int64_t)1 << k, ((int64_t)1 << k) + 1}) if (d > 0 && 64 * d <= most) check(64 * d);
  for (int i = 0; i < 20000; ++i) check(64 * (1 + (int64_t)rnd((1u << 25) - 1)));
  const nsn::Geometry::Div none = {0u, 0};  // no groups
  for (int i = 0; i < 1000; ++i) if (nsn::tokens_div(64 * (int)rnd(1u << 25), none) != 0) ++bad;
  printf("%ld\n", bad);
}
"""


def test_reciprocals_divide_every_multiple_of_64(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    source, program = tmp_path / "div.cpp", tmp_path / "div"
    source.write_text(PROGRAM)
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-I", build.CSRC, str(source), "-o", str(program)],
                   check=True, capture_output=True)
    assert subprocess.run([str(program)], check=True, capture_output=True, text=True).stdout.strip() == "0"
