"""Launches stay below the 2^32 threads that HIP counts (csrc/launch_limit.h): a larger one would
run only the rest of the division by 2^32, without an error.  Host code only."""

import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2106_12736_amd", "csrc")

SOURCE = r"""
#include "launch_limit.h"
#undef NDEBUG
#include <cassert>

int main() {
  static_assert(fdc::launch_counts(4194303, 1024) && !fdc::launch_counts(4194304, 1024), "");
  static_assert(!fdc::launch_counts(5000000, 1024) && fdc::launch_counts(16777215, 256), "");
  const long long totals[] = {1, 4194303, 4194304, 5000000, 2 * 4194303LL, 2 * 4194303LL + 1, 16777216, (1LL << 32) - 1};
  for (int threads : {64, 256, 1024})
    for (long long total : totals) {
      long long next = 0;  // every workgroup once, in order
      const int err = fdc::in_launches(total, threads, 0, [&](std::uint32_t n, std::uint32_t first) {
        assert(n > 0 && first == next && fdc::launch_counts(n, threads));
        next += n;
        return 0;
      });
      assert(err == 0 && next == total);
    }
  int calls = 0;  // an error ends it
  assert(fdc::in_launches(3 * 4194303LL, 1024, 0, [&](std::uint32_t, std::uint32_t) { return ++calls == 2 ? 7 : 0; }) == 7);
  assert(calls == 2);
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ is needed")
def test_launches_fit_the_thread_count(tmp_path):
    src, exe = tmp_path / "launches.cpp", tmp_path / "launches"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True, timeout=120)
    subprocess.run([str(exe)], check=True, timeout=60)


def test_large_grids_go_through_the_limit():
    """Every kernel is launched by the one function that refuses an uncounted launch, and Full FDC's,
    whose grids can pass the limit at accepted sizes, are cut."""
    internal = open(os.path.join(CSRC, "internal.h")).read()
    body = internal[internal.index("timed_launch("):]
    assert body.index("launch_counts(grid.x, block.x)") < body.index("hipLaunchKernelGGL(")
    for name in sorted(os.listdir(CSRC)):
        text = open(os.path.join(CSRC, name)).read()
        if name != "internal.h":
            assert "hipLaunchKernelGGL(" not in text and "hipExtLaunchKernelGGL(" not in text and "<<<" not in text, name
    full = open(os.path.join(CSRC, "full_fdc.hip")).read()
    launchers = full[full.index("hipError_t launch_full_contract("):]
    assert len(re.findall(r"\bin_launches\(", launchers)) == len(re.findall(r"\btimed_launch\(", launchers)) == 5
