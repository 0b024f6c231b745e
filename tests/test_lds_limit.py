"""A kernel's dynamic LDS limit (csrc/lds_limit.h) is raised once on every device it is launched
on, and again after a failure.  Host code only: compiled against two stand-ins of the HIP runtime
functions it calls, which record the calls."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

SOURCE = r"""
#include "lds_limit.h"
#include <cassert>
#include <vector>

static int device = 0;
static hipError_t answer = hipSuccess;
static std::vector<int> calls;  // devices the attribute was set on

extern "C" hipError_t hipGetDevice(int *d) { *d = device; return hipSuccess; }
extern "C" hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute a, int bytes) {
  assert(a == hipFuncAttributeMaxDynamicSharedMemorySize && bytes == 100000);
  calls.push_back(device);
  return answer;
}
void kernel_a() {}
void kernel_b(int) {}

int main() {
  for (int i = 0; i < 3; ++i) assert(fdc::allow_lds<kernel_a>(100000) == hipSuccess);
  assert(calls == std::vector<int>({0}));
  device = 1;  // another device of the same process
  for (int i = 0; i < 3; ++i) assert(fdc::allow_lds<kernel_a>(100000) == hipSuccess);
  assert(calls == std::vector<int>({0, 1}));
  device = 0;
  assert(fdc::allow_lds<kernel_a>(100000) == hipSuccess && calls.size() == 2);
  assert(fdc::allow_lds<kernel_b>(100000) == hipSuccess && calls.size() == 3);  // each kernel has its own
  device = 2, answer = hipErrorInvalidValue;
  assert(fdc::allow_lds<kernel_a>(100000) == hipErrorInvalidValue);
  answer = hipSuccess;
  assert(fdc::allow_lds<kernel_a>(100000) == hipSuccess && calls.size() == 5);
  assert(fdc::allow_lds<kernel_a>(100000) == hipSuccess && calls.size() == 5);
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")),
                    reason="g++ and the HIP headers are needed")
def test_lds_limit_is_raised_on_every_device(tmp_path):
    src, exe = tmp_path / "limit.cpp", tmp_path / "limit"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"), "-I",
                    os.path.join(ROOT, "paper_2106_12736_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, timeout=120)
    subprocess.run([str(exe)], check=True, timeout=60)
    # the kernels with more than 64 KB go through it
    for name in ("full_fdc.hip", "small.hip", "tail.hip"):
        text = open(os.path.join(ROOT, "paper_2106_12736_amd", "csrc", name)).read()
        assert "hipFuncSetAttribute" not in text and "allow_lds<" in text
