"""The LDS limit of a kernel is set on every device that launches it, and asked for again after a failure.  A host
program with the runtime's two functions replaced: no device is needed."""
import os
import subprocess

from conftest import ROOT

PROGRAM = r"""
#include "gsi_lds_limit.h"
#include <cstdio>

static int device = 0, calls = 0, failures = 0;
extern "C" hipError_t hipGetDevice(int* d) { *d = device; return hipSuccess; }
extern "C" hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute a, int bytes) {
  ++calls;
  if (a != hipFuncAttributeMaxDynamicSharedMemorySize || bytes != 4711) return hipErrorInvalidValue;
  return failures-- > 0 ? hipErrorOutOfMemory : hipSuccess;
}
#define CHECK(x) if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; }

int main() {
  static gsi::LdsLimit one, two;
  failures = 1;
  CHECK(one.allow(&device, 4711) == hipErrorOutOfMemory);
  failures = 0;
  CHECK(one.allow(&device, 4711) == hipSuccess && calls == 2);  // a failure is not kept
  CHECK(one.allow(&device, 4711) == hipSuccess && calls == 2);
  for (int d : {1, 63, 7}) {
    device = d;
    const int before = calls;
    CHECK(one.allow(&device, 4711) == hipSuccess && calls == before + 1);
    CHECK(one.allow(&device, 4711) == hipSuccess && calls == before + 1);
  }
  device = 0;
  CHECK(one.allow(&device, 4711) == hipSuccess && calls == 5);
  CHECK(two.allow(&device, 4711) == hipSuccess && calls == 6);  // another kernel
  device = 64;  // beyond what is remembered: set each time
  CHECK(one.allow(&device, 4711) == hipSuccess && one.allow(&device, 4711) == hipSuccess && calls == 8);
  return 0;
}
"""


def test_every_device_and_after_a_failure(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    csrc = os.path.join(ROOT, "paper_2605_03109_amd", "csrc")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    r = subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{csrc}", f"-I{rocm}/include", str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_no_kernel_sets_its_limit_once_per_process():
    csrc = os.path.join(ROOT, "paper_2605_03109_amd", "csrc")
    for name in sorted(os.listdir(csrc)):
        text = open(os.path.join(csrc, name)).read()
        assert name == "gsi_lds_limit.h" or "hipFuncSetAttribute" not in text, name
