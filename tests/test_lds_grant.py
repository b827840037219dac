"""Dynamic LDS grants (lds_grant.cpp) against a counted stand-in for the two HIP
calls it makes: the attribute is set once per kernel, device and larger size,
from any thread, and again after a refusal.  CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1209_5553_amd", "csrc")
HIP_INCLUDE = "/opt/rocm/include"

DRIVER = r"""
#include "lds_grant.h"
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>

static thread_local int dev = 0;
static std::atomic<int> calls{0};
static std::atomic<bool> refuse{false};
extern "C" hipError_t hipGetDevice(int* d) { *d = dev; return hipSuccess; }
extern "C" hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) {
  ++calls;
  return refuse ? hipErrorInvalidValue : hipSuccess;
}
static char k0, k1;
static void expect(int n, const char* what) {
  if (calls != n) { std::printf("%s: %d calls, expected %d\n", what, calls.load(), n); std::exit(1); }
}
int main() {
  using erem::lds_grant;
  lds_grant(&k0, 90000); expect(1, "first");
  lds_grant(&k0, 90000); lds_grant(&k0, 70000); expect(1, "same or less");
  lds_grant(&k0, 100000); expect(2, "more");
  lds_grant(&k1, 70000); expect(3, "another kernel");
  dev = 1;
  lds_grant(&k0, 70000); expect(4, "another device");
  refuse = true;
  if (lds_grant(&k0, 150000) == hipSuccess) { std::puts("refusal lost"); return 1; }
  refuse = false;
  lds_grant(&k0, 150000); expect(6, "again after a refusal");
  dev = 0;
  lds_grant(&k0, 100000); expect(6, "the first device keeps its own");
  std::vector<std::thread> t;
  for (int i = 0; i < 8; ++i) t.emplace_back([i] { dev = i % 4; for (int j = 0; j < 100; ++j) lds_grant(&k1, 80000); });
  for (auto& x : t) x.join();
  expect(10, "four devices from eight threads");
  std::puts("ok");
}
"""


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(HIP_INCLUDE), reason="g++ or HIP headers missing")
def test_lds_grants_are_kept_per_kernel_and_device(tmp_path):
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text(DRIVER)
    b = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", HIP_INCLUDE, str(src),
                        os.path.join(CSRC, "lds_grant.cpp"), "-pthread", "-o", str(exe)],
                       capture_output=True, text=True, timeout=300)
    assert b.returncode == 0, b.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
