"""More than 64 KB of dynamic LDS is allowed per kernel and per device, whichever thread launches first.
Runs on the host: the two HIP calls are stand-ins that count."""
import glob
import os
import shutil
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_13319_amd", "csrc")

PROGRAM = r"""
#include <stdio.h>
#include <thread>
#include <vector>
#include "lds_limit.h"
static thread_local int device = 0;
static std::atomic<int> asked[80];
static std::atomic<bool> refuse{false};
extern "C" hipError_t hipGetDevice(int* d) { *d = device; return hipSuccess; }
extern "C" hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute a, int v) {
  if (a != hipFuncAttributeMaxDynamicSharedMemorySize || v != 163840) return hipErrorInvalidValue;
  if (refuse) return hipErrorInvalidValue;
  asked[device]++;
  return hipSuccess;
}
#define WANT(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)
int main() {
  static std::atomic<uint64_t> one{0}, other{0}, many{0};
  auto allow = [](std::atomic<uint64_t>& d, int dev) { device = dev; return pipesd::allow_lds(d, nullptr, 163840); };
  refuse = true;
  WANT(allow(one, 0) != hipSuccess);
  refuse = false;
  for (int i = 0; i < 3; ++i) WANT(allow(one, 0) == hipSuccess);
  WANT(asked[0] == 1);  // (the refused call was not taken for an answer, the later ones were not repeated)
  for (int i = 0; i < 3; ++i) WANT(allow(one, 1) == hipSuccess);
  WANT(asked[1] == 1 && asked[0] == 1);  // another device
  WANT(allow(other, 0) == hipSuccess && asked[0] == 2);  // another kernel
  WANT(allow(one, 70) == hipSuccess && allow(one, 70) == hipSuccess && asked[70] == 2);
  std::vector<std::thread> t;
  for (int i = 0; i < 8; ++i) t.emplace_back([i] { device = i % 4 + 8; for (int j = 0; j < 100; ++j) (void)pipesd::allow_lds(many, nullptr, 163840); });
  for (auto& x : t) x.join();
  for (int d = 8; d < 12; ++d) WANT(asked[d] == 1 || asked[d] == 2);
  return 0;
}
"""


def test_asked_once_per_kernel_and_device(tmp_path):
    cxx = shutil.which("g++") or "/opt/rocm/llvm/bin/clang++"
    (tmp_path / "t.cpp").write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", CSRC,
                    "-o", str(tmp_path / "t"), str(tmp_path / "t.cpp")], check=True)
    r = subprocess.run([str(tmp_path / "t")], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


def test_every_launcher_asks_through_it():
    """No launcher keeps a flag of its own, which would speak for the first device only."""
    for path in glob.glob(os.path.join(CSRC, "*.hip")):
        assert "hipFuncSetAttribute" not in open(path).read(), path
