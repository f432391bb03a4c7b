"""The permission for more than 64 KB of dynamic LDS belongs to a kernel on one device: the launchers ask for it once per
device, from any number of threads, and again after a failure (host code over stand-ins for the two runtime calls)."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_18719_amd", "csrc")

PROGRAM = r"""
#include "lds_limit.h"
#include <cstdio>
#include <thread>
#include <vector>
static thread_local int device = 0;
static std::atomic<int> calls[80];
static std::atomic<bool> failing{false};
extern "C" hipError_t hipGetDevice(int* d) { *d = device; return hipSuccess; }
extern "C" hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute a, int bytes) {
  if (a != hipFuncAttributeMaxDynamicSharedMemorySize || bytes != 70000) return hipErrorInvalidValue;
  ++calls[device];
  return failing ? hipErrorOutOfMemory : hipSuccess;
}
#define CHECK(x) if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; }
int main() {
  static vla::LdsLimit small, limit, other;
  CHECK(small.allow(nullptr, 65536) == hipSuccess && calls[0] == 0);
  failing = true;
  CHECK(limit.allow(nullptr, 70000) != hipSuccess && calls[0] == 1);
  failing = false;
  CHECK(limit.allow(nullptr, 70000) == hipSuccess && calls[0] == 2);
  CHECK(limit.allow(nullptr, 70000) == hipSuccess && calls[0] == 2);
  device = 1;  // a second device of the process
  CHECK(limit.allow(nullptr, 70000) == hipSuccess && calls[1] == 1);
  CHECK(limit.allow(nullptr, 70000) == hipSuccess && calls[1] == 1);
  device = 0;
  CHECK(limit.allow(nullptr, 70000) == hipSuccess && calls[0] == 2);
  CHECK(other.allow(nullptr, 70000) == hipSuccess && calls[0] == 3);  // another kernel
  device = 70;
  for (int i = 1; i <= 2; ++i) CHECK(limit.allow(nullptr, 70000) == hipSuccess && calls[70] == i);
  // no thread goes on before its device's call has been made
  static vla::LdsLimit shared;
  std::atomic<int> wrong{0};
  std::vector<std::thread> ts;
  for (int t = 0; t < 8; ++t)
    ts.emplace_back([&, t] {
      device = 8 + t % 4;
      for (int i = 0; i < 1000; ++i)
        if (shared.allow(nullptr, 70000) != hipSuccess || calls[device] < 1) ++wrong;
    });
  for (auto& t : ts) t.join();
  CHECK(wrong == 0);
  return 0;
}
"""


def test_asked_once_per_kernel_and_device(tmp_path):
    if shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"):
        pytest.skip("no host compiler or HIP headers")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-isystem",
                        "/opt/rocm/include", str(src), "-o", str(exe), "-pthread"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


def test_every_launcher_asks_through_it():
    """Outside the header the attribute is set only by the decode layer kernel's occupancy query, unconditionally."""
    uses = {f: len(re.findall(r"hipFuncSetAttribute\(", open(os.path.join(CSRC, f)).read())) for f in os.listdir(CSRC)}
    assert {f: n for f, n in uses.items() if n} == {"lds_limit.h": 1, "decode_layer.hip": 1}
