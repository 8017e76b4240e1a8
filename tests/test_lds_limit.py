"""The dynamic LDS limit of a kernel is set on every device that launches it. The header is
compiled for the host against a HIP runtime of this test's own: the two functions that it
calls, with a current device per thread and a record of the calls."""
import glob
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2212_11142_amd", "csrc")

PROGRAM = r"""
#include "lds_limit.h"
#include <cstdio>
#include <thread>
#include <vector>

static thread_local int device = 0;
static std::atomic<int> calls[128];
static std::atomic<int> failures{0};  // so many calls fail
extern "C" hipError_t hipGetDevice(int *d) { *d = device; return hipSuccess; }
extern "C" hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute a, int bytes) {
  if (!f || a != hipFuncAttributeMaxDynamicSharedMemorySize || bytes != 131072) return hipErrorInvalidValue;
  if (failures.load() > 0) { --failures; return hipErrorInvalidDevice; }
  ++calls[device];
  return hipSuccess;
}
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
  static bgp::LdsLimit a, b;
  const int k = 0;
  for (int r = 0; r < 3; ++r)
    for (int d : {0, 1, 7}) {
      device = d;
      CHECK(a.set(&k, 131072) == hipSuccess);
      CHECK(calls[d] == 1);
    }
  device = 1;
  CHECK(b.set(&k, 131072) == hipSuccess && calls[1] == 2);  // another kernel's own
  device = 2;
  failures = 1;
  CHECK(a.set(&k, 131072) == hipErrorInvalidDevice && calls[2] == 0);
  CHECK(a.set(&k, 131072) == hipSuccess && calls[2] == 1);
  device = 63;
  CHECK(a.set(&k, 131072) == hipSuccess && a.set(&k, 131072) == hipSuccess && calls[63] == 1);
  device = 64;
  CHECK(a.set(&k, 131072) == hipSuccess && a.set(&k, 131072) == hipSuccess && calls[64] == 2);
  std::vector<std::thread> ts;
  for (int t = 0; t < 8; ++t)
    ts.emplace_back([&k, t] {
      for (int r = 0; r < 1000; ++r) {
        device = 10 + (t + r) % 8;
        if (a.set(&k, 131072) != hipSuccess) calls[100] = 1;
      }
    });
  for (auto &t : ts) t.join();
  CHECK(calls[100] == 0);
  for (int d = 10; d < 18; ++d) CHECK(calls[d] >= 1);
  std::printf("ok\n");
  return 0;
}
"""


def test_set_once_per_device(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I" + CSRC,
                    "-I" + os.path.join(rocm, "include"), str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and out.stdout == "ok\n", out.stdout


def test_no_other_place_sets_it():
    """Every kernel with a raised limit goes through the class, none through a flag."""
    for path in glob.glob(os.path.join(CSRC, "*.hip")):
        text = open(path).read()
        assert "hipFuncSetAttribute" not in text, path
        assert not re.search(r"\bstatic bool\b", text), path
