"""Kernels that need more LDS than a launch gets by default have their limit raised on every device they run on.

A host program stands in for the HIP runtime's two devices and launches; the library's own launch functions run, no
device is used.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2605_24882_amd")
CLANG = "/opt/rocm/llvm/bin/clang++"

STAND_IN = r"""
#include <cstdio>
#include <math.h>
#include <set>
#include <utility>
#include "csrc/gf_internal.h"
#include "csrc/k_solve.h"

static int device = 0, launches = 0, below = 0;
static std::set<std::pair<int, const void *>> raised;
struct Config { dim3 g, b; size_t lds; hipStream_t s; };
static Config config;
extern "C" {
hipError_t hipGetDevice(int *d) { *d = device; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int) {
  raised.insert({device, f});
  return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
  config = {g, b, lds, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s) {
  *g = config.g, *b = config.b, *lds = config.lds, *s = config.s;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **, size_t, hipStream_t) {
  ++launches;
  if (!raised.count({device, f})) ++below;
  return hipSuccess;
}
}

int main() {
  gf::CycleArgs<double> a;
  gf::CycleArgs<float> b;
  a.p = b.p = 2;
  a.lds = b.lds = 100 << 10;
  for (int d : {0, 1, 0, 1}) {
    device = d;
    for (bool same : {false, true}) {
      gf::coarse_cycle<double>(a, 1, same, nullptr);
      gf::coarse_cycle<float>(b, 1, same, nullptr);
    }
    if (!gf::launch_coarse_both(nullptr, nullptr, 150, nullptr, 1, nullptr, nullptr, nullptr)) return 2;
  }
  std::printf("%d of %d launches with the default limit\n", below, launches);
  return launches == 20 && below == 0 ? 0 : 1;
}
"""


@pytest.mark.skipif(not os.path.exists(CLANG), reason="needs the ROCm compiler")
def test_every_device_gets_the_limit(tmp_path):
    src, exe = tmp_path / "stand_in.cpp", str(tmp_path / "stand_in")
    src.write_text(STAND_IN)
    cmd = [CLANG, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + PKG, str(src), "-o", exe,
           "-L" + PKG, "-lgfield", "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath," + PKG, "-Wl,-rpath,/opt/rocm/lib"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
