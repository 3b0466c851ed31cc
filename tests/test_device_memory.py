"""Device memory that freed blocks hold back is given up before an allocation fails.

A host program stands in for the HIP allocator (a budget of one megabyte) and drives the library's own buffers: the
library is loaded, no device is used.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2605_24882_amd")
CLANG = "/opt/rocm/llvm/bin/clang++"

STAND_IN = r"""
#include <cstdio>
#include <cstdlib>
#include <map>
#include "csrc/gf_internal.h"

static std::map<void *, size_t> blocks;
static size_t used = 0, budget = 1 << 20;
static hipError_t last = hipSuccess;
extern "C" {
hipError_t hipMalloc(void **p, size_t n) {
  if (used + n > budget) return last = hipErrorOutOfMemory;
  blocks[*p = std::malloc(n)] = n;
  used += n;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  used -= blocks.at(p);
  blocks.erase(p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemset(void *, int, size_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
}

#define EXPECT(x)                                        \
  if (!(x)) {                                            \
    std::printf("line %d: %s is false\n", __LINE__, #x); \
    return 1;                                            \
  }

int main() {
  auto a = std::make_shared<gf::Pool>(), b = std::make_shared<gf::Pool>();
  {
    gf::PBuf<char> x, y;
    x.alloc(a, 500 << 10);
    y.alloc(b, 300 << 10);
  }
  EXPECT(used >= (size_t)800 << 10);  // both pools keep their block
  try {
    gf::DBuf<char> d;
    d.alloc(900 << 10);
    EXPECT(used == (size_t)900 << 10);
    EXPECT(hipGetLastError() == hipSuccess);
  } catch (...) {
    std::printf("a buffer that fits beside no kept block was refused\n");
    return 1;
  }
  {
    gf::PBuf<char> x;
    x.alloc(a, 600 << 10);
  }
  try {  // the other pool's block as well
    gf::PBuf<char> y;
    y.alloc(b, 600 << 10);
  } catch (...) {
    std::printf("a block that fits beside no kept block was refused\n");
    return 1;
  }
  bool refused = false;
  try {
    gf::DBuf<char> d;
    d.alloc(2 << 20);
  } catch (...) {
    refused = true;
  }
  EXPECT(refused);
  a.reset();
  b.reset();
  EXPECT(used == 0);
  return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(CLANG), reason="needs the ROCm compiler")
def test_kept_blocks_are_given_up(tmp_path):
    src, exe = tmp_path / "stand_in.cpp", str(tmp_path / "stand_in")
    src.write_text(STAND_IN)
    cmd = [CLANG, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + PKG, str(src), "-o", exe,
           "-L" + PKG, "-lgfield", "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath," + PKG, "-Wl,-rpath,/opt/rocm/lib"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
