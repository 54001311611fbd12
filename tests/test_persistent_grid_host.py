"""The persistent kernels' grid: one occupancy query per kernel and device, with
more kernels and devices than one GPU's launches need (host code, compiled here
with the runtime's three calls counted and answered by the test)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

PROGRAM = r"""
#include "persistent_grid.hpp"
#include <stdio.h>
static int g_dev, g_queries;
extern "C" {
hipError_t hipGetDevice(int* d) { *d = g_dev; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int dev) { *v = 256 - dev; return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int, size_t) {
  ++g_queries;
  *n = 1 + (int)((uintptr_t)f & 1);
  return hipSuccess;
}
}
int main() {
  int wrong = 0;
  for (int round = 0; round < 3; ++round)
    for (g_dev = 0; g_dev < 8; ++g_dev)
      for (uintptr_t k = 1; k <= 16; ++k)
        wrong += pulse::persistent_grid((const void*)k, 1024) != (256 - g_dev) * (1 + (int)(k & 1));
  printf("%d %d\n", g_queries, wrong);
}
"""


def test_one_query_per_kernel_and_device(tmp_path):
    if not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime_api.h")):
        pytest.skip("no HIP headers")
    src, exe = tmp_path / "grid.cpp", tmp_path / "grid"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"), "-I",
                    os.path.join(ROOT, "paper_2602_03839_amd", "csrc"), str(src), "-o", str(exe), "-pthread"], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()
    assert out == ["128", "0"]
