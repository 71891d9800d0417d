"""The projections' launch plans on the CPU: a small program over the library's own planners
(linked from libspp.so, with the host stand-ins' headers) checks, for every row count of a pass,
that the work buffer sized at model creation holds the split-K partials of its plans, and that
it is not sized for projections that no pass runs."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2606_29565_amd")
STUB = os.path.join(ROOT, "tests", "cpu_runtime")

PROGRAM = r"""
#include <cstdio>
#include "plans.hpp"
using namespace spp;
int main() {
  struct Model { const char* name; Shape s; bool fp4; } models[] = {
      {"tiny-f32", {2, 256, 4, 4, 64, 1024, 4096, 1e-5f, 1e4, 0}, false},
      {"f32", {2, 1024, 16, 4, 64, 2784, 4096, 1e-5f, 1e4, 0}, false},
      {"small", {2, 256, 4, 2, 64, 512, 2048, 1e-5f, 1e4, 1}, false},
      {"narrow", {2, 512, 8, 2, 64, 1344, 2048, 1e-5f, 1e4, 1}, false},
      {"mid", {2, 2048, 16, 4, 128, 5632, 32000, 1e-5f, 1e4, 1}, false},
      {"8b", {32, 4096, 32, 8, 128, 14336, 128256, 1e-5f, 5e5, 1}, false},
      {"32b", {64, 5120, 64, 8, 128, 27648, 152064, 1e-5f, 1e6, 1}, false},
      {"fp4-small", {2, 256, 4, 2, 64, 384, 2048, 1e-5f, 1e4, 1}, true},
      {"fp4-mid", {2, 2048, 16, 4, 128, 5632, 32000, 1e-5f, 1e4, 1}, true},
      {"70b", {80, 8192, 64, 8, 128, 28672, 128256, 1e-5f, 5e5, 1}, true}};
  const int kMax = 4200;
  for (const Model& m : models) {
    size_t most = 0;
    for (int M = 1; M <= kMax; ++M) {
      const StepPlans p = step_plans(m.s, m.fp4, M);
      most = std::max(most, partial_elems(m.s, p, M));  // what passes of up to M rows write
      if (M <= 700 || M % 37 == 0 || M == kMax) {
        const size_t have = partial_elems_upto(m.s, m.fp4, M);
        if (have < most || have > most + most / 2) {
          std::printf("%s: up to %d rows write %zu floats of partials, the buffer has %zu\n", m.name, M,
                      most, have);
          return 1;
        }
      }
    }
  }
  std::printf("OK\n");
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_partials_buffer_holds_every_pass(tmp_path):
    src, exe = tmp_path / "plans.cpp", str(tmp_path / "plans")
    src.write_text(PROGRAM)
    lib = os.path.join(PKG, "libspp.so")
    cmd = ["g++", "-std=c++17", "-O1", "-I", STUB, "-I", os.path.join(ROOT, "include"), "-I",
           os.path.join(PKG, "csrc"), str(src), lib, "-Wl,-rpath," + PKG, "-Wl,--allow-shlib-undefined",
           "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), (r.stdout + r.stderr)[-2000:]
