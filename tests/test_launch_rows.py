"""The rows of work counts that a call reserves (wg_rows_of) against the
workgroups of the inertia search's launches (lone_blocks), each of which writes
one, over every number of lanes per wavelength at the edges of its range and
numbers of models far above that of the wavelengths (models without wavelengths
are allowed).  Compiled for the host from the library's own header."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include <hip/hip_runtime.h>
#include "masw_internal.hpp"
using namespace masw;
int main() {
  const int64_t n_max = 32 * 1024;  // 8 lanes: up to 32 wavelengths per SIMD
  long bad = 0, seen = 0;
  for (int S : {64, 32, 8})
    for (int64_t n : {int64_t(1), int64_t(2), int64_t(9), int64_t(2048), int64_t(2049), int64_t(4096), int64_t(4097),
                      int64_t(10001), n_max})
      for (int64_t models : {int64_t(1), int64_t(2), n / 2, n - 1, n, n + 1, 4 * n, int64_t(8000), int64_t(10000),
                             int64_t(1) << 20, int64_t(0x7fffffff)}) {
        if (models < 1) continue;
        ++seen;
        const int64_t blocks = lone_blocks(n, models, S);
        // every run, and every model that starts inside one, has a wavefront
        const int64_t waves = blocks * kInertiaWaves, extra = lone_extra(n, models, S);
        const bool ok = blocks <= wg_rows_of(n) && waves >= lone_runs(n, S) + extra &&
                        (S == 64 || models < 2 || (extra >= 1 && extra <= models));
        if (!ok) {
          ++bad;
          std::printf("S=%d n=%ld models=%ld: %ld workgroups, %ld rows\n", S, long(n), long(models), long(blocks),
                      long(wg_rows_of(n)));
        }
      }
  std::printf("%ld cases, %ld bad\n", seen, bad);
  return bad != 0;
}
"""


def test_rows_cover_the_inertia_launches(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    src, exe = tmp_path / "rows.hip", str(tmp_path / "rows")
    src.write_text(SOURCE)
    b = subprocess.run([hipcc, "--cuda-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                        os.path.join(ROOT, "paper_2003_02256_amd", "csrc"), str(src), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert b.returncode == 0, b.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    print(r.stdout)
    assert r.returncode == 0, (r.returncode, r.stdout[-2000:], r.stderr[-2000:])
