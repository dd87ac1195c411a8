"""Host-callable pieces of the native code, compiled for the CPU and run there:
the ranges that kernels index with, and bookkeeping that no GPU run can show."""
import os
import subprocess

import pytest

from paper_2606_06510_amd.build import CSRC, hipcc


def run_host(tmp_path, body):
    """Compile ``body`` (a main() and what it needs) against the library's
    headers for the host only, run it, and return what it printed."""
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(body)
    r = subprocess.run([hipcc(), "-x", "hip", "--offload-host-only", "--offload-arch=gfx950",
                        "-std=c++17", "-O1", "-Wall", "-Wno-unused-function", "-I", CSRC,
                        str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


def test_rebase_table_row_stays_in_the_table(tmp_path):
    """every pair of exponents a row maximum and a 64-k segment can have, the 0
    of an all-zero segment among them, gives a row of the five"""
    out = run_host(tmp_path, r"""
#include <cstdio>
#include "oz2_internal.h"
int main() {
  int lo = 9, hi = -9, bad = 0;
  for (int E = -1073; E <= 1024; ++E) {
    for (int Et = -1073; Et <= E; ++Et) {
      const int r = oz2_rebase_row(E, Et);
      lo = r < lo ? r : lo;
      hi = r > hi ? r : hi;
      bad += r != (E - Et < 4 ? E - Et : 4);
    }
    const int z = oz2_rebase_row(E, 0);   // an all-zero segment
    lo = z < lo ? z : lo;
    hi = z > hi ? z : hi;
  }
  std::printf("%d %d %d", lo, hi, bad);
}
""")
    assert out == "0 4 0"
