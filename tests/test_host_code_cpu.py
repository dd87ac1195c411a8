"""Host-callable pieces of the native code, compiled for the CPU and run there:
the ranges that kernels index with, and bookkeeping that no GPU run can show."""
import os
import subprocess

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


def test_pool_keeps_what_a_capture_has_taken(tmp_path):
    """the internal workspace grows by freeing its buffer after a
    synchronisation, but a buffer taken under capture stays allocated until
    release, and stays in use where no larger one can be had"""
    out = run_host(tmp_path, r"""
#include <cstdio>
#include <cstdlib>
#include <set>
#include "oz2_pool.h"
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s", __LINE__, #x); return 1; } } while (0)
struct Fake {
  std::set<void*> live;
  char space[64];
  int next = 0, syncs = 0;
  bool full = false, broken = false;
  bool alloc(void** p, size_t) {
    if (full) return false;
    live.insert(*p = &space[next++]);
    return true;
  }
  void free(void* p) { if (!live.erase(p)) std::abort(); }
  bool sync() { ++syncs; return !broken; }
  bool has(void* p) const { return live.count(p) != 0; }
};
int main() {
  Fake mem;
  Oz2Pool pool;
  const size_t MiB = (size_t)1 << 20;
  void *a, *b, *c, *d, *e;
  CHECK(pool.get(10, false, mem, &a) == Oz2Pool::kOk && pool.bytes == MiB);
  CHECK(pool.get(2 * MiB, false, mem, &b) == Oz2Pool::kOk);       // plain growth
  CHECK(!mem.has(a) && mem.has(b) && mem.syncs == 1);
  CHECK(pool.get(MiB, true, mem, &c) == Oz2Pool::kOk && c == b);  // a capture takes b
  CHECK(pool.get(2 * MiB, false, mem, &c) == Oz2Pool::kOk && c == b);
  mem.full = true;                                                // no room for more
  CHECK(pool.get(4 * MiB, false, mem, &c) == Oz2Pool::kNoMem);
  CHECK(mem.has(b) && pool.get(2 * MiB, false, mem, &c) == Oz2Pool::kOk && c == b);
  mem.full = false;
  CHECK(pool.get(4 * MiB, false, mem, &c) == Oz2Pool::kOk && c != b);
  CHECK(mem.has(b) && mem.has(c));                                // b stays for its graph
  CHECK(pool.get(8 * MiB, false, mem, &d) == Oz2Pool::kOk);       // c was nobody's
  CHECK(mem.has(b) && !mem.has(c) && mem.has(d));
  CHECK(pool.get(8 * MiB, true, mem, &e) == Oz2Pool::kOk && e == d);
  CHECK(pool.get(9 * MiB, true, mem, &e) == Oz2Pool::kOk);        // (a capture that may allocate)
  CHECK(pool.get(10 * MiB, false, mem, &a) == Oz2Pool::kOk);
  CHECK(mem.live.size() == 4 && mem.has(b) && mem.has(d) && mem.has(e) && mem.has(a));
  mem.broken = true;
  CHECK(pool.get(11 * MiB, false, mem, &c) == Oz2Pool::kDevice && mem.has(a));
  pool.release(mem);
  CHECK(mem.live.empty() && !pool.ptr && !pool.held && pool.bytes == 0);
  std::printf("ok");
}
""")
    assert out == "ok"
