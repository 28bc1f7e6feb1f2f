"""Pieces of the device code compiled for the host and driven there: index
arithmetic at sizes that no test graph reaches."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1912_08950_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"

pytestmark = pytest.mark.skipif(not os.path.exists(CLANG) and not shutil.which("clang++"),
                                reason="needs clang++ (vector types)")

PRELUDE = r'''
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <type_traits>
#include <vector>
#define __device__
#define __forceinline__ inline
'''


def source(name):
    return open(os.path.join(CSRC, name)).read()


def between(text, start, end):
    i = text.index(start)
    return text[i:text.index(end, i)]


def run_host(tmp_path, prog):
    cpp, exe = tmp_path / "piece.cpp", tmp_path / "piece"
    cpp.write_text(PRELUDE + prog)
    cc = CLANG if os.path.exists(CLANG) else "clang++"
    subprocess.run([cc, "-std=c++17", "-O1", "-g", str(cpp), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and out.stdout.startswith("OK"), out.stdout + out.stderr


def test_in_edge_search_at_the_edge_limit(tmp_path):
    """dag_find over rows that end at DAG positions up to 2^32 - 1 (the most
    edges a graph may have), against std::lower_bound; the entries behind the
    row are smaller than any that is looked for.  The columns are reserved
    address space of which only the last pages are touched."""
    find = between(source("slim_tri.hip"), "typedef uint32_t find4_t", "__device__ __forceinline__ void wave_sync")
    run_host(tmp_path, r'''
#include <sys/mman.h>
constexpr uint32_t kFenceStep = 32;
struct TriArgs { const uint32_t* dag_col; const uint32_t* fence; };
''' + find + r'''
int main() {
  auto reserve = [](uint64_t bytes) {
    void* p = mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (p == MAP_FAILED) { printf("FAIL reserve\n"); exit(1); }
    return static_cast<uint32_t*>(p);
  };
  const uint64_t most = (uint64_t(1) << 32) - 1;
  uint32_t* col = reserve(4 * (most + 64));
  uint32_t* fence = reserve(4 * (most / kFenceStep + 64));
  TriArgs a{col, fence};
  uint64_t n = 0;
  for (uint64_t hi = most - 40; hi <= most; ++hi)
    for (uint64_t len : {1, 2, 3, 4, 7, 8, 9, 15, 16, 17, 31, 32, 33, 64, 65, 200, 1000}) {
      const uint64_t lo = hi - len;
      for (uint64_t p = lo; p < hi; ++p) col[p] = 100 + 3 * (uint32_t)(p - lo);
      for (uint64_t p = hi; p < most + 64; ++p) col[p] = 0;
      for (uint64_t q = lo / kFenceStep; q <= most / kFenceStep + 8; ++q) fence[q] = col[q * kFenceStep];
      for (uint32_t x = 99; x <= 101 + 3 * len; ++x, ++n) {
        const uint32_t want = (uint32_t)(std::lower_bound(col + lo, col + hi, x) - col);
        const uint32_t got = dag_find(a, (uint32_t)lo, (uint32_t)hi, x);
        if (got != want) {
          printf("FAIL row [%llu, %llu) x %u: %u, not %u\n", (unsigned long long)lo, (unsigned long long)hi, x, got, want);
          return 1;
        }
      }
    }
  printf("OK %llu searches\n", (unsigned long long)n);
  return 0;
}
''')
