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


def test_scan_window_loads_stay_inside_the_in_edges(tmp_path):
    """The window loads of a scan, windows past the run's end included (three
    are in flight), read the record of an in-edge of the batch: the first
    window's in-edge and the mask are set up as tri_batch does, and the
    records are an array that refuses other indexes."""
    load = between(source("slim_tri.hip"), "auto load = [&](uint32_t win, Win& x) {", "uint32_t qcnt = 0;")
    consts = "".join(between(source("slim_tri.hip"), f"constexpr int {c} =", "\n") + "\n"
                     for c in ("kItemBits", "kDepth"))
    run_host(tmp_path, r'''
constexpr uint32_t kWave = 64;
''' + consts + r'''
struct uint2 { uint32_t x, y; };
static uint32_t g_lane;
static uint32_t __builtin_popc(uint32_t v) { return (uint32_t)__builtin_popcount(v); }
#define __popc __builtin_popc
static uint32_t mbcnt(uint32_t m, uint32_t from, uint32_t v) {
  const uint64_t below = (uint64_t(1) << g_lane) - 1;
  return v + (uint32_t)__builtin_popcount(m & (uint32_t)(below >> from));
}
#define __builtin_amdgcn_mbcnt_lo(m, v) mbcnt(m, 0, v)
#define __builtin_amdgcn_mbcnt_hi(m, v) mbcnt(m, 32, v)
struct Records {
  std::vector<uint2> v;
  uint2 operator[](uint32_t k) const {
    if (k >= v.size()) { printf("FAIL in-edge %u of %zu\n", k, v.size()); exit(1); }
    return v[k];
  }
};
template <int kQuad>
struct Window {
  struct vec { uint32_t v[kQuad]; };
  uint32_t row, rec;
  vec w;
};
template <int kQuad, int kM>
void drive(const std::vector<uint32_t>& len) {  // items of each in-edge
  using Win = Window<kQuad>;
  struct { uint32_t mask[2 * (kM + 2 * kDepth)]; Records ie_scan; } S{};
  std::vector<uint32_t> pre;
  uint32_t W = 0;
  for (uint32_t l : len) {
    pre.push_back(W);
    S.ie_scan.v.push_back({0u - kQuad * W, W});
    W += (l + kQuad - 1) / kQuad;
  }
  std::vector<uint32_t> dag(kQuad * W + 4);
  struct { struct { const uint32_t* dag_col; } a; } C{{dag.data()}};
  const uint32_t kTW = 8, nk = (uint32_t)pre.size();
  for (uint32_t s0 = 0; s0 < W; s0 += kM * kWave) {
    memset(S.mask, 0, sizeof(S.mask));
    for (uint32_t p : pre)
      if (p > s0 && p - s0 <= (uint32_t)kM * kWave) S.mask[(p - s0 - 1) >> 5] |= 1u << ((p - s0 - 1) & 31u);
    const uint32_t n = std::min<uint32_t>(W - s0, kM * kWave), nwin = (n + kWave - 1) / kWave;
    for (uint32_t w = 0; w < kTW; ++w)
      for (g_lane = 0; g_lane < kWave; ++g_lane) {
        uint32_t wi = nwin * w / kTW;
        const uint32_t we = nwin * (w + 1) / kTW;
        if (wi >= we) continue;
        uint32_t kcur = 0;
        for (uint32_t k = 0; k < nk; ++k)
          if (pre[k] <= s0 + wi * kWave) kcur = k;
        const uint32_t item0 = kQuad * s0;
        const uint32_t lim = kQuad * (n < we * kWave ? n : we * kWave);
        const uint32_t lane = g_lane;
''' + load.replace("Smem::kM", "kM") + r'''
        Win x[kDepth];
        for (int d = 0; d < kDepth; ++d) load(wi + d, x[d]);
        for (; wi < we; wi += kDepth)
          for (int d = 0; d < kDepth; ++d) {
            if (wi + d < we) {  // the in-edge of the lane's quad
              const uint32_t q = s0 + (wi + d) * kWave + lane;
              uint32_t want = 0;
              for (uint32_t k = 0; k < nk; ++k)
                if (pre[k] <= q) want = k;
              if (q < W && x[d].rec >> kItemBits != want) { printf("FAIL window\n"); exit(1); }
            }
            load(wi + d + kDepth, x[d]);
          }
      }
  }
}
int main() {
  for (uint32_t n : {1, 2, 63, 64, 65, 350, 384, 512})
    for (uint32_t l : {1, 3, 4, 5, 17, 64, 300}) {
      const std::vector<uint32_t> len(n, l);
      drive<4, 512>(len);
      drive<4, 256>(len);
      drive<1, 256>(len);
    }
  printf("OK\n");
  return 0;
}
''')


def test_a_captured_batch_is_kept_only_under_the_same_knobs(tmp_path):
    """Every knob that reaches the captured launches is part of the key under
    which a batch's capture is replayed."""
    import re
    tuning = between(source("slim_internal.h"), "struct Tuning {", "Tuning& tuning();")
    same = between(source("slim_batch.hip"), "bool same_knobs(", "void drop_graph(")
    knobs = re.findall(r"^  int (\w+) =", tuning, flags=re.M)
    assert {"tri_tile", "eo_rounds", "eo_list_try"} <= set(knobs)
    checks = "".join(f'''
  {{
    Tuning a, b;
    b.{k} = a.{k} + 1;
    if (same_knobs(a, b) || !same_knobs(b, b)) {{ printf("FAIL {k}\\n"); return 1; }}
  }}''' for k in knobs)
    run_host(tmp_path, tuning + same + "int main() {" + checks + '''
  printf("OK\\n");
  return 0;
}
''')
