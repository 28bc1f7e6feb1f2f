// Triangle listing with selection and deletion marks (Triangle p-1-Reduction,
// section 4.3: every triangle of the input graph runs kernel `p-1-reduction`
// once; a selected triangle deletes one uniformly chosen edge).
//
// Vertices are ranked by (degree, id) and every edge points from lower to
// higher rank.  A triangle y < x < w (in rank) is found exactly once, from
// its middle vertex x: the edge (y,x) is an in-edge of x, w lies in out(x)
// and in out(y) above x.  Work is organised over tiles of CSR entries: the
// rows of a tile are middle vertices, their backward entries are the
// in-edges, and their out-lists sit in an LDS hash keyed by (w, row).  Each
// in-edge (y,x) scans the part of out(y) ranked above x, the suffix after x of
// the sorted row; the scan items of all in-edges of a batch are spread over
// the lanes, kQuad consecutive ones per lane.
//
// What bounds the scan is vector-instruction issue (on graphs far larger than
// the L2s also the traffic of the rows: 0.86 of a copy's rate at R-MAT scale
// 24), then LDS traffic, so an item costs as little as possible: one
// multiply-add, one 4-byte read of a 65536-bit filter and one bit test.  At
// scale 24 a quarter of the items are triangles and at most 3% more pass the
// filter; only those go to a per-wave stack, 64 at a time, for the exact look-up
// in the hash, the Philox draw of the id-sorted triple and the marks.  Probing
// the hash itself for every item (two 16-byte LDS reads and four key compares)
// took 4.08e10 vector instructions and 111.6 ms on that graph; filter, stack and
// 4-item lanes take 2.77e10 and, with the steps noted further down, 79.4 ms.
// The in-edge of a lane's quad comes from a bit mask of the in-edge starts (two
// bit counts) instead of a scalar loop over the boundaries inside a window.
//
// Deletion marks: (x,w) lies in the tile's own out-lists and (y,x) is an
// in-edge of the batch: byte flags in LDS; (y,w) is a byte store into
// the global per-edge mark bytes over DAG positions (the first two are
// flushed there too).  Every mark sets a value to 1 and nothing is cleared,
// so the result does not depend on the order in which triangles are found.
//
// Variants (section 4.3), in the general instantiation of the kernel:
// Triangle p-2-Reduction marks the two edges other than the drawn one;
// Min-Count p-1-Reduction first runs a counting pass (its own instantiation:
// every triangle adds 1 to each of its edges, with LDS counters for (y,x) and
// (x,w) and a global atomic for (y,w); no hash of the triple) and then marks,
// in each selected triangle, the edge of fewest triangles (ties: the drawn
// index among the tied edges).
//
// Edge-Once p-1-Reduction (section 4.3 with the conditions of section 6.2)
// runs in rounds.  Bids (pass 2 of this kernel): every selected triangle
// with no closed edge writes its priority, (Philox word 2, third vertex),
// into each of its three edges by an atomic minimum.  Acceptance (an
// edge-parallel kernel, no listing): the key on an edge names its holder
// triangle through the third vertex, and a triangle that holds the minimum
// on all three of its edges is considered -- it deletes its drawn edge and
// closes all three.  Triangles that share an edge with a considered one are
// decided against by that closed edge; an edge no undecided triangle bid on
// is closed between rounds.  The minimum of one edge compares triangles
// that differ only in their third vertex, so these per-edge keys order them
// as (word 2, a, b, c) does, and the rounds reach the set that the walk in
// that priority order reaches.  Closed in-edges are not scanned and closed
// out-list entries are not hashed, so later rounds list fewer triangles.
// Once the undecided triangles fit a list (kEoListPerEdge records per
// edge), the bidding pass that finds them appends them, and all later rounds
// run over the list (two small kernels) instead of listing triangles again;
// each of those rounds copies its bidders into a second list, which the
// next round reads, so a round costs in proportion to the undecided count.
#include <type_traits>

#include "slim_internal.h"

namespace slim {

constexpr int kTB = 512;             // threads per block
constexpr int kTW = kTB / kWave;     // waves per block
constexpr int kTT = 1024;            // CSR entries per tile
constexpr int kEntries = kTT / kTB;  // consecutive tile entries per thread
constexpr int kWavesPerEU = kTriResident * kTW / 4;  // four SIMDs per CU
constexpr int kHashCap = 2048;       // out-list entries hashed per pass
constexpr int kHashPer = kHashCap / kTB;  // most hashed entries per thread
constexpr int kPosBits = 11;         // bits of a position in the hashed range
constexpr int kBucketBits = 10;      // hash buckets of four slots (load <= 1/2)
constexpr int kBuckets = 1 << kBucketBits;
constexpr int kFiltWords = 2048;     // words of the filter: 65536 bits
constexpr int kQ = 128;              // per-wave candidate stack (records)
constexpr int kItemBits = 17;        // scan items of one mask pass: at most 2^17
// Windows whose loads are in flight together: p-1 at R-MAT scale 24 takes
// 102.6 ms with two, 98.9 with three and 98.5 with four (whose batch of 256
// graphs is 0.5% slower).
constexpr int kDepth = 3;
constexpr uint32_t kEmpty = 0xffffffffu;
constexpr uint32_t kDead = 0xffffffffu;  // Edge-Once list record of a decided triangle

static_assert(kEntries * kTB == kTT && kEntries == 2, "two tile entries per thread");
static_assert(kHashCap <= 2 * kBuckets && kHashCap <= (1 << kPosBits), "a position fits a slot's low bits");

// In-edges per batch (kB) and words of the in-edge mask (kM) of each
// instantiation: as many as two blocks per CU allow in LDS; the general and
// Edge-Once ones also keep per-in-edge counts or bids (larger batches cut
// the per-batch setup and barriers).
constexpr int kLdsPerBlock = 160 * 1024 / kTriResident;
template <int kMode>
constexpr int kBatchOf = kMode == kModePlain ? 512 : (kMode == kModeEO ? 352 : 384);
template <int kMode>
constexpr int kMaskOf = kMode == kModePlain ? 512 : 256;

// Scan items per lane of a window.  Four (one 16-byte load, one in-edge
// search and one address for four items) is the fastest at R-MAT scale 24:
// 102.6 ms per p-1 call against 112.6 with two and 133 with one.  The
// counting pass takes one: every hit is a global atomic on its {y,w} edge,
// and only consecutive items in consecutive lanes let the atomics of a line
// travel together (scale 20: 4.25 ms with one, 6.97 ms with four).
template <int kMode>
constexpr int kQuadOf = kMode == kModeCount ? 1 : 4;

template <int kB_, int kM_, int kQuad_>
struct TriSmem {
  static constexpr int kB = kB_, kM = kM_, kQuad = kQuad_;
  static_assert(kB <= kTB && kM <= kTB, "one thread per in-edge and per mask word in the setup");
  static_assert(kM * kWave * kQuad <= (1 << kItemBits) && kB <= (1 << (32 - kItemBits)),
                "a candidate's in-edge and item share one word");
  uint32_t filt[kFiltWords];  // bit set: some hashed key may have it
  uint4 bucket[kBuckets];     // slots: (hash << kPosBits) | position in range, or kEmpty
  uint2 xw[kHashCap];         // {rank id, original (local) id} of each hashed entry
  uint8_t xflag[kHashCap];    // deletion mark of each hashed entry
  uint32_t srow[kTT];  // row of each tile entry (after the max-scan)
  uint16_t bw[kTT];    // local indices of the tile's backward entries, in order, and,
                       //   from the end down, of its forward entries
  // the batch's in-edges that have something to scan, in order
  uint2 ie_scan[kB];      // {scan begin - first item, row constant of the hash}
  uint4 ie_tri[kB];       // {end item, y old id, x old id, row's first position | length << 16}
  uint32_t ie_pre[kB];    // first quad
  uint8_t ie_flag[kB];    // deletion mark of (y,x)
  uint64_t mask[kM + 2 * kDepth];  // bit i of a window: the next in-edge starts at its quad
                                   //   i + 1; the words from kM on stay 0
  union {
    uint32_t dpos[kHashCap];  // row start offset at each row's first hashed position, else 0
    uint2 queue[kTW][kQ];     // candidates {w, (in-edge << kItemBits) | item}
  } u;
  uint32_t wsum[kTW], wcnt[kTW], wmax[kTW];
  uint32_t bcast[4];
  uint64_t red[2][kTW];
};

template <int kB, int kM, int kQ>
struct TriSmemPlain {
  TriSmem<kB, kM, kQ> s;
};
// LDS of the general instantiation: per-edge triangle counts of the hashed
// range and of the batch's in-edges (accumulated in the counting pass, loaded
// for the Min-Count selection).
template <int kB, int kM, int kQ>
struct TriSmemGeneral {
  TriSmem<kB, kM, kQ> s;
  uint32_t xcnt[kHashCap];
  uint32_t ie_cnt[kB];
};
// LDS of the Edge-Once instantiation: the smallest bid on each in-edge of
// the batch, written to the global minimum once per batch, and the smallest
// priority word bid on each hashed out-list entry in the current pass.
template <int kB, int kM, int kQ>
struct TriSmemEO {
  TriSmem<kB, kM, kQ> s;
  uint64_t ie_key[kB];
  uint32_t xmin[kHashCap];
};

// A key is (w, row); rows are told apart by the position rs of their first
// entry in the hashed range.  Its 32-bit hash w * A + rs * B gives the home
// bucket (top 10 bits; a full bucket's keys go on to the next one), the 21 low
// bits kept beside the position in a slot, and the filter's word (top 11 bits)
// and bit (low 5).
__device__ __forceinline__ uint32_t hrow(uint32_t rs) { return rs * 0x85EBCA6Bu; }
__device__ __forceinline__ uint32_t hkey(uint32_t w, uint32_t row) {
  return (uint32_t)((uint64_t)w * 0x9E3779B1u + row);  // one multiply-add
}
// The filter's bit is moved to the sign of its word.
__device__ __forceinline__ bool hfilter(const uint32_t* filt, uint32_t h) {
  const uint32_t v = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(filt) +
                                                        ((h >> 19) & (4u * kFiltWords - 4u)));
  return (int32_t)(v << (h & 31u)) < 0;
}

// The hash bits of a slot, never all ones above a position (kEmpty is no key).
__device__ __forceinline__ uint32_t hslot(uint32_t h) { return min(h << kPosBits, 0xfffff000u); }

// Exact look-up of w, of hash h, in the row of positions [rsl & 0xffff, +
// (rsl >> 16)); pair: {rank id, local id} of the entry at qpos.  Slots fill in
// order and are never removed, so the key is in its home bucket unless that
// is full.  A slot whose hash bits agree differs from them by a position, any
// other by more: the smallest difference of the four is the one to verify.
// Only a verified key counts; where the smallest one is another key's (its 21
// bits agree) or the bucket is full, every slot from there on is verified.
// (With one-entry slots and linear probing 64 look-ups took two to three
// rounds of two dependent LDS reads.)
template <class Smem>
__device__ __forceinline__ bool hfind(const Smem& S, uint32_t w, uint32_t h, uint32_t rsl,
                                      uint32_t& qpos, uint2& pair) {
  uint32_t b = h >> (32 - kBucketBits);
  const uint32_t hs = hslot(h), rs = rsl & 0xffffu, len = rsl >> 16;
  const uint4 s = S.bucket[b];
  const uint32_t q = min(min(s.x ^ hs, s.y ^ hs), min(s.z ^ hs, s.w ^ hs));
  qpos = q & (kHashCap - 1);
  pair = S.xw[qpos];
  // positions past the range (q >= kHashCap: no hash bits agree) fail the row test
  bool hit = (pair.x == w) & (q - rs < len);
  if (!hit & ((q < (uint32_t)kHashCap) | (s.w != kEmpty))) {  // rare
    for (;;) {
      const uint4 v = S.bucket[b];
      const uint32_t c[4] = {v.x ^ hs, v.y ^ hs, v.z ^ hs, v.w ^ hs};
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (c[i] < (uint32_t)kHashCap && c[i] - rs < len && S.xw[c[i]].x == w) {
          qpos = c[i];
          hit = true;
        }
      if (hit | (v.w == kEmpty)) break;
      b = (b + 1) & (kBuckets - 1);
    }
    if (hit) pair = S.xw[qpos];
  }
  return hit;
}

// Number of entries of the sorted p[lo .. hi), hi - lo <= 4 * kVecs, that are
// below x (or equal to it, kEqual), from 16-byte loads aligned to 4 bytes; up
// to 4 * kVecs entries from lo on are read, inside the workspace.  (Offsets
// are compared: lo + 7 wraps for the last positions of 2^32 - 1 edges.)
typedef uint32_t find4_t __attribute__((ext_vector_type(4), aligned(4)));
template <int kVecs, bool kEqual>
__device__ __forceinline__ uint32_t count_below(const uint32_t* p, uint32_t lo, uint32_t hi,
                                                uint32_t x) {
  find4_t v[kVecs];
#pragma unroll
  for (int k = 0; k < kVecs; ++k) v[k] = *reinterpret_cast<const find4_t*>(p + lo + 4 * k);
  uint32_t n = 0;
#pragma unroll
  for (int k = 0; k < kVecs; ++k)
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i)
      n += (4 * k + i < hi - lo) & (kEqual ? v[k][i] <= x : v[k][i] < x);
  return n;
}

// First position in the sorted DAG range [lo, hi) whose rank id is >= x
// (the entry x itself in a valid input; hi if every entry is below x).  The
// fence samples of the line starts inside the range pick the one 128-byte
// line of dag_col that holds the answer, and the halving ends inside it: a
// search of a long row reads its samples (one or two lines) and one line of
// dag_col, instead of a new line for each of its first halvings.  64 lanes
// search 64 rows, so every step is 64 line accesses, and what bounds the
// searches is their number: the last four samples and the last eight entries
// are counted out of one and two wide loads in place of two and three
// halvings (p-1 at R-MAT scale 20: 3.43 -> 3.37 ms, scale 24: 95.7 -> 94.7 ms;
// with the wide loads for the entries alone 3.40 and 95.2 ms).
__device__ __forceinline__ uint32_t dag_find(const TriArgs& a, uint32_t lo, uint32_t hi,
                                             uint32_t x) {
  static_assert(kFenceStep == 32, "line starts are multiples of 32 positions");
  // line starts 32q inside [lo, hi): q in [qa, qe)
  const uint32_t qa = (lo >> 5) + ((lo & 31u) != 0), qe = (hi >> 5) + ((hi & 31u) != 0);
  if (qa < qe) {
    uint32_t l = qa, h = qe;  // first q whose line starts above x
    while (h - l > 4) {
      const uint32_t mid = l + ((h - l) >> 1);
      if (a.fence[mid] <= x)
        l = mid + 1;
      else
        h = mid;
    }
    l += count_below<1, true>(a.fence, l, h, x);
    if (l > qa) lo = (l - 1) << 5;  // the line of the last start at or below x
    const uint64_t lend = (uint64_t)l << 5;
    if (lend < hi) hi = (uint32_t)lend;
  }
  while (hi - lo > 8) {
    const uint32_t mid = lo + ((hi - lo) >> 1);
    if (a.dag_col[mid] < x)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo + count_below<2, false>(a.dag_col, lo, hi, x);
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct TriCtx {
  TriArgs a;
  uint32_t* xcnt;    // general instantiation only: per-edge counts of the hashed range
  uint32_t* ie_cnt;  //   and of the batch's in-edges
  uint64_t* ie_key;  // Edge-Once instantiation only
  uint32_t* xmin;    // Edge-Once instantiation only
  uint32_t cap;   // out-list entries hashed per pass (<= kHashCap)
  int64_t j0;
  uint32_t D0;    // first DAG position of the hashed range
  uint32_t hlen;  // number of hashed entries
  uint32_t thr_last;  // the tile's graph: largest selected Philox word 0 (if
  bool thr_any;       //   any is), Philox key, first vertex
  uint32_t k0, k1, vb;
  uint32_t op;    // the tile's graph's operation
  bool eo_later;  // an Edge-Once pass after the first bids: eids are known, closed edges skipped
  bool eo_append; // an Edge-Once bidding pass that also lists the bidding triangles
  uint64_t wcur;  // Edge-Once list slots reserved by this wave: next free one
  uint32_t wleft; //   and how many are left (the same in every lane of the wave)
  uint32_t achunk;  // slots a wave reserves at a time
  uint64_t n_tri, n_sel;
};

// Empties the hash, the filter and the flags of the hashed entries.
template <class Smem>
__device__ __forceinline__ void tri_clear_hash(Smem& S) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int i = 0; i < kBuckets; i += kTB)
    S.bucket[i + tid] = make_uint4(kEmpty, kEmpty, kEmpty, kEmpty);
  reinterpret_cast<uint4*>(S.filt)[tid] = make_uint4(0u, 0u, 0u, 0u);
  reinterpret_cast<uint32_t*>(S.xflag)[tid] = 0;
}
static_assert(kBuckets % kTB == 0 && kFiltWords / 4 == kTB && kHashCap / 4 == kTB,
              "whole vectors per thread");

// Hash the out-list entries [D0, D0 + len) into the cleared hash.  A thread
// takes `per` consecutive entries (the fewest that cover the range), so that
// the row of each comes from a max-scan over the row starts in dpos (all rows
// of the tile; every row start is 0 for one row).
template <class Smem>
__device__ void tri_build_hash(TriCtx& C, Smem& S, uint32_t len, bool all_rows) {
  const uint32_t tid = threadIdx.x, wave = tid / kWave;
  const uint32_t per = (len + kTB - 1) / kTB, q0 = tid * per;
  uint32_t w[kHashPer], o[kHashPer], g[kHashPer];
#pragma unroll
  for (uint32_t i = 0; i < (uint32_t)kHashPer; ++i)
    w[i] = i < per && q0 + i < len ? C.a.dag_col[C.D0 + q0 + i] : 0u;
#pragma unroll
  for (uint32_t i = 0; i < (uint32_t)kHashPer; ++i)
    o[i] = i < per && q0 + i < len ? C.a.order[w[i]] : 0u;
  if (all_rows) {
    uint32_t m = 0;
#pragma unroll
    for (uint32_t i = 0; i < (uint32_t)kHashPer; ++i) {
      m = max(m, i < per && q0 + i < len ? S.u.dpos[q0 + i] : 0u);
      g[i] = m;
    }
    const uint32_t incl = wave_incl_max(m);
    if (lane_id() == kWave - 1) S.wsum[wave] = incl;
    uint32_t before = __shfl_up(incl, 1, kWave);
    if (lane_id() == 0) before = 0;
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < (uint32_t)kTW; ++i)
      if (i < wave) before = max(before, S.wsum[i]);
#pragma unroll
    for (uint32_t i = 0; i < (uint32_t)kHashPer; ++i) g[i] = max(g[i], before);
  } else {
#pragma unroll
    for (uint32_t i = 0; i < (uint32_t)kHashPer; ++i) g[i] = 0;
  }
  const bool skip_closed = C.eo_later;
#pragma unroll
  for (uint32_t i = 0; i < (uint32_t)kHashPer; ++i) {
    const uint32_t q = q0 + i;
    if (i >= per || q >= len) break;
    S.xw[q] = make_uint2(w[i], o[i] - C.vb);
    if (C.xmin) C.xmin[q] = 0xffffffffu;
    // counts exist only for Min-Count graphs: loaded for their selection
    // pass, zeroed for their counting pass (other operations never read them)
    if (C.xcnt) C.xcnt[q] = C.a.pass == 1 && C.op == SLIM_OP_MCTR ? C.a.tcount[C.D0 + q] : 0u;
    // Edge-Once rounds after the first pass: a closed edge {x,w} decides
    // every triangle on it, so it is left out of the hash
    if (skip_closed && bit_get(C.a.closed, C.D0 + q)) continue;
    const uint32_t h = hkey(w[i], hrow(g[i]));
    atomicOr(&S.filt[h >> 21], 0x80000000u >> (h & 31u));
    uint32_t* slots = reinterpret_cast<uint32_t*>(S.bucket);
    uint32_t at = (h >> (32 - kBucketBits)) * 4;  // slot by slot through the buckets
    while (atomicCAS(&slots[at], kEmpty, hslot(h) | q) != kEmpty) at = (at + 1) & (4 * kBuckets - 1);
  }
  C.hlen = len;
  __syncthreads();
}

// Marks (counting pass: counts) of the hashed range, behind the barrier that
// ends the scan; a thread reads the flags that it clears for the next range.
template <class Smem>
__device__ void tri_flush_xflags(TriCtx& C, Smem& S) {
  if (C.xcnt && C.a.pass == 0) {  // counting pass: add the (x,w) counts of the range
    for (uint32_t q = threadIdx.x; q < C.hlen; q += kTB) {
      const uint32_t v = C.xcnt[q];
      if (v) atomicAdd(C.a.tcount + C.D0 + q, v);
    }
  } else {
    for (uint32_t i = threadIdx.x; 4 * i < C.hlen; i += kTB) {
      const uint32_t v = reinterpret_cast<const uint32_t*>(S.xflag)[i];
      if (v == 0) continue;
#pragma unroll
      for (uint32_t t = 0; t < 4; ++t)
        if ((v >> (8 * t)) & 1u) mark_set(C.a.marks, C.D0 + 4 * i + t);
    }
  }
}

// Forward entries among tile entries [ia, ib): their edge is in out(x) of the
// entry's own row, so the DAG position comes from the hash (a miss means the
// entry lies in another pass of a split row).  nfw: forward entries of the tile.
template <class Smem>
__device__ void tri_forward_eids(TriCtx& C, Smem& S, uint32_t nfw, uint32_t ia, uint32_t ib,
                                 bool all_rows) {
  if (C.hlen == 0) return;
  for (uint32_t f = threadIdx.x; f < nfw; f += kTB) {
    const uint32_t i = S.bw[kTT - 1 - f];
    if (i < ia || i >= ib) continue;
    const uint64_t j = (uint64_t)C.j0 + i;
    const uint32_t w = C.a.rcol[j];
    uint32_t rs = 0, len = C.hlen;
    if (all_rows) {
      const uint32_t fs = C.a.fstart[S.srow[i]];
      rs = fs - C.D0;
      len = C.a.fstart[S.srow[i] + 1] - fs;
    }
    uint32_t qpos;
    uint2 pair;
    if (hfind(S, w, hkey(w, hrow(rs)), rs | (len << 16), qpos, pair)) C.a.eid[j] = C.D0 + qpos;
  }
}

// Marks the edge of triangle (y,x,w) that does not contain vertex `excl`.
// The marks of (y,x) and (x,w) are byte flags in LDS.
template <class Smem>
__device__ __forceinline__ void tri_mark(uint8_t* marks, Smem& S, uint32_t excl, uint32_t x,
                                         uint32_t w, uint32_t k, uint32_t qpos, uint32_t p_yw) {
  if (excl != x) {  // {y,x}, the in-edge, or {x,w}, position qpos of the hashed range
    uint8_t* f = excl == w ? S.ie_flag + k : S.xflag + qpos;
    *f = 1u;
  } else {  // edge {y,w}: a byte store (nothing waits on it)
    mark_set(marks, p_yw);
  }
}

// Edge-Once bid: lowers *p to key; the plain load skips the atomic when the
// edge already holds a smaller key (values only decrease within a pass).
__device__ __forceinline__ void eo_bid(uint64_t* p, uint64_t key) {
  if (key < __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    __hip_atomic_fetch_min(p, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A candidate record looked up: true if (y, x, w) is a triangle.
struct TriHit {
  uint32_t k, qpos, p_yw;  // in-edge of the batch, position of {x,w}, DAG position of {y,w}
  uint32_t y, x, w;        // local ids
};
template <class Smem>
__device__ __forceinline__ bool tri_lookup(const Smem& S, uint2 rec, uint32_t item0, TriHit& t) {
  t.k = rec.y >> kItemBits;
  const uint2 sc = S.ie_scan[t.k];
  const uint4 tr = S.ie_tri[t.k];
  const uint32_t item = (rec.y & ((1u << kItemBits) - 1u)) + item0;
  t.p_yw = sc.x + item;
  t.y = tr.y;
  t.x = tr.z;
  // items past the in-edge's end fill up its last quad
  uint2 pair;
  const bool hit = item < tr.x && hfind(S, rec.x, hkey(rec.x, sc.y), tr.w, t.qpos, pair);
  t.w = pair.y;
  return hit;
}

// Philox words of the id-sorted triple (local ids) under the tile's graph's
// key.  The key is made opaque here so that the round keys are scalar adds at
// the point of use, not twenty values kept in registers across the scan.
__device__ __forceinline__ uint4 tri_words(const TriCtx& C, uint32_t t0, uint32_t t1, uint32_t t2) {
  uint32_t k0 = C.k0, k1 = C.k1;
  asm volatile("" : "+s"(k0), "+s"(k1));
  return philox4(t0, t1, t2, 0u, k0, k1);
}

// Edge-Once drain of the stacked candidates q[0 .. cnt) (cnt <= 64): a
// selected triangle with no closed edge bids its per-edge keys.  In the
// bidding pass that starts the triangle list, every bidding triangle is
// also appended to the list (one counter atomic per wave).  Counts the
// triangles and the bidding ones.
template <class Smem>
__device__ __forceinline__ void tri_drain_eo(TriCtx& C, Smem& S, const uint2* q, uint32_t cnt,
                                             uint32_t item0, uint32_t& n_tri, uint32_t& n_sel) {
  const uint32_t lane = lane_id();
  bool app = false;
  uint4 ra = make_uint4(0u, 0u, 0u, 0u), rb = ra;
  TriHit t;
  if (lane < cnt && tri_lookup(S, q[lane], item0, t)) {
    ++n_tri;
    const uint32_t k = t.k, qpos = t.qpos, p_yw = t.p_yw;
    const uint32_t ly = t.y, lx = t.x, lw = t.w;
    uint32_t t0 = ly, t1 = lx, t2 = lw;
    sort3(t0, t1, t2);
    const uint4 wr = tri_words(C, t0, t1, t2);
    // the in-edge and the hashed entry are open (closed ones are neither
    // scanned nor hashed); {y,w} is read here
    const bool open = C.thr_any && wr.x <= C.thr_last && !(C.eo_later && bit_get(C.a.closed, p_yw));
    if (open) {
      // per-edge keys (word 2, third vertex): {y,x} -> w, {x,w} -> y, {y,w} -> x
      const uint64_t hi = (uint64_t)wr.z << 32;
      // the scan of an in-edge begins right after its own position
      const uint32_t e_yx = S.ie_scan[k].x + Smem::kQuad * S.ie_pre[k] - 1u, e_xw = C.D0 + qpos;
      const uint64_t k_yx = hi | lw, k_xw = hi | ly, k_yw = hi | lx;
      uint64_t* mk = C.a.minkey;
      const uint32_t kk = __umulhi(wr.y, 3u);  // edge kk of ({t0,t1}, {t0,t2}, {t1,t2})
      const uint32_t excl = kk == 0 ? t2 : (kk == 1 ? t1 : t0);
      atomicMin((unsigned long long*)&C.ie_key[k], (unsigned long long)k_yx);  // LDS
      // {x,w} lies in the hashed range: a bid whose priority word is above
      // the smallest one this pass has bid on the entry cannot hold the
      // minimum (that one went to the global key), so only the others bid
      if (wr.z <= atomicMin(&C.xmin[qpos], wr.z)) eo_bid(mk + e_xw, k_xw);
      eo_bid(mk + p_yw, k_yw);
      ++n_sel;
      app = true;
      ra = make_uint4(e_yx, e_xw, p_yw, excl == lw ? e_yx : (excl == ly ? e_xw : p_yw));
      rb = make_uint4(wr.z, lw, ly, lx);
    }
  }
  if (C.eo_append) {  // the same in every lane of the block
    // slots come from the wave's reserved run first; the rest from a new run
    // of max(rest, achunk) slots, taken with one atomic on the list counter
    const uint64_t mask = __ballot(app);
    if (mask) {
      const uint32_t n = __popcll(mask), r = __popcll(mask & lanemask_lt());
      const uint32_t take0 = n < C.wleft ? n : C.wleft;
      const uint64_t base0 = C.wcur;
      uint64_t base1 = 0;
      if (n > take0) {
        const uint32_t need = n - take0, run = need > C.achunk ? need : C.achunk;
        unsigned long long nb = 0;
        if (lane == 0) nb = atomicAdd((unsigned long long*)C.a.eo_list_cnt, (unsigned long long)run);
        base1 = __shfl(nb, 0, kWave);
        C.wcur = base1 + need;
        C.wleft = run - need;
      } else {
        C.wcur += n;
        C.wleft -= n;
      }
      const uint64_t idx = r < take0 ? base0 + r : base1 + (r - take0);
      if (app && idx < C.a.eo_cap) {
        C.a.eo_list[2 * idx] = ra;
        C.a.eo_list[2 * idx + 1] = rb;
      }
    }
  }
}

// Look up the stacked candidates q[0 .. cnt) (cnt <= 64), one per lane, and
// hash, select and mark the triangles among them (the counting pass: count
// them on their edges).  Counts the triangles and the selected ones.
template <int kMode, class Smem>
__device__ __forceinline__ void tri_drain(TriCtx& C, Smem* Sp, const uint2* q, uint32_t cnt,
                                          uint32_t item0, uint32_t& n_tri, uint32_t& n_sel) {
  Smem& S = *Sp;
  if constexpr (kMode == kModeEO) {
    tri_drain_eo(C, S, q, cnt, item0, n_tri, n_sel);
    return;
  }
  const uint32_t lane = lane_id();
  if (lane >= cnt) return;
  TriHit t;
  if (!tri_lookup(S, q[lane], item0, t)) return;
  if constexpr (kMode == kModeCount) {  // one more triangle on each of its three edges
    atomicAdd(&C.xcnt[t.qpos], 1u);
    atomicAdd(C.a.tcount + t.p_yw, 1u);
    // the hits of the first two in-edges add together: where most items are
    // triangles the lanes of an atomic each would wait in line for one word
    // (K_1500: 2.91 ms by lane, 2.10 so; R-MAT scale 20: 4.15 and 4.00)
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const uint32_t k0 = __builtin_amdgcn_readfirstlane(t.k);
      const uint64_t same = __builtin_amdgcn_ballot_w64(t.k == k0);
      if (t.k == k0) {
        if (lane == (uint32_t)__builtin_ctzll(same)) atomicAdd(&C.ie_cnt[k0], (uint32_t)__popcll(same));
        return;
      }
    }
    atomicAdd(&C.ie_cnt[t.k], 1u);
    return;
  }
  ++n_tri;
  const uint32_t ly = t.y, lx = t.x, lw = t.w;
  uint32_t t0 = ly, t1 = lx, t2 = lw;
  sort3(t0, t1, t2);
  const uint4 wr = tri_words(C, t0, t1, t2);
  const uint32_t w0 = wr.x, w1 = wr.y;
  if (!(C.thr_any && w0 <= C.thr_last)) return;
  ++n_sel;
  // edge e of ({t0,t1}, {t0,t2}, {t1,t2}) is the one without excl[e]
  const uint32_t excl[3] = {t2, t1, t0};
  const uint32_t kk = __umulhi(w1, 3u);
  if constexpr (kMode == kModePlain) {
    tri_mark(C.a.marks, S, kk == 0 ? t2 : (kk == 1 ? t1 : t0), lx, lw, t.k, t.qpos, t.p_yw);
  } else if (C.op == SLIM_OP_MCTR) {
    uint32_t n[3];
#pragma unroll
    for (int e = 0; e < 3; ++e)
      n[e] = excl[e] == lw ? C.ie_cnt[t.k]
                           : (excl[e] == ly ? C.xcnt[t.qpos] : C.a.tcount[t.p_yw]);
    const uint32_t tmin = min(n[0], min(n[1], n[2]));
    const uint32_t nt = (n[0] == tmin) + (n[1] == tmin) + (n[2] == tmin);
    uint32_t pick = __umulhi(w1, nt), e = 0;
    for (; e < 3; ++e) {
      if (n[e] != tmin) continue;
      if (pick == 0) break;
      --pick;
    }
    tri_mark(C.a.marks, S, excl[e], lx, lw, t.k, t.qpos, t.p_yw);
  } else {
#pragma unroll
    for (int e = 0; e < 3; ++e)
      if ((C.op == SLIM_OP_TR2) ? (uint32_t)e != kk : (uint32_t)e == kk)
        tri_mark(C.a.marks, S, excl[e], lx, lw, t.k, t.qpos, t.p_yw);
  }
}

// One window of a scan: kQuad consecutive items per lane, which sit at any
// position (a vector load aligned to 4 bytes).
template <int kQuad>
struct TriWin {
  typedef uint32_t vec __attribute__((ext_vector_type(kQuad), aligned(4)));
  uint32_t row, rec;  // row constant of the hash; (in-edge << kItemBits) | first item
  vec w;
};
template <>
struct TriWin<1> {
  struct vec {
    uint32_t v;
    __device__ uint32_t operator[](int) const { return v; }
  };
  uint32_t row, rec;
  vec w;
};

// Process the in-edges bw[b0, b1) of the tile against the current hash.
template <int kMode, class Smem>
__device__ void tri_batch(TriCtx& C, Smem& S, uint32_t b0, uint32_t b1, bool all_rows) {
  constexpr bool kGeneral = kMode == kModeGeneral, kCount = kMode == kModeCount;
  constexpr int kQuad = Smem::kQuad;
  using Win = TriWin<kQuad>;
  const int tid = threadIdx.x;
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t lane = lane_id();
  const uint32_t nin = b1 - b0;
  // ---- setup: one thread per in-edge (y,x); x is found in sorted out(y) by
  // binary search, and the items are the entries of out(y) after it
  uint32_t e = 0, beg = 0, len = 0, c = 0, r = 0, rs = 0, rlen = C.hlen;
  if ((uint32_t)tid < nin) {
    const uint32_t i = S.bw[b0 + tid];
    const uint64_t j = (uint64_t)C.j0 + i;
    r = S.srow[i];
    c = C.a.col[j];
    const uint32_t y = C.a.rcol[j];
    const uint32_t x = C.a.rank[r];
    const uint2 yr = C.a.dag_rng[y];
    const uint32_t fs = C.a.fstart[r], fe = C.a.fstart[r + 1];
    bool closed = false;
    if (C.eo_later) {  // found by the first Edge-Once pass
      e = C.a.eid[j];
      closed = bit_get(C.a.closed, e);
    } else {
      e = dag_find(C.a, yr.x, yr.y, x);  // dag_col[e] == x
      C.a.eid[j] = e;
    }
    // out(x) empty: no triangle, no scan (e == yr.y only for inputs that
    // break the CSR contract: then nothing is scanned either); a closed
    // in-edge of an Edge-Once round is not scanned
    beg = fe > fs && e < yr.y && !closed ? e + 1 : yr.y;
    len = yr.y - beg;
    if (all_rows) {
      rs = fs - C.D0;
      rlen = fe - fs;
    }
  }
  const uint32_t nq = (len + kQuad - 1) / kQuad;
  if (tid < Smem::kB) S.ie_flag[tid] = 0;
  if (C.ie_key && tid < Smem::kB) C.ie_key[tid] = ~0ull;
  if (tid < Smem::kM) S.mask[tid] = 0;
  // ---- the in-edges with items, in order: index kc, first quad pre
  const uint32_t incl = wave_incl_sum32(nq);
  const uint64_t some = __ballot(nq != 0);
  if (lane == kWave - 1) {
    S.wsum[w] = incl;
    S.wcnt[w] = __popcll(some);
  }
  __syncthreads();
  uint32_t pre = incl - nq, kc = __popcll(some & lanemask_lt()), W = 0, nk = 0;
#pragma unroll
  for (int i = 0; i < kTW; ++i) {
    if ((uint32_t)i < w) {
      pre += S.wsum[i];
      kc += S.wcnt[i];
    }
    W += S.wsum[i];
    nk += S.wcnt[i];
  }
  W = __builtin_amdgcn_readfirstlane(W);
  nk = __builtin_amdgcn_readfirstlane(nk);
  if (nq) {
    S.ie_scan[kc] = make_uint2(beg - kQuad * pre, hrow(rs));
    S.ie_tri[kc] = make_uint4(kQuad * pre + len, c - C.vb, r - C.vb, rs | (rlen << 16));
    S.ie_pre[kc] = pre;
    if (kGeneral) C.ie_cnt[kc] = C.op == SLIM_OP_MCTR ? C.a.tcount[e] : 0u;
    if (kCount) C.ie_cnt[kc] = 0u;
  }
  // ---- items: quads [s0, s0 + n) per pass of the mask, in windows of 64
  // (one quad per lane); wave w takes a contiguous run of windows.  The
  // in-edge of a lane's quad is the number of mask bits below the lane, added
  // to the count of the windows before.
  uint2* q = S.u.queue[w];
  uint32_t n_tri = 0, n_sel = 0;
  for (uint32_t s0 = 0; s0 < W; s0 += Smem::kM * kWave) {
    if (s0) {
      __syncthreads();
      if (tid < Smem::kM) S.mask[tid] = 0;
      __syncthreads();
    }
    if (nq && pre > s0 && pre - s0 <= (uint32_t)Smem::kM * kWave)
      atomicOr(reinterpret_cast<uint32_t*>(S.mask) + ((pre - s0 - 1) >> 5), 1u << ((pre - s0 - 1) & 31u));
    __syncthreads();
    const uint32_t n = W - s0 < (uint32_t)Smem::kM * kWave ? W - s0 : Smem::kM * kWave;
    const uint32_t nwin = (n + kWave - 1) / kWave;
    uint32_t wi = nwin * w / kTW;
    const uint32_t we = nwin * (w + 1) / kTW;
    if (wi >= we) continue;
    uint32_t kcur = 0;
    {  // in-edge of the run's first quad: last k with ie_pre[k] <= it
      const uint32_t first = s0 + wi * kWave;
      uint32_t lo = 0, hi = nk;
      while (hi - lo > 1) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        if (S.ie_pre[mid] <= first)
          lo = mid;
        else
          hi = mid;
      }
      kcur = lo;
    }
    // loads are issued without a branch, so that the wait for one window
    // leaves the next one's load in flight; a window past the run's end (at
    // most 2 * kDepth - 1 of them) is the next wave's or has no mask bits, so
    // that k is an in-edge of the batch, and it and the lanes past the last
    // quad read the first columns (items past the end fail the look-up's end
    // test)
    const uint32_t item0 = kQuad * s0;
    const uint32_t lim = kQuad * (n < we * kWave ? n : we * kWave);
    auto load = [&](uint32_t win, Win& x) {
      const uint2 m = reinterpret_cast<const uint2*>(S.mask)[win];
      const uint32_t k = __builtin_amdgcn_mbcnt_hi(m.y, __builtin_amdgcn_mbcnt_lo(m.x, kcur));
      kcur += __popc(m.x) + __popc(m.y);
      const uint2 sc = S.ie_scan[k];
      const uint32_t item = win * (kWave * kQuad) + lane * kQuad;
      x.row = sc.y;
      x.rec = (k << kItemBits) | item;
      const uint32_t p = item < lim ? sc.x + item + item0 : 0u;
      x.w = *reinterpret_cast<const typename Win::vec*>(C.a.dag_col + p);
    };
    uint32_t qcnt = 0;
    auto probe = [&](const Win& x) {
      bool cand[kQuad];
#pragma unroll
      for (int j = 0; j < kQuad; ++j) cand[j] = hfilter(S.filt, hkey(x.w[j], x.row));
#pragma unroll
      for (int j = 0; j < kQuad; ++j) {
        const uint64_t bal = __builtin_amdgcn_ballot_w64(cand[j]);
        if (bal == 0) continue;
        const uint32_t before = __builtin_amdgcn_mbcnt_hi(
            (uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
        if (cand[j]) q[qcnt + before] = make_uint2(x.w[j], x.rec + j);
        qcnt += __popcll(bal);
        if (qcnt >= (uint32_t)kWave) {
          qcnt -= kWave;
          wave_sync();
          tri_drain<kMode>(C, &S, q + qcnt, kWave, item0, n_tri, n_sel);
          wave_sync();
        }
      }
    };
    Win x[kDepth];
#pragma unroll
    for (int d = 0; d < kDepth; ++d) load(wi + d, x[d]);
    for (; wi < we; wi += kDepth) {
#pragma unroll
      for (int d = 0; d < kDepth; ++d) {
        if (wi + d < we) probe(x[d]);
        load(wi + d + kDepth, x[d]);
      }
    }
    if (qcnt) {
      wave_sync();
      tri_drain<kMode>(C, &S, q, qcnt, item0, n_tri, n_sel);
      wave_sync();
    }
  }
  C.n_tri += n_tri;
  C.n_sel += n_sel;
  __syncthreads();
  // ---- finish: (y,x) marks, or the (y,x) counts of the counting pass
  if (nq) {
    if (kCount) {
      if (C.ie_cnt[kc]) atomicAdd(C.a.tcount + e, C.ie_cnt[kc]);
    } else if (S.ie_flag[kc]) {
      mark_set(C.a.marks, e);
    }
    if (C.ie_key && C.ie_key[kc] != ~0ull)  // the batch's {y,x} bids
      eo_bid(C.a.minkey + e, C.ie_key[kc]);
  }
  __syncthreads();
}

// Adds the block's triangle and selection counts to graph g's counters.
// Edge-Once bids add the undecided triangles to the round's counter (and,
// in the first round, T and the selected count to the graph's counters);
// acceptance passes report nothing.
template <class Smem>
__device__ void tri_flush_counts(TriCtx& C, Smem& S, uint32_t g) {
  const int tid = threadIdx.x, w = tid / kWave;
  const uint64_t s0 = wave_sum64(C.n_tri), s1 = wave_sum64(C.n_sel);
  const bool first = C.a.pass < 2 || (C.a.pass == 2 && C.a.round == 1);
  if (lane_id() == 0) {
    S.red[0][w] = s0;
    S.red[1][w] = s1;
  }
  __syncthreads();
  if (tid == 0) {
    uint64_t t0 = 0, t1 = 0;
    for (int i = 0; i < kTW; ++i) {
      t0 += S.red[0][i];
      t1 += S.red[1][i];
    }
    if (first && t0) atomicAdd((unsigned long long*)&C.a.counters[2 * g], (unsigned long long)t0);
    if (first && t1)
      atomicAdd((unsigned long long*)&C.a.counters[2 * g + 1], (unsigned long long)t1);
    if (C.a.pass == 2 && t1)
      atomicAdd((unsigned long long*)&C.a.eo_und[C.a.round], (unsigned long long)t1);
  }
  __syncthreads();
  C.n_tri = 0;
  C.n_sel = 0;
}

// Persistent blocks take tiles in increasing order from a counter, so the
// graph of a block's tiles never decreases: counts are flushed when it
// changes and at the end.
template <int kMode>
__global__ __launch_bounds__(kTB) __attribute__((amdgpu_waves_per_eu(kWavesPerEU))) void k_triangles(
    TriArgs a, uint32_t* tile_ctr, uint32_t cap) {
  constexpr bool kGeneral = kMode == kModeGeneral, kEO = kMode == kModeEO;
  constexpr bool kCount = kMode == kModeCount;
  constexpr int kB = kBatchOf<kMode>, kM = kMaskOf<kMode>, kQuad = kQuadOf<kMode>;
  using Smem =
      std::conditional_t<kGeneral || kCount, TriSmemGeneral<kB, kM, kQuad>,
                         std::conditional_t<kEO, TriSmemEO<kB, kM, kQuad>, TriSmemPlain<kB, kM, kQuad>>>;
  static_assert(sizeof(Smem) <= kLdsPerBlock, "the resident blocks of a CU share its LDS");
  __shared__ __align__(16) Smem SS;
  TriSmem<kB, kM, kQuad>& S = SS.s;
  TriCtx C;
  C.a = a;
  if constexpr (kGeneral || kCount) {
    C.xcnt = SS.xcnt;
    C.ie_cnt = SS.ie_cnt;
  } else {
    C.xcnt = nullptr;
    C.ie_cnt = nullptr;
  }
  if constexpr (kEO) {
    C.ie_key = SS.ie_key;
    C.xmin = SS.xmin;
  } else {
    C.ie_key = nullptr;
    C.xmin = nullptr;
  }
  C.cap = cap;
  C.op = 0;
  C.n_tri = 0;
  C.n_sel = 0;
  C.thr_last = 0;
  C.thr_any = false;
  C.k0 = C.k1 = C.vb = 0;
  C.eo_later = kEO && a.round > 1;
  C.eo_append = false;
  // Edge-Once rounds end once a bidding pass finds no undecided triangle:
  // bids of round r stop if round r-1 had none, acceptance if round r has
  // none.  Once the undecided triangles may fit the list (round r-1 had at
  // most eo_list_try percent of its capacity), the bidding pass of round r also
  // lists them; if they fit, later rounds run on the list instead of listing
  // triangles again, else the list is dropped at the start of round r+1.
  if (kEO) {
    if (a.round > 1 && a.eo_und[a.round - 1] == 0) return;
    const uint32_t listed = a.eo_state[0];
    if (listed != 0 && listed < a.round) return;
    // every wave may leave up to achunk reserved slots unused (marked dead
    // at the end); they count against the capacity like the triangles
    const uint64_t waves = (uint64_t)gridDim.x * kTW;
    const uint64_t ch = a.eo_cap / (8 * waves);
    C.achunk = (uint32_t)(ch < 256 ? ch : 256);
    C.wcur = 0;
    C.wleft = 0;
    // (another block of this pass may already have recorded the round)
    C.eo_append = a.round >= 2 && (listed == 0 || listed == a.round) &&
                  a.eo_und[a.round - 1] * 100 <= (uint64_t)a.eo_list_try * a.eo_cap;
    if (C.eo_append && threadIdx.x == 0) a.eo_state[0] = a.round;
  }
  const int tid = threadIdx.x, w = tid / kWave;
  const uint32_t lane = lane_id();
  if (tid < 2 * kDepth) S.mask[kM + tid] = 0;
  const uint64_t ntiles = a.ntiles;
  uint32_t gcur = 0xffffffffu;
  bool clean = false;  // the LDS of the tile setup and the hash is cleared
  for (;;) {
    // ---- the next tile's index, and the clears of its setup (behind the
    // barrier that ended the last tile's scan)
    if (tid == 0) S.bcast[0] = atomicAdd(tile_ctr, 1u);
    if (!clean) {
      reinterpret_cast<uint2*>(S.srow)[tid] = make_uint2(0u, 0u);
      reinterpret_cast<uint4*>(S.u.dpos)[tid] = make_uint4(0u, 0u, 0u, 0u);
      tri_clear_hash(S);
      clean = true;
    }
    __syncthreads();
    const uint64_t t = __builtin_amdgcn_readfirstlane(S.bcast[0]);
    if (t >= ntiles) break;
    const TileRec R = a.recs[t];
    const uint32_t gop = a.gd[R.g].op;
    // graphs without edges and tiles of graphs that list no triangles are
    // skipped; the counting pass visits Min-Count graphs only, the Edge-Once
    // passes Edge-Once graphs only
    bool skip = R.span == 0 || !op_lists_triangles(gop) ||
                (kEO ? gop != SLIM_OP_EOTR : (kCount ? gop != SLIM_OP_MCTR : gop == SLIM_OP_EOTR));
    // Edge-Once: a tile lists the same triangles in every pass, so one that
    // found no undecided triangle in a bidding pass has none later either
    if (kEO && C.eo_later && a.eo_live[t] + 1u < a.round) skip = true;
    if (skip) {
      __syncthreads();  // the index has been read
      continue;
    }
    if (R.g != gcur) {
      // the counting pass reports no triangle or selection counts
      if (gcur != 0xffffffffu && !kCount) tri_flush_counts(C, S, gcur);
      gcur = R.g;
      const GDesc& G = a.gd[gcur];
      C.thr_any = G.thr != 0;
      C.thr_last = __builtin_amdgcn_readfirstlane((uint32_t)(G.thr - 1));
      C.k0 = __builtin_amdgcn_readfirstlane(G.k0);
      C.k1 = __builtin_amdgcn_readfirstlane(G.k1);
      C.vb = __builtin_amdgcn_readfirstlane((uint32_t)G.vb);
      C.op = __builtin_amdgcn_readfirstlane(G.op);
    }
    clean = false;
    const uint64_t sel0 = C.n_sel;
    const int64_t j0 = R.j0;
    const uint32_t span = R.span;
    C.j0 = j0;
    // ---- rows of the tile's entries (two consecutive ones per thread): row
    // starts into srow, then a max-scan.  Entries up to the first start
    // belong to the row before lo.
    uint32_t rc[2] = {0u, 0u};
#pragma unroll
    for (uint32_t i = 0; i < 2; ++i)
      if (2u * tid + i < span) rc[i] = a.rcol[j0 + 2 * tid + i];
    for (uint64_t r = R.lo + (uint64_t)tid; r < R.hi; r += kTB) {
      const int64_t b = a.row_off[r], e = a.row_off[r + 1];
      const int64_t s = b - j0;
      if (e > b && s >= 0 && s < kTT) S.srow[s] = r;
    }
    __syncthreads();
    uint32_t row[2];
    {
      const uint2 v = reinterpret_cast<const uint2*>(S.srow)[tid];
      const uint32_t m = max(v.x, v.y);
      const uint32_t incl = wave_incl_max(m);
      if (lane == kWave - 1) S.wmax[w] = incl;
      uint32_t before = __shfl_up(incl, 1, kWave);
      if (lane == 0) before = 0;
      __syncthreads();
      before = max(before, R.lo > 0 ? R.lo - 1 : 0u);
#pragma unroll
      for (int i = 0; i < kTW; ++i)
        if (i < w) before = max(before, S.wmax[i]);
      row[0] = max(before, v.x);
      row[1] = max(before, m);
      reinterpret_cast<uint2*>(S.srow)[tid] = make_uint2(row[0], row[1]);
    }
    // ---- backward entries (the in-edges of the tile's rows) and forward
    // entries, each in CSR order
    uint64_t mb[2], mf[2];
    bool bk[2], fw[2];
#pragma unroll
    for (uint32_t i = 0; i < 2; ++i) {
      bk[i] = fw[i] = false;
      if (2u * tid + i < span) {
        const uint32_t rr = a.rank[row[i]];
        bk[i] = rc[i] < rr;
        fw[i] = rc[i] > rr;
        if (2u * tid + i == 0) S.bcast[1] = row[i];
        if (2u * tid + i == span - 1) S.bcast[2] = row[i];
      }
      mb[i] = __ballot(bk[i]);
      mf[i] = __ballot(fw[i]);
    }
    if (lane == 0)
      S.wcnt[w] = (uint32_t)(__popcll(mb[0]) + __popcll(mb[1])) |
                  ((uint32_t)(__popcll(mf[0]) + __popcll(mf[1])) << 16);
    __syncthreads();
    uint32_t first = 0, all = 0;
#pragma unroll
    for (int i = 0; i < kTW; ++i) {
      if (i < w) first += S.wcnt[i];
      all += S.wcnt[i];
    }
    const uint32_t nbw = __builtin_amdgcn_readfirstlane(all & 0xffffu);
    const uint32_t nfw = __builtin_amdgcn_readfirstlane(all >> 16);
    const uint32_t r_lo = __builtin_amdgcn_readfirstlane(S.bcast[1]);
    const uint32_t r_hi = __builtin_amdgcn_readfirstlane(S.bcast[2]);
    {
      const uint64_t lt = lanemask_lt();
      uint32_t ib = (first & 0xffffu) + __popcll(mb[0] & lt) + __popcll(mb[1] & lt);
      uint32_t jf = kTT - 1 - ((first >> 16) + __popcll(mf[0] & lt) + __popcll(mf[1] & lt));
#pragma unroll
      for (uint32_t i = 0; i < 2; ++i) {
        if (bk[i]) S.bw[ib++] = (uint16_t)(2 * tid + i);
        if (fw[i]) S.bw[jf--] = (uint16_t)(2 * tid + i);
      }
    }
    const uint32_t D0 = a.fstart[r_lo], D1 = a.fstart[r_hi + 1];
    const bool all_rows = D1 - D0 <= C.cap;
    if (all_rows)  // ---- all rows of the tile share one hash: their starts
      for (uint64_t r = r_lo + (uint64_t)tid; r <= r_hi; r += kTB) {
        const uint32_t fs = a.fstart[r], fe = a.fstart[r + 1];
        if (fe > fs) S.u.dpos[fs - D0] = fs - D0;
      }
    __syncthreads();
    // ---- passes: the whole tile (all_rows), or each (row, out-list chunk)
    // with its in-edges and forward entries; the hashed range is [pD0, pD0+plen)
    uint32_t r = r_lo, cur = 0, cb = 0, xe = 0, bh = 0, ea = 0, eb = 0;
    bool row_open = false, done = false, fresh = true;
    while (!done) {
      uint32_t pD0, plen, pb0, pb1, pfa, pfb;
      if (all_rows) {
        pD0 = D0;
        plen = D1 - D0;
        pb0 = 0;
        pb1 = nbw;
        pfa = 0;
        pfb = span;
        done = true;
      } else {
        if (!row_open) {  // find the next row with entries in the tile
          bool found = false;
          for (; r <= r_hi; ++r) {
            const int64_t rb = a.row_off[r], re = a.row_off[r + 1];
            ea = (uint32_t)((rb > j0 ? rb : j0) - j0);
            eb = (uint32_t)((re < j0 + (int64_t)span ? re : j0 + (int64_t)span) - j0);
            if (eb <= ea) continue;
            if (tid == 0) {  // first bw index at or past the end of row r in the tile
              uint32_t lo = cur, hi = nbw;
              while (lo < hi) {
                const uint32_t mid = lo + ((hi - lo) >> 1);
                if ((uint32_t)S.bw[mid] < eb)
                  lo = mid + 1;
                else
                  hi = mid;
              }
              S.bcast[2] = lo;
            }
            __syncthreads();
            bh = S.bcast[2];
            __syncthreads();
            cb = a.fstart[r];
            xe = a.fstart[r + 1];
            if (xe > cb || bh > cur) {
              found = true;
              break;
            }
            cur = bh;
          }
          if (!found) break;
          row_open = true;
        }
        pD0 = cb;
        plen = xe - cb < C.cap ? xe - cb : C.cap;
        pb0 = cur;
        pb1 = bh;
        pfa = ea;
        pfb = eb;
        cb += C.cap;
        if (cb >= xe) {  // last chunk of this row
          row_open = false;
          cur = bh;
          ++r;
        }
      }
      C.D0 = pD0;
      if (!fresh) {  // a later pass of a tile: behind the barrier that ended the last scan
        tri_clear_hash(S);
        __syncthreads();
      }
      fresh = false;
      tri_build_hash(C, S, plen, all_rows);
      if (!C.eo_later) tri_forward_eids(C, S, nfw, pfa, pfb, all_rows);
      for (uint32_t b0 = pb0; b0 < pb1; b0 += kB)
        tri_batch<kMode>(C, S, b0, b0 + kB < pb1 ? b0 + kB : pb1, all_rows);
      if (pb0 >= pb1) __syncthreads();  // as a batch ends
      tri_flush_xflags(C, S);
    }
    if (kEO) {  // record the round in which the tile still bid
      if (tid == 0) S.bcast[3] = 0;
      __syncthreads();
      if (C.n_sel != sel0) S.bcast[3] = 1;
      __syncthreads();
      if (tid == 0 && S.bcast[3]) a.eo_live[t] = a.round;
    }
  }
  if (gcur != 0xffffffffu && !kCount) tri_flush_counts(C, S, gcur);
  if (kEO && C.eo_append)  // the wave's unused reserved slots become dead records
    for (uint32_t i = lane; i < C.wleft; i += kWave)
      if (C.wcur + i < a.eo_cap)
        reinterpret_cast<uint32_t*>(a.eo_list + 2 * (C.wcur + i))[0] = kDead;
}

// ---- Edge-Once rounds on the triangle lists: records {e_yx, e_xw, e_yw,
// e_del} {word 2, third vertex of each of the three edges}.  In list 0 a
// reserved slot that stayed unused has e_yx = kDead.  Round r after the
// listing round L bids from list (r - L - 1) mod 2 and copies each triangle
// that bids (none of its edges closed) into the other list; a triangle whose
// edge closed is decided and dropped, so each round reads only the last
// round's bidders.
constexpr int kListBlock = 256;

// The listing round's bidders did not fit the list (the slots taken,
// unused reserved ones included, pass its capacity).
__device__ __forceinline__ bool eo_list_overflow(const TriArgs& a) {
  return a.eo_list_cnt[0] > a.eo_cap;
}

// Bids on the list start the round after the listing round, acceptance on
// the list in the listing round itself (unless the list overflowed).
__device__ __forceinline__ bool eo_listed_round(const TriArgs& a, bool accept) {
  const uint32_t listed = a.eo_state[0];
  return listed != 0 &&
         (listed < a.round || (accept && listed == a.round && !eo_list_overflow(a)));
}

// Start of round a.round.  A list that the previous round started but
// overflowed is dropped (that round accepted by the edges).  Then the bids are
// reset: through the records of the list that this round bids from, where its
// previous bidders are few (all of them bid on their three edges; a dead slot
// of the listing round's list bid nowhere), else by a sweep over the edges.
// From the second round on, the sweep closes every edge that no undecided
// triangle bid on in the previous round: every selected triangle on it is
// decided (every edge of a listed triangle got a bid, so the list path has
// nothing to close).  One launch, where the drop, the two ways to reset and
// the tile counter were four: 16 rounds of empty launches were most of a
// small graph's call.
__global__ __launch_bounds__(kListBlock) void k_eo_begin(TriArgs a, uint64_t m, uint32_t* tile_ctr) {
  const bool one = blockIdx.x == 0 && threadIdx.x == 0;
  if (one) *tile_ctr = 0;
  // the first thread may drop the list while others look: it writes the state
  // before the count, they read the count before the state, so whoever misses
  // the overflow sees the state already dropped (both words are read past the
  // caches, the first one awaited before the second; an acquire at device
  // scope would also empty the caches once per wave: 4.1 ms instead of 0.58
  // for a graph of 2e5 vertices)
  const uint64_t cnt0 = __hip_atomic_load(&a.eo_list_cnt[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  uint32_t listed = __hip_atomic_load(&a.eo_state[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (listed != 0 && listed + 1 == a.round && cnt0 > a.eo_cap) {
    if (one) {
      __hip_atomic_store(&a.eo_state[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&a.eo_list_cnt[1], (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&a.eo_list_cnt[0], (uint64_t)0, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
    listed = 0;
  }
  if (a.round > 1 && a.eo_und[a.round - 1] == 0) return;  // the rounds have ended
  if (listed != 0 && listed < a.round) {
    const uint32_t src = (a.round - listed - 1) & 1u;
    uint64_t n = a.eo_list_cnt[src];
    if (n <= kEoListClearMax) {
      if (n > a.eo_cap) n = a.eo_cap;
      const uint4* list = a.eo_list + (uint64_t)src * 2 * a.eo_cap;
      for (uint64_t i = blockIdx.x * (uint64_t)kListBlock + threadIdx.x; i < n;
           i += (uint64_t)gridDim.x * kListBlock) {
        const uint4 r0 = list[2 * i];
        if (r0.x == kDead) continue;
        a.minkey[r0.x] = ~0ull;
        a.minkey[r0.y] = ~0ull;
        a.minkey[r0.z] = ~0ull;
      }
      return;
    }
  }
  // a wave takes 64 edges, so the two bitmap words of its chunk are its own
  const uint32_t lane = lane_id();
  const uint64_t waves = (uint64_t)gridDim.x * (kListBlock / kWave);
  for (uint64_t c = blockIdx.x * (uint64_t)(kListBlock / kWave) + threadIdx.x / kWave;
       c * kWave < m; c += waves) {
    const uint64_t i = c * kWave + lane;
    bool dead = false;
    if (i < m) {
      dead = a.round > 1 && a.minkey[i] == ~0ull;
      a.minkey[i] = ~0ull;
    }
    const uint64_t bal = __ballot(dead);
    if (lane == 0 && bal) {
      a.closed[2 * c] |= (uint32_t)bal;
      a.closed[2 * c + 1] |= (uint32_t)(bal >> 32);
    }
  }
}

// Records a wave takes at a time, at most: it counts the ones that will bid,
// reserves that many slots of the other list with one atomic, then bids and
// copies them (one atomic per 64 records on the shared counter serialized the
// kernel).  A short list is spread over the waves, 64 records at least: a
// chain of 16 steps took 65 us for a few thousand records.
constexpr uint32_t kListSpan = 16 * kWave;

__device__ __forceinline__ bool eo_list_live(const TriArgs& a, const uint4& r0) {
  return r0.x != kDead && !bit_get(a.closed, r0.x) && !bit_get(a.closed, r0.y) &&
         !bit_get(a.closed, r0.z);
}

__global__ __launch_bounds__(kListBlock) void k_eo_list_bid(TriArgs a) {
  if (!eo_listed_round(a, false) || a.eo_und[a.round - 1] == 0) return;
  __shared__ uint64_t red[kListBlock / kWave];
  const uint32_t src = (a.round - a.eo_state[0] - 1) & 1u, dst = src ^ 1u;
  const uint4* from = a.eo_list + (uint64_t)src * 2 * a.eo_cap;
  uint4* to = a.eo_list + (uint64_t)dst * 2 * a.eo_cap;
  uint64_t n = a.eo_list_cnt[src];
  if (n > a.eo_cap) n = a.eo_cap;
  const uint32_t lane = lane_id();
  const uint64_t waves = (uint64_t)gridDim.x * (kListBlock / kWave);
  uint64_t und = 0;
  const uint64_t share = (n / waves + kWave - 1) / kWave * kWave;
  const uint64_t span = share < kWave ? kWave : share < kListSpan ? share : kListSpan;
  for (uint64_t b = (blockIdx.x * (uint64_t)(kListBlock / kWave) + threadIdx.x / kWave) * span;
       b < n; b += waves * span) {
    const uint64_t e = b + span < n ? b + span : n;
    uint64_t cnt = 0;
    for (uint64_t i = b + lane; i < e; i += kWave) cnt += eo_list_live(a, from[2 * i]);
    cnt = wave_sum64(cnt);
    if (cnt == 0) continue;
    unsigned long long base = 0;
    if (lane == 0) base = atomicAdd((unsigned long long*)&a.eo_list_cnt[dst], (unsigned long long)cnt);
    base = __shfl(base, 0, kWave);
    // the same records pass the same test again (this kernel changes no
    // closed bit), so exactly cnt slots from base are written; the first
    // lane has the lowest index, so it is in every iteration another lane is
    for (uint64_t i = b + lane; i < e; i += kWave) {
      const uint4 r0 = from[2 * i];
      const bool live = eo_list_live(a, r0);
      const uint64_t mask = __ballot(live);
      if (live) {
        const uint4 r1 = from[2 * i + 1];
        const uint64_t hi = (uint64_t)r1.x << 32;
        eo_bid(a.minkey + r0.x, hi | r1.y);
        eo_bid(a.minkey + r0.y, hi | r1.z);
        eo_bid(a.minkey + r0.z, hi | r1.w);
        ++und;
        const uint64_t j = base + __popcll(mask & lanemask_lt());
        if (j < a.eo_cap) {  // j < n <= eo_cap: at most every source record bids
          to[2 * j] = r0;
          to[2 * j + 1] = r1;
        }
      }
      base += __popcll(mask);
    }
  }
  const uint64_t t = wave_sum64(und);
  if (lane == 0) red[threadIdx.x / kWave] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t s = 0;
    for (int i = 0; i < kListBlock / kWave; ++i) s += red[i];
    if (s) atomicAdd((unsigned long long*)&a.eo_und[a.round], (unsigned long long)s);
  }
}

// Acceptance on the list.
__device__ __forceinline__ void eo_accept_list(const TriArgs& a) {
  const uint32_t listed = a.eo_state[0];
  // the list this round's bids came from has been read in full: clear its
  // count for the next round, which copies into it
  const uint32_t src = (a.round - listed - 1) & 1u;
  if (a.round > listed && blockIdx.x == 0 && threadIdx.x == 0) a.eo_list_cnt[src] = 0;
  if (a.eo_und[a.round] == 0) return;
  const uint32_t cur = a.round == listed ? 0u : src ^ 1u;
  const uint4* list = a.eo_list + (uint64_t)cur * 2 * a.eo_cap;
  uint64_t n = a.eo_list_cnt[cur];
  if (n > a.eo_cap) n = a.eo_cap;
  for (uint64_t i = blockIdx.x * (uint64_t)kListBlock + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * kListBlock) {
    const uint4 r0 = list[2 * i];
    if (r0.x == kDead) continue;
    const uint4 r1 = list[2 * i + 1];
    const uint64_t hi = (uint64_t)r1.x << 32;
    if (a.minkey[r0.x] != (hi | r1.y) || a.minkey[r0.y] != (hi | r1.z) ||
        a.minkey[r0.z] != (hi | r1.w))
      continue;
    bit_set(a.closed, r0.x);
    bit_set(a.closed, r0.y);
    bit_set(a.closed, r0.z);
    mark_set(a.marks, r0.w);
  }
}

// Acceptance of an Edge-Once round without a list: the key on DAG edge
// {a,b} (a's row) names its holder triangle {a,b,w} by the third vertex w.
// The edge facing the holder's largest id checks the holder's keys on the
// other two edges (binary searches in the DAG rows of their lower-ranked
// ends); if it holds all three minima the triangle is considered: its three
// edges close and its drawn edge k is marked.  A wave takes 64 consecutive
// vertices, whose DAG rows are one contiguous range: the lanes stride over
// it (coalesced key reads) and find each position's row among the 64 row
// starts by a search over the lanes.
__device__ __forceinline__ uint32_t dag_pos(const TriArgs& a, uint32_t ru, uint32_t rv) {
  const uint32_t lo_r = ru < rv ? ru : rv, hi_r = ru < rv ? rv : ru;
  const uint2 rg = a.dag_rng[lo_r];
  const uint32_t lo = dag_find(a, rg.x, rg.y, hi_r);
  return lo < rg.y && a.dag_col[lo] == hi_r ? lo : kDead;
}

__device__ __forceinline__ void eo_accept_edges(const TriArgs& a, uint64_t n) {
  if (a.eo_und[a.round] == 0) return;
  const uint32_t lane = lane_id();
  const uint64_t waves = (uint64_t)gridDim.x * (kListBlock / kWave);
  for (uint64_t g = blockIdx.x * (uint64_t)(kListBlock / kWave) + threadIdx.x / kWave;
       g * kWave < n; g += waves) {
    const uint64_t v0 = g * kWave;
    const uint64_t vend = v0 + kWave < n ? v0 + kWave : n;
    const uint32_t pend = a.fstart[vend];
    const uint32_t fs = v0 + lane < vend ? a.fstart[v0 + lane] : pend;  // row start per lane
    const uint32_t pbeg = __shfl(fs, 0, kWave);
    // 64-bit positions: with m near 2^32 a 32-bit base + 64 could wrap
    for (uint64_t base = pbeg; base < pend; base += kWave) {
      const uint64_t p = base + lane;
      uint32_t own = 0;  // last lane whose row starts at or before p
#pragma unroll
      for (uint32_t step = kWave / 2; step > 0; step >>= 1) {
        const uint32_t cand = own + step;
        if (__shfl(fs, (int)cand, kWave) <= p) own = cand;
      }
      if (p >= pend) continue;
      const uint32_t pos = (uint32_t)p;  // < pend <= 2^32 - 1
      const uint64_t mk = a.minkey[pos];
      if (mk == ~0ull) continue;
      const uint32_t v = (uint32_t)(v0 + own);
      uint32_t lo = 0, hi = a.gcount;  // the vertex's graph: last with vb <= v
      while (hi - lo > 1) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        if (a.gd[mid].vb <= v)
          lo = mid;
        else
          hi = mid;
      }
      const GDesc& G = a.gd[lo];
      const uint32_t vb = (uint32_t)G.vb;
      const uint32_t rb = a.dag_col[pos];
      const uint32_t la = v - vb, lb = a.order[rb] - vb, lw = (uint32_t)mk;
      if (!(lw > la && lw > lb)) continue;  // the edge facing the largest id decides
      const uint64_t hk = mk & 0xffffffff00000000ull;
      const uint32_t rw = a.rank[vb + lw];
      const uint32_t p_aw = dag_pos(a, a.rank[v], rw), p_bw = dag_pos(a, rb, rw);
      if (p_aw == kDead || p_bw == kDead) continue;  // only for inputs breaking the contract
      if (a.minkey[p_aw] != (hk | lb) || a.minkey[p_bw] != (hk | la)) continue;
      // considered: edge k of ({t0,t1}, {t0,t2}, {t1,t2}), t2 = lw the largest
      const uint32_t t0 = la < lb ? la : lb, t1 = la < lb ? lb : la;
      const uint4 wr = philox4(t0, t1, lw, 0u, G.k0, G.k1);
      const uint32_t kk = __umulhi(wr.y, 3u);
      const uint32_t p_t0w = la < lb ? p_aw : p_bw, p_t1w = la < lb ? p_bw : p_aw;
      bit_set(a.closed, pos);
      bit_set(a.closed, p_aw);
      bit_set(a.closed, p_bw);
      mark_set(a.marks, kk == 0 ? pos : (kk == 1 ? p_t0w : p_t1w));
    }
  }
}

__global__ __launch_bounds__(kListBlock) void k_eo_accept(TriArgs a, uint64_t n) {
  if (eo_listed_round(a, true))
    eo_accept_list(a);
  else
    eo_accept_edges(a, n);
}

// Blocks for `items` items, one per thread, at most eight per CU.
static unsigned eo_blocks(uint64_t items, int num_cu) {
  const uint64_t most = num_cu > 0 ? (uint64_t)num_cu * 8 : 2048, b = (items + kListBlock - 1) / kListBlock;
  return (unsigned)(b < 1 ? 1 : b < most ? b : most);
}

void eo_begin(const TriArgs& a, uint64_t m, uint32_t* tile_ctr, int num_cu, hipStream_t s) {
  hipLaunchKernelGGL(k_eo_begin, dim3(eo_blocks(m, 4 * num_cu)), dim3(kListBlock), 0, s, a, m, tile_ctr);
}

void eo_list_bids(const TriArgs& a, uint64_t m, int num_cu, hipStream_t s) {
  hipLaunchKernelGGL(k_eo_list_bid, dim3(eo_blocks(m, num_cu)), dim3(kListBlock), 0, s, a);
}

void eo_accept(const TriArgs& a, uint64_t m, uint64_t n, int num_cu, hipStream_t s) {
  hipLaunchKernelGGL(k_eo_accept, dim3(eo_blocks(m > n ? m : n, num_cu)), dim3(kListBlock), 0, s, a, n);
}

uint64_t tri_tile_max() { return kTT; }

void triangles(const TriArgs& a, int mode, uint32_t* tile_ctr, int num_cu,
               int blocks_per_cu, int chunk, hipStream_t s) {
  uint64_t blocks = (uint64_t)num_cu * blocks_per_cu;
  if (blocks > a.ntiles) blocks = a.ntiles;
  if (blocks < 1) blocks = 1;
  uint32_t cap = (uint32_t)chunk;
  if (cap > (uint32_t)kHashCap) cap = kHashCap;
  if (mode == kModeGeneral)
    hipLaunchKernelGGL(k_triangles<kModeGeneral>, dim3((unsigned)blocks), dim3(kTB), 0, s, a,
                       tile_ctr, cap);
  else if (mode == kModeCount)
    hipLaunchKernelGGL(k_triangles<kModeCount>, dim3((unsigned)blocks), dim3(kTB), 0, s, a,
                       tile_ctr, cap);
  else if (mode == kModeEO)
    hipLaunchKernelGGL(k_triangles<kModeEO>, dim3((unsigned)blocks), dim3(kTB), 0, s, a,
                       tile_ctr, cap);
  else
    hipLaunchKernelGGL(k_triangles<kModePlain>, dim3((unsigned)blocks), dim3(kTB), 0, s, a,
                       tile_ctr, cap);
}

}  // namespace slim
