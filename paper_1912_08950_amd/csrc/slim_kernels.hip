// HIP kernels of libslim (gfx950): graph-set tiles and gather, degree-rank
// relabelling, DAG orientation, CSR compaction and per-graph stats.
//
// Data layout (all in HBM, caller-provided workspace), over the union CSR of
// the set (n vertices, nnz entries, m = nnz/2 edges):
//   rank[n], order[n]   union id -> rank id and back; rank order = (degree, id)
//   rcol[nnz]           rank id of every CSR column (streamed by the orientation)
//   dag_col[m]          rank ids of the higher-ranked neighbours, rows laid
//                       out in union-id row order (a stream compaction of CSR)
//   dag_rng[n]          (begin, end) of row x of the DAG, indexed by rank id
//   eid[nnz]            for every CSR entry of a TR graph, the DAG position of its edge
//   marks[m]            deletion marks over DAG positions, one byte per edge
//                       (set by the triangle kernels with byte stores)
//   del[m/32]           the same marks packed into a bitmap for the compaction
//   minkey[m], closed[m/32]  Edge-Once bids and closed edges over DAG positions
#include "slim_internal.h"

namespace slim {

// ------------------------------------------------------------------ fills
__global__ void k_fill_u32(uint32_t* p, uint64_t len, uint32_t v) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < len;
       i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

__global__ void k_fill_i64(int64_t* p, uint64_t len, int64_t v) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < len;
       i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

static unsigned grid_for(uint64_t len, unsigned cap = 65536) {
  uint64_t b = (len + kBlock - 1) / kBlock;
  if (b < 1) b = 1;
  return (unsigned)(b < cap ? b : cap);
}

void fill_u32(uint32_t* p, uint64_t len, uint32_t v, hipStream_t s) {
  if (len) hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(len)), dim3(kBlock), 0, s, p, len, v);
}

void fill_i64(int64_t* p, uint64_t len, int64_t v, hipStream_t s) {
  if (len) hipLaunchKernelGGL(k_fill_i64, dim3(grid_for(len)), dim3(kBlock), 0, s, p, len, v);
}

// --------------------------------------------------------- deletion marks
// Word i of the bitmap gets bit b set iff byte 32i + b of the marks is set;
// each thread reads its 32 bytes as two uint4.
__global__ __launch_bounds__(kBlock) void k_pack_marks(const uint8_t* marks, uint32_t* del,
                                                       uint64_t m) {
  const uint64_t words = (m + 31) / 32;
  for (uint64_t i = blockIdx.x * (uint64_t)kBlock + threadIdx.x; i < words;
       i += (uint64_t)gridDim.x * kBlock) {
    uint32_t v = 0;
    if (32 * i + 32 <= m) {
      const uint4* q = reinterpret_cast<const uint4*>(marks + 32 * i);
      const uint4 a = q[0], b = q[1];
      const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
      for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if ((w[k] >> (8 * t)) & 0xffu) v |= 1u << (4 * k + t);
    } else {
      for (uint64_t e = 32 * i; e < m; ++e)
        if (marks[e]) v |= 1u << (e - 32 * i);
    }
    del[i] = v;
  }
}

void pack_marks(const uint8_t* marks, uint32_t* del, uint64_t m, hipStream_t s) {
  if (m) hipLaunchKernelGGL(k_pack_marks, dim3(grid_for((m + 31) / 32)), dim3(kBlock), 0, s, marks,
                            del, m);
}

// ------------------------------------------------------------------- scan
// Exclusive prefix sum of TI[len] into uint64[len+1] (out[len] = total):
// per-block reduce, recursive scan of the block sums, per-block apply.
constexpr int kScanItems = 8;
constexpr int kScanTile = kBlock * kScanItems;

__device__ __forceinline__ uint64_t block_excl_sum64(uint64_t v, uint64_t* total,
                                                     uint64_t* lds /*[kWavesPerBlock]*/) {
  const int w = threadIdx.x / kWave;
  uint64_t incl = wave_incl_sum64(v);
  if (lane_id() == kWave - 1) lds[w] = incl;
  __syncthreads();
  uint64_t before = 0, all = 0;
#pragma unroll
  for (int i = 0; i < kWavesPerBlock; ++i) {
    if (i < w) before += lds[i];
    all += lds[i];
  }
  __syncthreads();
  *total = all;
  return before + incl - v;
}

template <typename TI>
__global__ void k_scan_reduce(const TI* in, uint64_t len, uint64_t* bsum) {
  __shared__ uint64_t lds[kWavesPerBlock];
  const uint64_t base = (uint64_t)blockIdx.x * kScanTile;
  uint64_t s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    uint64_t i = base + (uint64_t)k * kBlock + threadIdx.x;
    if (i < len) s += (uint64_t)in[i];
  }
  uint64_t total;
  block_excl_sum64(s, &total, lds);
  if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

template <typename TI>
__global__ void k_scan_apply(const TI* in, uint64_t len, const uint64_t* bbase, uint64_t* out) {
  __shared__ uint64_t lds[kWavesPerBlock];
  const uint64_t base = (uint64_t)blockIdx.x * kScanTile + (uint64_t)threadIdx.x * kScanItems;
  uint64_t v[kScanItems];
  uint64_t s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    uint64_t i = base + k;
    v[k] = i < len ? (uint64_t)in[i] : 0;
    s += v[k];
  }
  uint64_t total;
  uint64_t run = block_excl_sum64(s, &total, lds) + (bbase ? bbase[blockIdx.x] : 0);
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    uint64_t i = base + k;
    if (i < len) out[i] = run;
    run += v[k];
    if (i + 1 == len) out[len] = run;
  }
}

static uint64_t scan_blocks(uint64_t len) { return (len + kScanTile - 1) / kScanTile; }

uint64_t scan_tmp_elems(uint64_t len) {
  uint64_t nb = scan_blocks(len);
  if (nb <= 1) return 0;
  return 2 * nb + 2 + scan_tmp_elems(nb);
}

template <typename TI>
void scan_excl(const TI* in, uint64_t len, uint64_t* out, uint64_t* tmp, hipStream_t s) {
  if (len == 0) {
    fill_i64(reinterpret_cast<int64_t*>(out), 1, 0, s);
    return;
  }
  uint64_t nb = scan_blocks(len);
  if (nb == 1) {
    hipLaunchKernelGGL(k_scan_apply<TI>, dim3(1), dim3(kBlock), 0, s, in, len,
                       (const uint64_t*)nullptr, out);
    return;
  }
  uint64_t* bsum = tmp;
  uint64_t* bbase = tmp + nb + 1;
  hipLaunchKernelGGL(k_scan_reduce<TI>, dim3((unsigned)nb), dim3(kBlock), 0, s, in, len, bsum);
  scan_excl<uint64_t>(bsum, nb, bbase, tmp + 2 * nb + 2, s);
  hipLaunchKernelGGL(k_scan_apply<TI>, dim3((unsigned)nb), dim3(kBlock), 0, s, in, len,
                     (const uint64_t*)bbase, out);
}

template void scan_excl<uint32_t>(const uint32_t*, uint64_t, uint64_t*, uint64_t*, hipStream_t);
template void scan_excl<uint64_t>(const uint64_t*, uint64_t, uint64_t*, uint64_t*, hipStream_t);

// ------------------------------------------------------- degree ranking
// Vertices are ranked by degree, those of equal degree by id (a wave takes 64
// ids at a time in their order, and the LDS serves the lanes of one atomic in
// theirs).  Any total order finds the same triangles, but the scan items depend
// on it: where degrees are tied or close and ids follow the graph's parts, this
// order points every edge the same way and leaves nothing to scan (K_4000,4000,
// p-1: 15.9 ms with ties in any order, 1.9 so; K_3000,2990 with degrees within
// 1/64 in any order too: 4.5 and 1.3).
//
// A counting sort: degree classes, exact below 1024, then 64 per doubling; a
// block takes consecutive ids and counts them by class (in the setup), the
// counts of each class are summed up over the blocks, the block hands out the
// places in the order of its ids, and a last launch orders the classes that
// hold several degrees.  Two passes over the offsets and four launches, the
// setup among them (R-MAT scale 20: k_class_sum 5 us, k_rank 16, k_rank_wide 7;
// 90001 vertices: 5, 11 and 5; three 8-bit passes of a stable radix sort took
// 17 launches and 130 us at scale 20); a small graph is one block's work.
constexpr uint32_t kDegExact = 1024, kDegExactLog = 10, kDegFine = 64;
constexpr uint32_t kDegClasses = kDegExact + (32 - kDegExactLog) * kDegFine;
constexpr uint32_t kRankBlocks = 1024;    // most blocks of the histogram
constexpr uint32_t kFineBins = 4096;      // degrees of a class that are counted in LDS

__host__ __device__ inline uint32_t deg_class(uint32_t d) {
  if (d < kDegExact) return d;
  const uint32_t e = 31 - __builtin_clz(d);
  return kDegExact + (e - kDegExactLog) * kDegFine + ((d >> (e - 6)) & (kDegFine - 1));
}

__device__ __forceinline__ uint32_t degree_of(const int64_t* row_off, uint64_t v) {
  return (uint32_t)(row_off[v + 1] - row_off[v]);
}

// Exclusive sum of cls[0 .. n) in LDS, n <= kMax, in place, by one block.
template <uint32_t kMax>
__device__ void class_scan(uint32_t* cls, uint32_t n, uint32_t* wtot) {
  constexpr uint32_t kPer = (kMax + kBlock - 1) / kBlock;
  const uint32_t t = threadIdx.x, w = t / kWave;
  uint32_t v[kPer], s = 0;
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i) {
    const uint32_t k = t * kPer + i;
    v[i] = k < n ? cls[k] : 0u;
    s += v[i];
  }
  const uint32_t incl = wave_incl_sum32(s);
  if (lane_id() == kWave - 1) wtot[w] = incl;
  __syncthreads();
  uint32_t run = incl - s;
  for (uint32_t i = 0; i < w; ++i) run += wtot[i];
#pragma unroll
  for (uint32_t i = 0; i < kPer; ++i) {
    const uint32_t k = t * kPer + i;
    if (k < n) cls[k] = run;
    run += v[i];
  }
  __syncthreads();
}

// The ranks of a graph of n <= kRankSmall vertices, by one block: every degree
// is a class of its own, every wave takes a run of ids.  bin[i][d] has the
// counts, then the next places, of waves 2i (low half) and 2i + 1 in degree d.
constexpr uint32_t kSmallBins = (uint32_t)kRankSmall;
__device__ void rank_small(const int64_t* row_off, uint32_t n, uint32_t* order, uint32_t* rank,
                           uint32_t (&bin)[2][kSmallBins], uint32_t* wtot) {
  static_assert(kWavesPerBlock == 4 && kSmallBins < (1u << 16), "two waves' places per word");
  constexpr uint32_t kSteps = kSmallBins / kBlock;
  const uint32_t t = threadIdx.x, w = t / kWave, lane = lane_id();
  const uint32_t steps = (n + kBlock - 1) / kBlock, v0 = w * steps * kWave + lane;
  uint32_t d[kSteps];
#pragma unroll
  for (uint32_t k = 0; k < kSteps; ++k) {
    const uint32_t v = v0 + k * kWave;
    d[k] = k < steps && v < n ? min(degree_of(row_off, v), kSmallBins - 1) : kSmallBins;
  }
#pragma unroll
  for (uint32_t k = 0; k < 2 * kSteps; ++k) (&bin[0][0])[k * kBlock + t] = 0;
  __syncthreads();
  uint32_t* mine = bin[w / 2];
  const uint32_t shift = 16 * (w & 1);
#pragma unroll
  for (uint32_t k = 0; k < kSteps; ++k)
    if (d[k] < kSmallBins) atomicAdd(&mine[d[k]], 1u << shift);
  __syncthreads();
  uint32_t c0[kSteps], c1[kSteps], sum = 0;
#pragma unroll
  for (uint32_t k = 0; k < kSteps; ++k) {
    c0[k] = bin[0][t * kSteps + k];
    c1[k] = bin[1][t * kSteps + k];
    sum += (c0[k] & 0xffffu) + (c0[k] >> 16) + (c1[k] & 0xffffu) + (c1[k] >> 16);
  }
  const uint32_t incl = wave_incl_sum32(sum);
  if (lane == kWave - 1) wtot[w] = incl;
  __syncthreads();
  uint32_t run = incl - sum;
  for (uint32_t i = 0; i < w; ++i) run += wtot[i];
#pragma unroll
  for (uint32_t k = 0; k < kSteps; ++k) {
    const uint32_t s1 = run + (c0[k] & 0xffffu), s2 = s1 + (c0[k] >> 16), s3 = s2 + (c1[k] & 0xffffu);
    bin[0][t * kSteps + k] = run | (s1 << 16);
    bin[1][t * kSteps + k] = s2 | (s3 << 16);
    run = s3 + (c1[k] >> 16);
  }
  __syncthreads();
#pragma unroll
  for (uint32_t k = 0; k < kSteps; ++k) {
    if (d[k] >= kSmallBins) continue;
    const uint32_t x = (atomicAdd(&mine[d[k]], 1u << shift) >> shift) & 0xffffu;
    rank[v0 + k * kWave] = x;
    order[x] = v0 + k * kWave;
  }
}

// 12 n bytes >= 49164 (blocks - 1), of which 20 KB + 9.8 KB a block are used.
RankWork rank_work(uint64_t n, uint32_t* ws) {
  const uint64_t tiles = (n + kTile - 1) / kTile;
  const uint64_t per = (tiles + kRankBlocks - 1) / kRankBlocks;
  RankWork r{};
  r.span = per * kTile;
  r.blocks = (uint32_t)((n + r.span - 1) / r.span);
  r.first = ws;
  r.total = ws + kDegClasses + 64;
  r.cnt = r.total + kDegClasses + 64;
  return r;
}

// Block b's class counts, in the LDS words cls.
__device__ void class_hist(const int64_t* row_off, uint64_t n, const RankWork& r, uint64_t b,
                           uint32_t* cls) {
  for (uint32_t i = threadIdx.x; i < kDegClasses; i += kBlock) cls[i] = 0;
  __syncthreads();
  const uint64_t v0 = b * r.span, v1 = v0 + r.span < n ? v0 + r.span : n;
  for (uint64_t v = v0 + threadIdx.x; v < v1; v += kBlock)
    atomicAdd(&cls[deg_class(degree_of(row_off, v))], 1u);
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < kDegClasses; i += kBlock)
    r.cnt[(uint64_t)i * r.blocks + b] = cls[i];
}

// The vertices of a class in earlier blocks, in place of its counts, and in all;
// a wave per class.
__global__ __launch_bounds__(kBlock) void k_class_sum(RankWork r) {
  const uint32_t c = blockIdx.x * kWavesPerBlock + threadIdx.x / kWave, lane = lane_id();
  uint32_t* cnt = r.cnt + (uint64_t)c * r.blocks;
  uint32_t run = 0;
  for (uint32_t b0 = 0; b0 < r.blocks; b0 += 4 * kWave) {
    uint32_t v[4];
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
      const uint32_t b = b0 + k * kWave + lane;
      v[k] = b < r.blocks ? cnt[b] : 0u;
    }
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
      const uint32_t incl = wave_incl_sum32(v[k]);
      if (b0 + k * kWave + lane < r.blocks) cnt[b0 + k * kWave + lane] = run + incl - v[k];
      run += (uint32_t)__builtin_amdgcn_readlane(incl, kWave - 1);
    }
  }
  if (lane == 0) r.total[c] = run;
}
static_assert(kDegClasses % kWavesPerBlock == 0, "whole blocks");

// A vertex of a class of one degree gets its rank; the others are laid out by
// class, in the order of their ids, in `wide`.
__global__ __launch_bounds__(kBlock) void k_rank(const int64_t* row_off, uint64_t n, RankWork r,
                                                 uint32_t* order, uint32_t* rank, uint32_t* wide) {
  __shared__ uint32_t next[kDegClasses];  // the block's next place in each class
  // and each wave's first one, in kTile vertices
  __shared__ __align__(16) uint32_t place[kWavesPerBlock][kDegClasses];
  __shared__ uint32_t wtot[kWavesPerBlock];
  const uint32_t b = blockIdx.x;
  const uint64_t v0 = b * r.span, v1 = v0 + r.span < n ? v0 + r.span : n;
  // classes of the next kTile vertices, a run of kTile / 4 per wave
  uint32_t c[kItems];
  uint32_t* mine = place[threadIdx.x / kWave];
  const uint32_t at = threadIdx.x / kWave * (kItems * kWave) + lane_id();
  auto classes = [&](uint64_t t0) {
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      const uint64_t v = t0 + at + k * kWave;
      c[k] = v < v1 ? deg_class(degree_of(row_off, v)) : kDegClasses;
    }
  };
  classes(v0);
  constexpr uint32_t kPer = (kDegClasses + kBlock - 1) / kBlock;
  uint32_t ahead[kPer];  // vertices of the thread's classes in earlier blocks
#pragma unroll
  for (uint32_t k = 0; k < kPer; ++k) {
    const uint32_t i = k * kBlock + threadIdx.x;
    ahead[k] = i < kDegClasses ? r.cnt[(uint64_t)i * r.blocks + b] : 0u;
    if (i < kDegClasses) next[i] = r.total[i];
  }
  for (uint64_t t0 = v0; t0 < v1; t0 += kTile) {
    uint4* zero = reinterpret_cast<uint4*>(place);
    for (uint32_t i = threadIdx.x; i < kWavesPerBlock * kDegClasses / 4; i += kBlock)
      zero[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    uint32_t nth[kItems];  // of the wave's vertices of its class
#pragma unroll
    for (int k = 0; k < kItems; ++k) nth[k] = c[k] < kDegClasses ? atomicAdd(&mine[c[k]], 1u) : 0u;
    if (t0 == v0) class_scan<kDegClasses>(next, kDegClasses, wtot);
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
      const uint32_t i = k * kBlock + threadIdx.x;
      if (i >= kDegClasses) continue;
      uint32_t run = next[i];
      if (t0 == v0) {
        if (b == 0) r.first[i] = run;
        run += ahead[k];
      }
#pragma unroll
      for (int w = 0; w < kWavesPerBlock; ++w) {
        const uint32_t cnt = place[w][i];
        place[w][i] = run;
        run += cnt;
      }
      next[i] = run;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      if (c[k] >= kDegClasses) continue;
      const uint32_t v = (uint32_t)(t0 + at + k * kWave), x = mine[c[k]] + nth[k];
      if (c[k] < kDegExact) {
        rank[v] = x;
        order[x] = v;
      } else {
        wide[x] = v;
      }
    }
    if (t0 + kTile < v1) {
      classes(t0 + kTile);
      __syncthreads();  // the places have been read
    }
  }
  if (b == 0 && threadIdx.x == 0) r.first[kDegClasses] = (uint32_t)n;
}

// Class kDegExact + blockIdx.x by degree: a counting sort by what the degrees
// of the class differ in, whose places one wave takes, kItems loads in flight;
// beyond kFineBins degrees (from 2^19 on, where the class has at most nnz / 2^19
// vertices) a vertex counts those before it.
__global__ __launch_bounds__(kBlock) void k_rank_wide(const int64_t* row_off, const uint32_t* first,
                                                      const uint32_t* wide, uint32_t* order,
                                                      uint32_t* rank) {
  __shared__ uint32_t bin[kFineBins];
  __shared__ uint32_t wtot[kWavesPerBlock];
  const uint32_t c = kDegExact + blockIdx.x;
  const uint32_t s = first[c], len = first[c + 1] - s;
  if (len == 0) return;
  const uint32_t degrees = 1u << ((c - kDegExact) / kDegFine + kDegExactLog - 6);
  const uint32_t* in = wide + s;
  if (degrees > kFineBins) {
    for (uint32_t i = threadIdx.x; i < len; i += kBlock) {
      const uint32_t v = in[i], d = degree_of(row_off, v);
      uint32_t x = s;
      for (uint32_t k = 0; k < len; ++k) {
        const uint32_t dk = degree_of(row_off, in[k]);
        x += dk < d || (dk == d && k < i);
      }
      rank[v] = x;
      order[x] = v;
    }
    return;
  }
  for (uint32_t i = threadIdx.x; i < degrees; i += kBlock) bin[i] = 0;
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < len; i += kBlock)
    atomicAdd(&bin[degree_of(row_off, in[i]) & (degrees - 1)], 1u);
  __syncthreads();
  class_scan<kFineBins>(bin, degrees, wtot);
  if (threadIdx.x >= kWave) return;
  for (uint64_t i0 = threadIdx.x; i0 < len; i0 += kItems * kWave) {
    uint32_t v[kItems], d[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k) v[k] = i0 + k * kWave < len ? in[i0 + k * kWave] : 0u;
#pragma unroll
    for (int k = 0; k < kItems; ++k) d[k] = degree_of(row_off, v[k]) & (degrees - 1);
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
      if (i0 + k * kWave >= len) continue;
      const uint32_t x = s + atomicAdd(&bin[d[k]], 1u);
      rank[v[k]] = x;
      order[x] = v[k];
    }
  }
}

void degree_rank(const int64_t* row_off, uint64_t n, uint64_t nnz, const RankWork& r, uint32_t* wide,
                 uint32_t* order, uint32_t* rank, hipStream_t s) {
  if (n <= kRankSmall) return;  // ranked by the setup
  hipLaunchKernelGGL(k_class_sum, dim3(kDegClasses / kWavesPerBlock), dim3(kBlock), 0, s, r);
  hipLaunchKernelGGL(k_rank, dim3(r.blocks), dim3(kBlock), 0, s, row_off, n, r, order, rank, wide);
  const uint64_t most = nnz < 0xffffffffu ? nnz : 0xffffffffu;  // no degree is larger
  if (most >= kDegExact)
    hipLaunchKernelGGL(k_rank_wide, dim3(deg_class((uint32_t)most) + 1 - kDegExact), dim3(kBlock),
                       0, s, row_off, (const uint32_t*)r.first, (const uint32_t*)wide, order, rank);
}

// ------------------------------------------------ spectral thresholds
// Keep probability of an edge whose smaller degree is d (section 4.2.1).
__device__ __forceinline__ double spectral_p(double ups, uint32_t d) {
  const double pe = ups / (double)d;
  return pe > 1.0 ? 1.0 : pe;
}
__device__ __forceinline__ uint64_t spectral_thr(double ups, uint32_t d) {
  const double pe = spectral_p(ups, d);
  return pe >= 1.0 ? (uint64_t(1) << 32) : (uint64_t)floor(pe * 4294967296.0);
}
// The threshold that an edge has if this end has the smaller degree, at most
// 2^32 - 1.  The quotient, the product and the floor do not decrease as d
// falls, so an edge's threshold is the larger one of its ends': one division
// per vertex and one 4-byte gather per entry in place of a division and the
// two offsets of the other end.
__device__ __forceinline__ uint32_t vertex_thr(double ups, uint32_t d) {
  const uint64_t t = d ? spectral_thr(ups, d) : 0u;
  return t < 0xffffffffu ? (uint32_t)t : 0xffffffffu;
}

// --------------------------------------------------------- small writes
// Copies up to 512 bytes of host data to device memory as a kernel argument,
// so that a call can set up its descriptors without a host-to-device copy
// (and stays capturable in a HIP graph).
struct Blob {
  uint32_t w[128];
};

__global__ void k_put(uint32_t* dst, Blob b, uint32_t words) {
  if (threadIdx.x < words) dst[threadIdx.x] = b.w[threadIdx.x];
}

void put_bytes(void* dst, const void* src, uint32_t bytes, hipStream_t s) {
  Blob b{};
  __builtin_memcpy(b.w, src, bytes);
  hipLaunchKernelGGL(k_put, dim3(1), dim3(128), 0, s, static_cast<uint32_t*>(dst), b,
                     (bytes + 3) / 4);
}

// ------------------------------------------------------ CSR tile machinery
// Last graph g with tile0[g] <= t (tile0 is non-decreasing; graphs without
// tiles are skipped over).
__device__ __forceinline__ uint32_t graph_of_tile(const uint64_t* tile0, uint32_t count,
                                                  uint64_t t) {
  uint32_t lo = 0, hi = count;
  while (hi - lo > 1) {
    const uint32_t mid = lo + ((hi - lo) >> 1);
    if (tile0[mid] <= t)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// Record of tile t of a set; the first rows at or past its first entry and
// past its last one are searched together.
__device__ __forceinline__ TileRec tile_rec(const int64_t* row_off, uint32_t g, uint64_t vb,
                                            uint64_t nv, uint64_t eb, uint64_t ne, uint64_t tg,
                                            bool last, uint64_t tile) {
  const uint64_t end = eb + ne, ve = vb + nv;
  const int64_t j0 = (int64_t)(eb + tg * tile);
  const uint64_t left = end > (uint64_t)j0 ? end - (uint64_t)j0 : 0;
  const uint32_t span = (uint32_t)(left < tile ? left : tile);
  const int64_t j1 = j0 + span;
  uint64_t l0 = vb, h0 = ve, l1 = vb, h1 = ve;  // first rows in [vb, ve] with row_off[r] >= j0, j1
  while (l0 < h0 || l1 < h1) {
    const uint64_t m0 = l0 + ((h0 - l0) >> 1), m1 = l1 + ((h1 - l1) >> 1);
    const int64_t v0 = row_off[m0], v1 = row_off[m1];  // m <= ve: row_off has an end entry
    if (l0 < h0) {
      if (v0 < j0) l0 = m0 + 1;
      else h0 = m0;
    }
    if (l1 < h1) {
      if (v1 < j1) l1 = m1 + 1;
      else h1 = m1;
    }
  }
  TileRec R;
  R.j0 = j0;
  R.span = span;
  R.g = g;
  R.lo = (uint32_t)l0;
  R.hi = last ? (uint32_t)ve : (uint32_t)l1;
  R.last = last ? 1u : 0u;
  R.pad = 0;
  return R;
}

// ------------------------------------------------------------- setup
// One launch for everything that waits for nothing but the CSR: the header
// of a one-graph set, tile records, cleared arrays, the ranks of a small
// graph or the class counts of a larger one.  Every job has blocks of its own.
__global__ __launch_bounds__(kBlock) void k_setup(SetupArgs a) {
  __shared__ uint32_t bins[2][kSmallBins];
  __shared__ uint32_t wtot[kWavesPerBlock];
  static_assert(kDegClasses <= 2 * kSmallBins, "the classes fit the bins");
  uint32_t job = 0, b = blockIdx.x;
  while (b >= a.nb[job]) b -= a.nb[job++];  // the grid is the sum of nb
  const uint64_t t = b * (uint64_t)kBlock + threadIdx.x, nt = a.nb[job] * (uint64_t)kBlock;
  if (job == kJobHeader) {
    if (threadIdx.x < a.hdr_words) a.hdr_dst[threadIdx.x] = a.hdr[threadIdx.x];
  } else if (job == kJobRank) {
    rank_small(a.row_off, (uint32_t)a.n, a.order, a.rank, bins, wtot);
  } else if (job == kJobHist) {
    class_hist(a.row_off, a.n, a.rank_work, b, bins[0]);
  } else if (job == kJobThr) {
    for (uint64_t v = t; v < a.n; v += nt) a.thr[v] = vertex_thr(a.ups, degree_of(a.row_off, v));
  } else if (job < kJobFill) {
    const RecJob& r = a.rec[job - kJobRecs];
    for (uint64_t i = t; i < r.ntiles; i += nt) {
      if (r.count == 0) {  // one graph: the whole CSR
        r.recs[i] = tile_rec(a.row_off, 0, 0, a.n, 0, a.nnz, i, i + 1 == r.ntiles, r.tile);
      } else {
        const uint32_t g = graph_of_tile(r.tile0, r.count, i);
        const GDesc& G = a.gd[g];
        r.recs[i] = tile_rec(a.row_off, g, G.vb, G.nv, G.eb, G.ne, i - r.tile0[g],
                             i + 1 == r.tile0[g + 1], r.tile);
      }
    }
  } else {
    const FillJob& f = a.fill[job - kJobFill];
    const uint4 v = make_uint4(f.v, f.v, f.v, f.v);
    for (uint64_t i = t; i < f.quads; i += nt) f.p[i] = v;
  }
}

void setup(SetupArgs& a, hipStream_t s) {
  auto blocks = [](uint64_t items, uint32_t cap) {
    const uint64_t g = (items + kBlock - 1) / kBlock;
    return (uint32_t)(g < cap ? g : cap);
  };
  a.nb[kJobHeader] = a.hdr_words ? 1 : 0;
  a.nb[kJobRank] = a.order && a.n <= kRankSmall && a.n ? 1 : 0;
  for (int i = 0; i < kMaxRecs; ++i) a.nb[kJobRecs + i] = blocks(a.rec[i].ntiles, 4096);
  for (int i = 0; i < kMaxFills; ++i) a.nb[kJobFill + i] = blocks(a.fill[i].quads, 1024);
  a.nb[kJobThr] = a.thr ? blocks(a.n, 4096) : 0;
  a.nb[kJobHist] = a.order && a.n > kRankSmall ? a.rank_work.blocks : 0;
  uint64_t grid = 0;
  for (int i = 0; i < kSetupJobs; ++i) grid += a.nb[i];
  if (grid) hipLaunchKernelGGL(k_setup, dim3((unsigned)grid), dim3(kBlock), 0, s, a);
}

// Union CSR of a set: block-sized chunks of each graph's row offsets
// (shifted by the graph's first entry) and columns (shifted by its first
// vertex).
__global__ __launch_bounds__(kBlock) void k_gather(const GDesc* gd, uint32_t count,
                                                   const uint64_t* vtile0,
                                                   const uint64_t* etile0, uint64_t nvt,
                                                   uint64_t net, uint64_t N, uint64_t NNZ,
                                                   int64_t* urow, uint32_t* ucol) {
  if (blockIdx.x == 0 && threadIdx.x == 0) urow[N] = (int64_t)NNZ;
  for (uint64_t t = blockIdx.x; t < nvt + net; t += gridDim.x) {
    const bool vert = t < nvt;
    const uint64_t tt = vert ? t : t - nvt;
    const uint64_t* pre = vert ? vtile0 : etile0;
    const uint32_t g = graph_of_tile(pre, count, tt);
    const GDesc& G = gd[g];
    const uint64_t i0 = (tt - pre[g]) * kTile;
    if (vert) {
      const uint64_t i1 = i0 + kTile < G.nv ? i0 + kTile : G.nv;
      // (a spectral graph's thresholds lie in its output offsets until the
      // scatter pass writes those)
      uint32_t* thr = G.op == SLIM_OP_SPECTRAL ? static_cast<uint32_t*>(G.out_row) : nullptr;
      for (uint64_t i = i0 + threadIdx.x; i < i1; i += kBlock) {
        urow[G.vb + i] = G.in_row[i] + (int64_t)G.eb;
        if (thr) thr[i] = vertex_thr(G.ups, degree_of(G.in_row, i));
      }
    } else {
      const uint64_t i1 = i0 + kTile < G.ne ? i0 + kTile : G.ne;
      const uint32_t vb = (uint32_t)G.vb;
      for (uint64_t i = i0 + threadIdx.x; i < i1; i += kBlock) ucol[G.eb + i] = G.in_col[i] + vb;
    }
  }
}

// The thresholds of a gathered set's spectral graphs, as k_gather writes them,
// from the union's offsets.
__global__ __launch_bounds__(kBlock) void k_spectral_thr(const GDesc* gd, uint32_t count,
                                                         const uint64_t* vtile0, uint64_t nvt,
                                                         const int64_t* urow) {
  for (uint64_t t = blockIdx.x; t < nvt; t += gridDim.x) {
    const uint32_t g = graph_of_tile(vtile0, count, t);
    const GDesc& G = gd[g];
    if (G.op != SLIM_OP_SPECTRAL) continue;
    const uint64_t i0 = (t - vtile0[g]) * kTile;
    const uint64_t i1 = i0 + kTile < G.nv ? i0 + kTile : G.nv;
    uint32_t* thr = static_cast<uint32_t*>(G.out_row);
    for (uint64_t i = i0 + threadIdx.x; i < i1; i += kBlock)
      thr[i] = vertex_thr(G.ups, degree_of(urow, G.vb + i));
  }
}

void spectral_thr(const GDesc* gd, uint32_t count, const uint64_t* vtile0, uint64_t nvt,
                  const int64_t* urow, hipStream_t s) {
  if (nvt)
    hipLaunchKernelGGL(k_spectral_thr, dim3((unsigned)(nvt < 65536 ? nvt : 65536)), dim3(kBlock), 0,
                       s, gd, count, vtile0, nvt, urow);
}

void gather(const GDesc* gd, uint32_t count, const uint64_t* vtile0, const uint64_t* etile0,
            uint64_t nvt, uint64_t net, uint64_t N, uint64_t NNZ, int64_t* urow, uint32_t* ucol,
            hipStream_t s) {
  uint64_t blocks = nvt + net;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_gather, dim3((unsigned)blocks), dim3(kBlock), 0, s, gd, count, vtile0,
                     etile0, nvt, net, N, NNZ, urow, ucol);
}

// Entries of a tile by lane: wave w has the kWaveSpan entries from
// w * kWaveSpan on, in groups of 256, lane l the four consecutive ones from
// 4l on in each group (one 16-byte load aligned to 4 bytes).
constexpr int kGroups = kItems / 4;
constexpr int kWaveSpan = kGroups * 4 * kWave;
typedef uint32_t vec4_t __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ uint32_t entry_of(int g) {
  return (threadIdx.x / kWave) * kWaveSpan + g * 4 * kWave + lane_id() * 4;
}

struct TileRows {
  uint32_t srow[kTile];
  uint32_t wmax[kWavesPerBlock];
};

// Rows of the thread's tile entries: row starts into L.srow, then a max-scan.
// Entries before the first start belong to the row before lo.
__device__ void tile_rows(const int64_t* row_off, int64_t j0, uint32_t lo, uint32_t hi, TileRows& L,
                          uint32_t (&row)[kGroups][4]) {
  const uint32_t t = threadIdx.x, w = t / kWave, lane = lane_id();
  uint4* s4 = reinterpret_cast<uint4*>(L.srow);
#pragma unroll
  for (int k = 0; k < kTile / 4 / kBlock; ++k) s4[k * kBlock + t] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  for (uint64_t r = lo + (uint64_t)t; r < hi; r += kBlock) {
    const int64_t b = row_off[r], e = row_off[r + 1];
    const int64_t s = b - j0;
    if (e > b && s >= 0 && s < kTile) L.srow[s] = r;
  }
  __syncthreads();
  uint32_t carry = 0;
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    uint4 v = s4[entry_of(g) / 4];
    v.y = max(v.x, v.y);
    v.z = max(v.y, v.z);
    v.w = max(v.z, v.w);
    const uint32_t incl = wave_incl_max(v.w);
    uint32_t before = __shfl_up(incl, 1, kWave);
    if (lane == 0) before = 0;
    before = max(before, carry);
    row[g][0] = max(before, v.x);
    row[g][1] = max(before, v.y);
    row[g][2] = max(before, v.z);
    row[g][3] = max(before, v.w);
    carry = max(carry, (uint32_t)__builtin_amdgcn_readlane(incl, kWave - 1));
  }
  if (lane == 0) L.wmax[w] = carry;
  __syncthreads();
  uint32_t base = lo > 0 ? lo - 1 : 0;
  for (uint32_t i = 0; i < w; ++i) base = max(base, L.wmax[i]);
#pragma unroll
  for (int g = 0; g < kGroups; ++g)
#pragma unroll
    for (int k = 0; k < 4; ++k) row[g][k] = max(row[g][k], base);
}

// The thread's entries of src[j0 .. j0 + span); the others are 0.
__device__ __forceinline__ void load_entries(const uint32_t* src, int64_t j0, uint32_t span,
                                             uint32_t (&v)[kGroups][4]) {
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    const uint32_t i = entry_of(g);
    const uint32_t* p = src + j0 + i;
    if (i + 4 <= span) {
      const vec4_t x = *reinterpret_cast<const vec4_t*>(p);
#pragma unroll
      for (int k = 0; k < 4; ++k) v[g][k] = x[k];
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) v[g][k] = i + k < span ? p[k] : 0u;
    }
  }
}

// ------------------------------------------------ flag stream compaction
// Both passes are bound by HBM where nothing is gathered (edge sampling at
// R-MAT scale 24, 2.1 GB of columns: count 0.84 ms, of which the Philox draws
// issue for about 0.75, scatter 0.73 ms for 3.5 GB).  What they cost before,
// 1.42 and 1.31 ms, was latency: one entry per lane and load, each load
// behind the last one's store, and a row search of five block barriers.
//
// Policies decide per CSR entry j (union row r) whether it is kept and what
// is written; kept entries keep their CSR order, so rows stay sorted.  A
// policy's Ctx holds what it needs of the tile's graph, `source` is the array
// a pass streams, `fetch` the gather that a decision needs (all of a thread's
// gathers are issued before the first decision).
//
// Orientation: keep (r,c) iff rank(c) > rank(r) and write rank(c).  The
// counting pass gathers rank(c) once per entry and streams it to rcol; the
// scatter pass and the triangle kernel read rcol instead of gathering.
struct OrientPolicy {
  static constexpr bool kOut = false;
  const uint32_t* col;
  const uint32_t* rank;
  uint32_t* rcol;
  struct Ctx {};
  __device__ Ctx ctx(const GDesc&) const { return {}; }
  __device__ bool needs_rows(const Ctx&) const { return true; }
  __device__ const uint32_t* source(const Ctx&) const { return col; }
  __device__ uint32_t fetch(const Ctx&, uint32_t c) const { return rank[c]; }
  __device__ bool flag(const Ctx&, uint32_t, uint32_t rc, uint32_t r) const { return rc > rank[r]; }
  __device__ void stream(const Ctx&, int64_t j, uint32_t n, const uint32_t (&rc)[4]) const {
    if (n == 4) {
      *reinterpret_cast<vec4_t*>(rcol + j) = vec4_t{rc[0], rc[1], rc[2], rc[3]};
    } else {
      for (uint32_t k = 0; k < n; ++k) rcol[j + k] = rc[k];
    }
  }
  __device__ const uint32_t* values(const Ctx&) const { return rcol; }
  __device__ uint32_t value(const Ctx&, uint32_t v) const { return v; }
};

// Output of a compression job, per graph: a graph of a triangle operation
// keeps (r,c) iff its edge is not marked deleted; an ES graph keeps {a<b}
// (local ids) iff Philox(a,b,0,1) word 0 >= thr; a spectral sparsification
// graph keeps {a<b} iff Philox(a,b,0,2) word 0 < floor(p_ab 2^32) with
// p_ab = min(1, upsilon / min(d_a, d_b)) in double precision (section 4.2.1)
// and weighs it 1/p_ab.  Written values are local ids.  The count pass reads
// a spectral graph's vertex thresholds from its output offsets, which the
// scatter pass then overwrites: a second output pass over the set needs them
// written again (spectral_thr).  R-MAT scale 22: count pass 1.50 ms with the
// degrees gathered and divided per entry, 1.17 ms with the thresholds.
// kMode: the mode of every graph of the set (0 triangle operations, 1 ES, 2
// spectral), or kMixed: a pass over one kind of graph keeps only that kind's
// values in registers (edge sampling at R-MAT scale 24: 1.73 ms with the
// mixed passes, 1.51 ms so).
constexpr uint32_t kMixed = 3;
template <uint32_t kMode>
struct OutPolicy {
  static constexpr bool kOut = true;
  const uint32_t* col;
  const uint32_t* eid;
  const uint32_t* del;   // deletion marks: a bitmap, or NULL:
  const uint8_t* marks;  //   a byte per edge
  const int64_t* row_off;
  uint64_t m;
  struct Ctx {
    uint64_t thr;
    double ups;
    const uint32_t* vthr;       // spectral: threshold of each vertex
    uint32_t vb, k0, k1, any_mode;
  };
  __device__ static uint32_t mode(const Ctx& x) { return kMode == kMixed ? x.any_mode : kMode; }
  __device__ Ctx ctx(const GDesc& G) const {
    return Ctx{G.thr, G.ups, static_cast<const uint32_t*>(G.out_row), (uint32_t)G.vb, G.k0, G.k1,
               G.op == SLIM_OP_ES ? 1u : (G.op == SLIM_OP_SPECTRAL ? 2u : 0u)};
  }
  __device__ bool needs_rows(const Ctx& x) const { return mode(x) != 0; }
  __device__ const uint32_t* source(const Ctx& x) const { return mode(x) ? col : eid; }
  __device__ uint32_t fetch(const Ctx& x, uint32_t v) const {
    if (mode(x) == 0) {  // v >= m only for inputs breaking the contract
      if (!del) return v < m ? (uint32_t)marks[v] << (v & 31u) : 0u;
      return v < m ? del[v >> 5] : 0u;
    }
    if (mode(x) == 2) return x.vthr[v - x.vb];
    return 0u;
  }
  __device__ bool flag(const Ctx& x, uint32_t v, uint32_t got, uint32_t r) const {
    if (mode(x) == 0) return v >= m || !((got >> (v & 31u)) & 1u);
    const uint32_t c = v - x.vb, rl = r - x.vb;
    const uint32_t a = min(c, rl), b = max(c, rl);
    uint32_t w0, w1;
    philox_w01(a, b, 0u, mode(x), x.k0, x.k1, w0, w1);
    if (mode(x) == 1) return !((uint64_t)w0 < x.thr);
    const uint32_t thr = max(got, x.vthr[rl]);
    if (w0 < thr || thr != 0xffffffffu) return w0 < thr;
    // w0 is 2^32 - 1: only a threshold of 2^32 keeps it
    return spectral_thr(x.ups, min(degree_of(row_off, v), degree_of(row_off, r))) >> 32;
  }
  __device__ void stream(const Ctx&, int64_t, uint32_t, const uint32_t (&)[4]) const {}
  __device__ const uint32_t* values(const Ctx&) const { return col; }
  __device__ uint32_t value(const Ctx& x, uint32_t v) const { return v - x.vb; }
  __device__ float weight(const Ctx& x, uint32_t c, uint32_t r) const {
    return (float)(1.0 / spectral_p(x.ups, min(degree_of(row_off, c), degree_of(row_off, r))));
  }
};

// The count pass keeps the ballots of every group (masks, 512 B per tile: for
// each wave and group one per position in the lane's four entries), so the
// scatter pass neither recomputes the flags (Philox draws, bitmap gathers) nor
// needs the rows of its entries.
template <class P>
__global__ __launch_bounds__(kBlock) void k_compact_count(P p, const int64_t* row_off,
                                                          const GDesc* gd, const TileRec* recs,
                                                          uint32_t* tile_cnt, uint64_t* masks) {
  __shared__ TileRows L;
  __shared__ uint32_t wsum[kWavesPerBlock];
  const TileRec R = recs[blockIdx.x];
  const typename P::Ctx x = p.ctx(gd[R.g]);
  const uint32_t w = threadIdx.x / kWave, lane = lane_id();
  uint32_t v[kGroups][4], got[kGroups][4], row[kGroups][4] = {};
  load_entries(p.source(x), R.j0, R.span, v);
#pragma unroll
  for (int g = 0; g < kGroups; ++g)
#pragma unroll
    for (int k = 0; k < 4; ++k) got[g][k] = entry_of(g) + k < R.span ? p.fetch(x, v[g][k]) : 0u;
  if (p.needs_rows(x)) tile_rows(row_off, R.j0, R.lo, R.hi, L, row);
  uint32_t cnt = 0;
  uint64_t mine = 0;
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    const uint32_t i = entry_of(g);
    if (i < R.span) p.stream(x, R.j0 + i, min(R.span - i, 4u), got[g]);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool f = i + k < R.span && p.flag(x, v[g][k], got[g][k], row[g][k]);
      const uint64_t m = __ballot(f);
      mine = lane == (uint32_t)(4 * g + k) ? m : mine;
      cnt += __popcll(m);
    }
  }
  if (lane < (uint32_t)kItems) masks[(uint64_t)blockIdx.x * kChunks + w * kItems + lane] = mine;
  if (lane == 0) wsum[w] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t s = 0;
    for (int i = 0; i < kWavesPerBlock; ++i) s += wsum[i];
    tile_cnt[blockIdx.x] = s;
  }
}

// Counters of graph g's job.
__device__ __forceinline__ void put_stats(const GDesc* gd, uint32_t count, uint32_t g,
                                          const uint64_t* counters, uint64_t kept) {
  const GDesc& G = gd[g];
  // gd[count] describes the union: its stats pointer, if set, is an array
  // of one record per graph (the per-graph copy a batch keeps)
  slim_stats_t* all = gd[count].stats;
  if (!G.stats && !all) return;
  const uint64_t m = G.ne / 2, m_out = kept / 2;
  const bool tr = op_lists_triangles(G.op) && counters;
  slim_stats_t st;
  st.n = G.nv;
  st.m_in = m;
  st.triangles = tr ? counters[2 * g] : 0;
  st.selected = tr ? counters[2 * g + 1] : 0;
  st.deleted = m - m_out;
  st.m_out = m_out;
  if (G.stats) *G.stats = st;
  if (all) all[g] = st;
}

// Kept entries go to the tile's graph's output behind those of the graph's
// earlier tiles; the tile also writes the row starts it owns and, if it is
// the graph's last tile, the end offset and the job's counters.  Kept values
// are gathered in LDS, so that the output is written in whole lines.  Where
// no graph has more than kSelfScan tiles, a tile adds up the counts of the
// tiles before it by itself (tile_base is NULL): that is at most 24 loads per
// thread in place of the scan's one to three launches (with the header and the
// stats as launches too, sampling a 2000-vertex graph took six launches and 29
// us; three and 14.8 us now).
template <class P, typename OffT>
__global__ __launch_bounds__(kBlock) void k_compact_scatter(
    P p, const int64_t* row_off, const GDesc* gd, uint32_t count, const uint64_t* tile0,
    const TileRec* recs, const uint32_t* tile_cnt, const uint64_t* tile_base,
    const uint64_t* masks, const uint64_t* counters) {
  __shared__ TileRows L;
  __shared__ uint32_t kept[kTile];
  __shared__ uint64_t cmask[kChunks];
  __shared__ uint32_t wsum[kWavesPerBlock], gsum[kWavesPerBlock][kGroups];
  __shared__ uint64_t before[kWavesPerBlock];
  const TileRec R = recs[blockIdx.x];
  const GDesc& G = gd[R.g];
  const typename P::Ctx x = p.ctx(G);
  // rows only for the weights of spectral sparsification
  const bool weights = P::kOut && G.out_w && G.op == SLIM_OP_SPECTRAL;
  const uint32_t w = threadIdx.x / kWave, lane = lane_id();
  uint64_t mine = 0;  // the count pass's ballots
  if (lane < (uint32_t)kItems) mine = masks[(uint64_t)blockIdx.x * kChunks + w * kItems + lane];
  uint32_t v[kGroups][4], row[kGroups][4];
  load_entries(p.values(x), R.j0, R.span, v);
  const uint64_t first = tile0[R.g];
  uint64_t sum = 0;
  if (!tile_base)
    for (uint64_t t = first + threadIdx.x; t < blockIdx.x; t += kBlock) sum += tile_cnt[t];
  if (weights) tile_rows(row_off, R.j0, R.lo, R.hi, L, row);
  if (lane < (uint32_t)kItems) cmask[w * kItems + lane] = mine;
  uint32_t total = 0;
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    if (lane == 0) gsum[w][g] = total;  // kept before the group in this wave
#pragma unroll
    for (int k = 0; k < 4; ++k)
      total += __builtin_popcount(__builtin_amdgcn_readlane((uint32_t)mine, 4 * g + k)) +
               __builtin_popcount(__builtin_amdgcn_readlane((uint32_t)(mine >> 32), 4 * g + k));
  }
  sum = wave_sum64(sum);
  if (lane == 0) {
    wsum[w] = total;
    before[w] = sum;
  }
  __syncthreads();
  uint32_t wbase = 0, all = 0;
  uint64_t base = 0;
#pragma unroll
  for (uint32_t i = 0; i < (uint32_t)kWavesPerBlock; ++i) {
    if (i < w) wbase += wsum[i];
    all += wsum[i];
    base += before[i];
  }
  if (tile_base) base = tile_base[blockIdx.x] - tile_base[first];
  float* kw = reinterpret_cast<float*>(L.srow);
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    uint64_t m[4];
    uint32_t pos = wbase + gsum[w][g];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)mine, 4 * g + k);
      const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(mine >> 32), 4 * g + k);
      m[k] = ((uint64_t)hi << 32) | lo;
      pos = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, pos));
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (!((m[k] >> lane) & 1u)) continue;
      kept[pos] = p.value(x, v[g][k]);
      if constexpr (P::kOut)
        if (weights) kw[pos] = p.weight(x, v[g][k], row[g][k]);
      ++pos;
    }
  }
  __syncthreads();
  const uint64_t cap = G.cap;
  const uint32_t n_out = base < cap ? (uint32_t)min((uint64_t)all, cap - base) : 0u;  // all, for inputs that meet the contract
  uint32_t* out = G.out_col + base;
  for (uint32_t i = threadIdx.x; i < n_out; i += kBlock) {
    out[i] = kept[i];
    if constexpr (P::kOut)
      if (weights) G.out_w[base + i] = kw[i];
  }
  OffT* rstart = static_cast<OffT*>(G.out_row);
  for (uint64_t r = R.lo + (uint64_t)threadIdx.x; r < R.hi; r += kBlock) {
    const int64_t s = row_off[r] - R.j0;
    uint64_t o = base + all;
    if (s >= 0 && s < (int64_t)R.span) {
      // entry s: lane sl's k-th of group sg of wave sw
      const uint32_t sw = (uint32_t)s / kWaveSpan, sg = (uint32_t)s / (4 * kWave) % kGroups;
      const uint32_t sl = (uint32_t)s / 4 % kWave, k = (uint32_t)s % 4;
      const uint64_t lt = (uint64_t(1) << sl) - 1;
      uint32_t q = gsum[sw][sg];
      for (uint32_t i = 0; i < sw; ++i) q += wsum[i];
#pragma unroll
      for (uint32_t i = 0; i < 4; ++i) {
        const uint64_t mk = cmask[sw * kItems + 4 * sg + i];
        q += __popcll(mk & (i < k ? (lt << 1) | 1 : lt));
      }
      o = base + q;
    }
    rstart[r - G.vb] = (OffT)(o < cap ? o : cap);
  }
  if (R.last && threadIdx.x == 0) {
    const uint64_t o = base + all;
    rstart[G.nv] = (OffT)(o < cap ? o : cap);
    if constexpr (P::kOut) put_stats(gd, count, R.g, counters, o);
  }
}

// Count, scan (of many tiles), scatter.
template <class P, typename OffT>
void compact(const P& p, const int64_t* row_off, const GDesc* gd, uint32_t count,
             const uint64_t* tile0, const TileRec* recs, uint64_t ntiles, bool self_scan,
             uint32_t* tile_cnt, uint64_t* masks, uint64_t* tile_base, uint64_t* scan_tmp,
             const uint64_t* counters, hipStream_t s) {
  hipLaunchKernelGGL(k_compact_count<P>, dim3((unsigned)ntiles), dim3(kBlock), 0, s, p, row_off,
                     gd, recs, tile_cnt, masks);
  if (!self_scan) scan_excl<uint32_t>(tile_cnt, ntiles, tile_base, scan_tmp, s);
  hipLaunchKernelGGL((k_compact_scatter<P, OffT>), dim3((unsigned)ntiles), dim3(kBlock), 0, s, p,
                     row_off, gd, count, tile0, recs, (const uint32_t*)tile_cnt,
                     (const uint64_t*)(self_scan ? nullptr : tile_base), (const uint64_t*)masks,
                     counters);
}

void orient(const int64_t* row_off, const uint32_t* col, const uint32_t* rank, uint32_t* rcol,
            const GDesc* gd_union, const uint64_t* tile0, const TileRec* recs, uint64_t ntiles,
            uint32_t* tile_cnt, uint64_t* masks, uint64_t* tile_base, uint64_t* scan_tmp,
            hipStream_t s) {
  OrientPolicy p{col, rank, rcol};
  compact<OrientPolicy, uint32_t>(p, row_off, gd_union, 0, tile0, recs, ntiles,
                                  ntiles <= kSelfScan, tile_cnt, masks, tile_base, scan_tmp,
                                  nullptr, s);
}

void compact_out(const int64_t* row_off, const uint32_t* col, const uint32_t* eid,
                 const uint32_t* del, const uint8_t* marks, uint64_t m, const GDesc* gd,
                 uint32_t count, const uint64_t* tile0, const TileRec* recs, uint64_t ntiles, uint64_t most_tiles,
                 uint32_t* tile_cnt, uint64_t* masks, uint64_t* tile_base, uint64_t* scan_tmp,
                 const uint64_t* counters, uint32_t kinds, hipStream_t s) {
  auto go = [&](auto policy) {
    compact<decltype(policy), int64_t>(policy, row_off, gd, count, tile0, recs, ntiles,
                                       most_tiles <= kSelfScan, tile_cnt, masks, tile_base,
                                       scan_tmp, counters, s);
  };
  switch (kinds) {
    case 1u << 0: go(OutPolicy<0>{col, eid, del, marks, row_off, m}); break;
    case 1u << 1: go(OutPolicy<1>{col, eid, del, marks, row_off, m}); break;
    case 1u << 2: go(OutPolicy<2>{col, eid, del, marks, row_off, m}); break;
    default: go(OutPolicy<kMixed>{col, eid, del, marks, row_off, m});
  }
}

// ------------------------------------------------------------ validation
// err bits: 1 offsets, 2 id >= n, 4 self-loop, 8 unsorted/duplicate, 16 asymmetric
__global__ void k_validate_offsets(const int64_t* row_off, uint64_t n, uint64_t nnz,
                                   uint32_t* err) {
  for (uint64_t r = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; r <= n;
       r += (uint64_t)gridDim.x * blockDim.x) {
    bool bad = false;
    if (r == 0 && row_off[0] != 0) bad = true;
    if (r == n && row_off[n] != (int64_t)nnz) bad = true;
    if (r < n && row_off[r + 1] < row_off[r]) bad = true;
    if (bad) atomicOr(err, 1u);
  }
}

__global__ __launch_bounds__(kBlock) void k_validate_entries(const int64_t* row_off,
                                                             const uint32_t* col, uint64_t n,
                                                             const TileRec* recs,
                                                             uint32_t* err) {
  __shared__ TileRows L;
  const TileRec R = recs[blockIdx.x];
  uint32_t row[kGroups][4];
  tile_rows(row_off, R.j0, R.lo, R.hi, L, row);
#pragma unroll
  for (int g = 0; g < kGroups; ++g)
    reinterpret_cast<uint4*>(L.srow)[entry_of(g) / 4] =
        make_uint4(row[g][0], row[g][1], row[g][2], row[g][3]);
  uint32_t e = 0;
  for (int i = 0; i < kItems; ++i) {  // a thread reads the rows it wrote
    const uint32_t at = entry_of(i / 4) + i % 4;
    if (at >= R.span) continue;
    const uint64_t j = (uint64_t)R.j0 + at;
    const uint32_t r = L.srow[at];
    const uint32_t c = col[j];
    if ((uint64_t)c >= n) {
      e |= 2u;
      continue;
    }
    if (c == r) e |= 4u;
    if ((int64_t)j > row_off[r] && col[j - 1] >= c) e |= 8u;
    int64_t lo = row_off[c], hi = row_off[c + 1];
    while (lo < hi) {
      const int64_t mid = lo + ((hi - lo) >> 1);
      if (col[mid] < r)
        lo = mid + 1;
      else
        hi = mid;
    }
    if (!(lo < row_off[c + 1] && col[lo] == r)) e |= 16u;
  }
  if (e) atomicOr(err, e);
}

void validate_offsets(const int64_t* row_off, uint64_t n, uint64_t nnz, uint32_t* err,
                      hipStream_t s) {
  hipLaunchKernelGGL(k_validate_offsets, dim3(grid_for(n + 1)), dim3(kBlock), 0, s, row_off, n,
                     nnz, err);
}

void validate_entries(const int64_t* row_off, const uint32_t* col, uint64_t n,
                      const TileRec* recs, uint64_t ntiles, uint32_t* err, hipStream_t s) {
  hipLaunchKernelGGL(k_validate_entries, dim3((unsigned)ntiles), dim3(kBlock), 0, s, row_off,
                     col, n, recs, err);
}

}  // namespace slim
