// Sorting DAG rows by rank id.
//
// The triangle kernel finds the in-neighbour edge (y,x) inside out(y) by
// binary search and scans only the part of out(y) ranked above x, which is
// the suffix of a sorted row.  Rows of up to kSortShort entries are sorted by
// one thread each in registers, rows up to 2048 by one wave in registers (a
// bitonic network over 64 lanes x E values: pairs within a lane are exchanged
// in registers, pairs across lanes by a lane shuffle, so no LDS traffic and no
// barrier), up to 4096 by one block in LDS, longer rows by one block in global
// memory.  Whoever sorts a row also writes the fence samples of the line
// starts inside it.
#include "slim_internal.h"

namespace slim {

constexpr uint32_t kSortShort = 32;
constexpr uint32_t kWaveSortMax = 2048;
constexpr uint32_t kBlockSortMax = 4096;
constexpr uint32_t kPad = 0xffffffffu;  // larger than every rank id (n <= 2^32-1)
constexpr int kLongBlock = 1024;

__device__ __forceinline__ uint32_t pow2_ceil(uint32_t v) {
  uint32_t p = 1;
  while (p < v) p <<= 1;
  return p;
}

// Sorted entry v at DAG position pos.
__device__ __forceinline__ void put_sorted(uint32_t* dag_col, uint32_t* fence, uint32_t pos,
                                           uint32_t v) {
  dag_col[pos] = v;
  if (pos % kFenceStep == 0) fence[pos / kFenceStep] = v;
}

// Bitonic sort of the row [beg, beg + len), len <= N, in one thread's
// registers, padded with kPad; loads and stores of four entries aligned to 4
// bytes (up to three entries past the row are read, inside the workspace).
typedef uint32_t row4_t __attribute__((ext_vector_type(4), aligned(4)));
template <int N>
__device__ __forceinline__ void thread_sort(uint32_t* dag_col, uint32_t* fence, uint32_t beg,
                                            uint32_t len) {
  uint32_t v[N];
#pragma unroll
  for (int i = 0; i < N; i += 4) {
    row4_t x = {kPad, kPad, kPad, kPad};
    if ((uint32_t)i < len) x = *reinterpret_cast<const row4_t*>(dag_col + beg + i);
#pragma unroll
    for (int k = 0; k < 4; ++k) v[i + k] = (uint32_t)(i + k) < len ? x[k] : kPad;
  }
#pragma unroll
  for (int k = 2; k <= N; k <<= 1) {
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1) {
#pragma unroll
      for (int r = 0; r < N; ++r) {
        if ((r & j) != 0) continue;
        const uint32_t lo = min(v[r], v[r | j]), hi = max(v[r], v[r | j]);
        v[r] = (r & k) == 0 ? lo : hi;
        v[r | j] = (r & k) == 0 ? hi : lo;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < N; i += 4) {
    if ((uint32_t)i + 4 <= len) {
      *reinterpret_cast<row4_t*>(dag_col + beg + i) = row4_t{v[i], v[i + 1], v[i + 2], v[i + 3]};
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if ((uint32_t)(i + k) < len) dag_col[beg + i + k] = v[i + k];
    }
  }
  // a row of at most 32 entries holds at most one line start
  const uint32_t line = (beg + kFenceStep - 1) / kFenceStep * kFenceStep - beg;
  if (line < len) {
    uint32_t f = v[0];
#pragma unroll
    for (int i = 1; i < N; ++i) f = line == (uint32_t)i ? v[i] : f;
    fence[(beg + line) / kFenceStep] = f;
  }
}
static_assert(kSortShort <= kFenceStep, "one line start per short row");

// DAG ranges by rank, the short rows sorted, the longer ones listed by
// length: wave_list, block_list, huge_list, their counts in counts[0..2]
// (one atomic per list and step of a block).  A thread sorts its row with
// the smallest network that its wave's longest short row needs: a network of
// 32 is 480 instructions for 64 rows, and no step waits on memory, where an
// insertion sort in LDS was a serial chain as long as the square of the
// wave's longest row.  Ranges, sort, lists and fence are one launch (R-MAT
// scale 24: 0.43 ms, 1.05 ms as three launches with insertion sorts; 90001
// vertices of degree 23: 11 us, 68 us; counting each entry's place in LDS took
// 2.9 ms and 27 us).
__global__ __launch_bounds__(kBlock) void k_sort_short(const uint32_t* fstart, const uint32_t* rank,
                                                       uint64_t n, uint2* dag_rng,
                                                       uint32_t* dag_col, uint32_t* fence,
                                                       uint32_t* wave_list, uint32_t* block_list,
                                                       uint32_t* huge_list, uint32_t* counts,
                                                       uint32_t per) {
  __shared__ uint32_t wcnt[kWavesPerBlock][3], at[3];
  const uint32_t t = threadIdx.x, w = t / kWave;
  uint32_t* lists[3] = {wave_list, block_list, huge_list};
  auto listed = [](uint32_t len, int c) {
    return c == 0   ? len > kSortShort && len <= kWaveSortMax
           : c == 1 ? len > kWaveSortMax && len <= kBlockSortMax
                    : len > kBlockSortMax;
  };
  const uint64_t step = (uint64_t)kBlock * per;
  for (uint64_t v0 = blockIdx.x * step; v0 < n; v0 += gridDim.x * step) {
    uint32_t cnt[3] = {0, 0, 0};
#pragma unroll 1
    for (uint32_t k = 0; k < per; ++k) {
      const uint64_t v = v0 + (uint64_t)k * kBlock + t;
      uint32_t beg = 0, len = 0;
      if (v < n) {
        beg = fstart[v];
        const uint32_t e = fstart[v + 1];
        len = e - beg;
        dag_rng[rank[v]] = make_uint2(beg, e);
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) cnt[c] += __popcll(__ballot(listed(len, c)));
      if (len > kSortShort) len = 0;
      if (__ballot(len > 16))
        thread_sort<32>(dag_col, fence, beg, len);
      else if (__ballot(len > 8))
        thread_sort<16>(dag_col, fence, beg, len);
      else if (__ballot(len > 0))
        thread_sort<8>(dag_col, fence, beg, len);
    }
    if (lane_id() == 0)
      for (int c = 0; c < 3; ++c) wcnt[w][c] = cnt[c];
    __syncthreads();
    if (t < 3) {
      uint32_t all = 0;
      for (int i = 0; i < kWavesPerBlock; ++i) all += wcnt[i][t];
      at[t] = all ? atomicAdd(&counts[t], all) : 0u;
    }
    __syncthreads();
    if (cnt[0] | cnt[1] | cnt[2]) {
      uint32_t pos[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        pos[c] = at[c];
        for (uint32_t i = 0; i < w; ++i) pos[c] += wcnt[i][c];
      }
#pragma unroll 1
      for (uint32_t k = 0; k < per; ++k) {
        const uint64_t v = v0 + (uint64_t)k * kBlock + t;
        const uint32_t len = v < n ? fstart[v + 1] - fstart[v] : 0u;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const uint64_t bal = __ballot(listed(len, c));
          if (listed(len, c)) lists[c][pos[c] + __popcll(bal & lanemask_lt())] = (uint32_t)v;
          pos[c] += __popcll(bal);
        }
      }
    }
    __syncthreads();  // wcnt and at are free
  }
}

// The value of lane ^ d, d a power of two known at compile time: a register
// move for 1, 2 and 8 (quad permutations, a rotation of 16 by 8), a swizzle
// without an address for 4 and 16, the general lane shuffle for 32.  Rows of
// up to 512 entries (E <= 8) use it: the listed rows of 256 graphs 646 -> 566
// us; with 16 and 32 values per lane the shuffles are faster (R-MAT scale 24:
// 1.68 ms, 2.22 ms with moves for every E).
__device__ __forceinline__ uint32_t lane_xor(uint32_t v, uint32_t d) {
  switch (d) {
    case 1: return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xf, 0xf, true);   // quad_perm 1,0,3,2
    case 2: return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xf, 0xf, true);   // quad_perm 2,3,0,1
    case 8: return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xf, 0xf, true);  // row_ror:8
    case 4: return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (4 << 10) | 0x1f);    // xor 4 in 32 lanes
    case 16: return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (16 << 10) | 0x1f);  // xor 16
    default: return __shfl_xor(v, (int)d, kWave);
  }
}

// Bitonic sort of one row of len <= 64 * E entries in the registers of one
// wave: element i = lane * E + r sits in register r of its lane, padded with
// kPad past len.  Step (k, j) pairs i with i ^ j; the lower index of the pair
// keeps the minimum where (i & k) == 0, the maximum elsewhere.
template <int E>
__device__ __forceinline__ void wave_sort_regs(uint32_t* dag_col, uint32_t* fence, uint32_t beg,
                                               uint32_t len) {
  const uint32_t* row = dag_col + beg;
  const uint32_t lane = lane_id();
  uint32_t v[E];
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const uint32_t i = lane * E + r;
    v[r] = i < len ? row[i] : kPad;
  }
#pragma unroll
  for (uint32_t k = 2; k <= 64u * E; k <<= 1) {
#pragma unroll
    for (uint32_t j = k >> 1; j > 0; j >>= 1) {
      if (j < (uint32_t)E) {  // the pair is in this lane: registers r and r | j
#pragma unroll
        for (int r = 0; r < E; ++r) {
          if ((r & j) != 0) continue;
          const bool up = ((lane * E + r) & k) == 0;
          const uint32_t a = v[r], b = v[r | j];
          const uint32_t lo = a < b ? a : b, hi = a < b ? b : a;
          v[r] = up ? lo : hi;
          v[r | j] = up ? hi : lo;
        }
      } else {  // the partner is register r of lane ^ (j / E)
        const uint32_t lj = j / E;
        const bool lower = (lane & lj) == 0;
#pragma unroll
        for (int r = 0; r < E; ++r) {
          const bool up = ((lane * E + r) & k) == 0;
          const uint32_t o = E <= 8 ? lane_xor(v[r], lj) : __shfl_xor(v[r], (int)lj, kWave);
          const uint32_t lo = v[r] < o ? v[r] : o, hi = v[r] < o ? o : v[r];
          v[r] = lower == up ? lo : hi;
        }
      }
    }
  }
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const uint32_t i = lane * E + r;
    if (i < len) put_sorted(dag_col, fence, beg + i, v[r]);
  }
}

// The listed rows, in one launch: waves take the rows of the wave list (the
// register sort with the fewest values per lane that holds the row), then
// blocks those of the other two.
__global__ __launch_bounds__(kLongBlock) void k_sort_long(const uint32_t* fstart, uint32_t* dag_col,
                                                          uint32_t* fence,
                                                          const uint32_t* wave_list,
                                                          const uint32_t* block_list,
                                                          const uint32_t* huge_list,
                                                          const uint32_t* counts) {
  __shared__ uint32_t s[kBlockSortMax];
  const uint32_t n_wave = counts[0], n_block = counts[1], n_huge = counts[2];
  for (uint32_t i = blockIdx.x + gridDim.x * (threadIdx.x / kWave); i < n_wave;
       i += gridDim.x * (kLongBlock / kWave)) {
    const uint32_t u = __builtin_amdgcn_readfirstlane(wave_list[i]);
    const uint32_t beg = fstart[u], len = fstart[u + 1] - beg;
    if (len <= 64)
      wave_sort_regs<1>(dag_col, fence, beg, len);
    else if (len <= 128)
      wave_sort_regs<2>(dag_col, fence, beg, len);
    else if (len <= 256)
      wave_sort_regs<4>(dag_col, fence, beg, len);
    else if (len <= 512)
      wave_sort_regs<8>(dag_col, fence, beg, len);
    else if (len <= 1024)
      wave_sort_regs<16>(dag_col, fence, beg, len);
    else
      wave_sort_regs<32>(dag_col, fence, beg, len);
  }
  // one block per row (2048 < len <= 4096): bitonic sort in LDS
  for (uint32_t i = blockIdx.x; i < n_block; i += gridDim.x) {
    const uint32_t beg = fstart[block_list[i]], len = fstart[block_list[i] + 1] - beg;
    const uint32_t P = pow2_ceil(len);
    for (uint32_t k = threadIdx.x; k < P; k += kLongBlock) s[k] = k < len ? dag_col[beg + k] : kPad;
    __syncthreads();
    for (uint32_t k = 2; k <= P; k <<= 1) {
      for (uint32_t j = k >> 1; j > 0; j >>= 1) {
        for (uint32_t t = threadIdx.x; t < P / 2; t += kLongBlock) {
          const uint32_t a = ((t & ~(j - 1)) << 1) | (t & (j - 1));
          const uint32_t b = a | j;
          const bool up = (a & k) == 0;
          const uint32_t va = s[a], vb = s[b];
          if ((va > vb) == up) {
            s[a] = vb;
            s[b] = va;
          }
        }
        __syncthreads();
      }
    }
    for (uint32_t k = threadIdx.x; k < len; k += kLongBlock)
      put_sorted(dag_col, fence, beg + k, s[k]);
    __syncthreads();
  }
  // one block per row (len > 4096): bitonic sort in place in global memory.
  // Every merge is ascending (the first step of a merge pairs i with its
  // mirror i ^ (k-1)), so the virtual +inf padding past `len` never moves and
  // pairs that reach past the end are skipped.
  for (uint32_t i = blockIdx.x; i < n_huge; i += gridDim.x) {
    const uint32_t beg = fstart[huge_list[i]], len = fstart[huge_list[i] + 1] - beg;
    uint32_t* a = dag_col + beg;
    const uint32_t P = pow2_ceil(len);
    for (uint32_t k = 2; k <= P; k <<= 1) {
      for (uint32_t j = k >> 1; j > 0; j >>= 1) {
        for (uint32_t t = threadIdx.x; t < P / 2; t += kLongBlock) {
          const uint32_t lo = ((t & ~(j - 1)) << 1) | (t & (j - 1));
          const uint32_t hi = (j == (k >> 1)) ? (lo ^ (k - 1)) : (lo | j);
          if (hi < len) {
            const uint32_t va = a[lo], vb = a[hi];
            if (va > vb) {
              a[lo] = vb;
              a[hi] = va;
            }
          }
        }
        __threadfence_block();
        __syncthreads();
      }
    }
    for (uint32_t k = threadIdx.x; k < len; k += kLongBlock)
      if ((beg + k) % kFenceStep == 0) fence[(beg + k) / kFenceStep] = a[k];
  }
}

void sort_rows(const uint32_t* fstart, const uint32_t* rank, uint64_t n, uint64_t m, uint2* dag_rng,
               uint32_t* dag_col, uint32_t* fence, uint32_t* lists, uint32_t* counts, int num_cu,
               hipStream_t s) {
  uint32_t* wave_list = lists;
  uint32_t* block_list = lists + n;
  uint32_t* huge_list = lists + 2 * n;
  // rows per thread and step: four share the list atomics of a large graph,
  // one spreads a small one over the CUs
  const uint32_t per = n >= (1u << 18) ? 4 : 1;
  uint64_t g = (n + kBlock * per - 1) / (kBlock * per);
  if (g > 16384) g = 16384;
  if (g < 1) g = 1;
  hipLaunchKernelGGL(k_sort_short, dim3((unsigned)g), dim3(kBlock), 0, s, fstart, rank, n, dag_rng,
                     dag_col, fence, wave_list, block_list, huge_list, counts, per);
  // a wave for each row that may be listed, two blocks per CU at most (K_1500:
  // 54 us with n / 32 blocks, half as many, 32 so, 40 with a block for each;
  // K_1500,1500: 54, 35, 48; G(4000), degree 1000: 40, 24, 30)
  uint64_t rows = m / (kSortShort + 1);
  if (rows > n) rows = n;
  if (rows == 0 || n <= kSortShort) return;  // a row has fewer than n entries
  uint64_t gl = (uint64_t)(num_cu > 0 ? num_cu : 256) * 2;
  const uint64_t need = (rows + kLongBlock / kWave - 1) / (kLongBlock / kWave);
  if (gl > need) gl = need;
  hipLaunchKernelGGL(k_sort_long, dim3((unsigned)gl), dim3(kLongBlock), 0, s, fstart, dag_col,
                     fence, wave_list, block_list, huge_list, counts);
}

}  // namespace slim
