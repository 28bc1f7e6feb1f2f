// Accuracy metric of a compression (section 5): the Kullback-Leibler
// divergence D_KL(P||Q) = sum_k P(k) log2(P(k)/Q(k)) of the degree
// distribution Q of the compressed graph from the distribution P of its
// input, P(k) and Q(k) being the fractions of vertices of degree k.
//
// Two degree histograms (bins 0..n): degrees below kHistLds, where almost all
// vertices of a power-law graph fall, in LDS counters; the bins above are
// cleared, counted by a second pass over the offsets, and read, only as far
// as the largest degree.  Then the sum of the terms over the bins: per block
// in a fixed tree, then the block partials in order, so the result is
// reproducible; bins past the largest degree would add zeros.  Bound by HBM,
// 16 bytes of offsets per vertex.  Clearing and reading all n + 1 bins cost
// 32 bytes per vertex more, and 2048 blocks that each add their counters to
// the same few bins wait on those atomics: 4.2e6 vertices of degree at most
// 128 took 138 us, 39 us now.
#include <math.h>

#include "slim_batch.h"

namespace slim {

constexpr int kHistLds = 4096;   // degrees below this are counted in LDS
constexpr int kHistBlocks = 512; // most blocks per histogram
constexpr int kKlBlocks = 1024;  // most blocks of the partial sums

struct KlArgs {
  const int64_t* row_off[2];  // P, Q
  uint64_t* hist[2];
  uint64_t n;
};

// Counts are at most n < 2^32, so the high words of the bins stay 0; that of a
// bin in the middle of Q's low ones holds the largest degree of either graph
// (the workspace has no other word to spare while the partial sums are
// written).  In the bin of degree 0 it would wait on the atomics of the bins
// beside it, in the last low bin on those of P's first bins, a multiple of the
// memory channels' interleave away (4.2e6 vertices: 47.6 and 44.1 us, 38.9 here).
__device__ __forceinline__ uint32_t* top_degree(const KlArgs& a) {
  const uint64_t bin = a.n < (uint64_t)kHistLds / 2 ? a.n : (uint64_t)kHistLds / 2;
  return reinterpret_cast<uint32_t*>(a.hist[1] + bin) + 1;
}

__device__ __forceinline__ uint64_t degree_bin(const KlArgs& a, int s, uint64_t v) {
  const int64_t d = a.row_off[s][v + 1] - a.row_off[s][v];
  const uint64_t k = d > 0 ? (uint64_t)d : 0u;
  return k < a.n ? k : a.n;
}

// Clears the low bins of both histograms, the largest degree among them.
__global__ __launch_bounds__(kBlock) void k_kl_clear(KlArgs a) {
  const uint64_t i = blockIdx.x * (uint64_t)kBlock + threadIdx.x;
  if (i < (uint64_t)kHistLds && i <= a.n) a.hist[0][i] = a.hist[1][i] = 0;
}

// Degrees below kHistLds of graph blockIdx.y, and the largest degree.
__global__ __launch_bounds__(kBlock) void k_deg_hist(KlArgs a) {
  __shared__ uint32_t h[kHistLds];
  __shared__ uint32_t wtop[kWavesPerBlock];
  const int s = blockIdx.y;
  for (int i = threadIdx.x; i < kHistLds; i += kBlock) h[i] = 0;
  __syncthreads();
  uint32_t top = 0;
  for (uint64_t v = blockIdx.x * (uint64_t)kBlock + threadIdx.x; v < a.n;
       v += (uint64_t)gridDim.x * kBlock) {
    const uint64_t k = degree_bin(a, s, v);
    top = max(top, (uint32_t)k);
    if (k < (uint64_t)kHistLds) atomicAdd(&h[k], 1u);
  }
  for (int d = kWave / 2; d > 0; d >>= 1) top = max(top, (uint32_t)__shfl_xor(top, d, kWave));
  if (lane_id() == 0) wtop[threadIdx.x / kWave] = top;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < kWavesPerBlock; ++i) top = max(top, wtop[i]);
    if (top) atomicMax(top_degree(a), top);
  }
  for (int i = threadIdx.x; i < kHistLds; i += kBlock)
    if (h[i]) atomicAdd((unsigned long long*)&a.hist[s][i], (unsigned long long)h[i]);
}

// Bins from kHistLds to the largest degree (none: both kernels return).
__global__ __launch_bounds__(kBlock) void k_kl_clear_high(KlArgs a) {
  const uint64_t top = *top_degree(a);
  for (uint64_t k = kHistLds + blockIdx.x * (uint64_t)kBlock + threadIdx.x; k <= top;
       k += (uint64_t)gridDim.x * kBlock)
    a.hist[0][k] = a.hist[1][k] = 0;
}

__global__ __launch_bounds__(kBlock) void k_deg_hist_high(KlArgs a) {
  if (*top_degree(a) < (uint32_t)kHistLds) return;
  const int s = blockIdx.y;
  for (uint64_t v = blockIdx.x * (uint64_t)kBlock + threadIdx.x; v < a.n;
       v += (uint64_t)gridDim.x * kBlock) {
    const uint64_t k = degree_bin(a, s, v);
    if (k >= (uint64_t)kHistLds) atomicAdd((unsigned long long*)&a.hist[s][k], 1ull);
  }
}

__device__ __forceinline__ double block_sum(double v, double* red) {
  for (int d = kWave / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, kWave);
  const int w = threadIdx.x / kWave;
  if (lane_id() == 0) red[w] = v;
  __syncthreads();
  double t = 0;
  if (threadIdx.x == 0)
    for (int i = 0; i < kWavesPerBlock; ++i) t += red[i];
  __syncthreads();
  return t;
}

// Block b adds the terms of bins b*kBlock + i*stride + t; a bin present in
// P and absent from Q makes the term (and the sum) +infinity.
__global__ __launch_bounds__(kBlock) void k_kl_partial(KlArgs a, double inv_n, double* part) {
  __shared__ double red[kWavesPerBlock];
  const uint64_t top = *top_degree(a);
  double acc = 0;
  for (uint64_t k = blockIdx.x * (uint64_t)kBlock + threadIdx.x; k <= top;
       k += (uint64_t)gridDim.x * kBlock) {
    const uint32_t cp = (uint32_t)a.hist[0][k], cq = (uint32_t)a.hist[1][k];
    if (cp) acc += cq ? (double)cp * inv_n * log2((double)cp / (double)cq) : __builtin_inf();
  }
  const double t = block_sum(acc, red);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

__global__ __launch_bounds__(kBlock) void k_kl_final(const double* part, uint32_t nb,
                                                     double* out) {
  __shared__ double red[kWavesPerBlock];
  double acc = 0;
  for (uint32_t i = threadIdx.x; i < nb; i += kBlock) acc += part[i];
  const double t = block_sum(acc, red);
  if (threadIdx.x == 0) *out = t;
}

namespace {

struct KlLayout {
  uint64_t hp, hq, part, total;
};

KlLayout kl_layout(uint64_t n) {
  KlLayout L{};
  auto al = [](uint64_t x) { return (x + 255) / 256 * 256; };
  L.hp = 0;
  L.hq = al(L.hp + 8 * (n + 1));
  L.part = al(L.hq + 8 * (n + 1));
  L.total = al(L.part + 8 * (uint64_t)kKlBlocks);
  return L;
}

}  // namespace
}  // namespace slim

using namespace slim;

extern "C" {

int slim_degree_kl_workspace(uint64_t n, uint64_t* bytes) {
  if (!bytes) return fail(SLIM_EINVAL, "bytes is NULL");
  if (n > 0xffffffffull) return fail(SLIM_EINVAL, "n = %llu exceeds 2^32-1", (unsigned long long)n);
  *bytes = kl_layout(n).total;
  return ok();
}

int slim_degree_kl(const int64_t* d_row_off_p, const int64_t* d_row_off_q, uint64_t n,
                   void* d_ws, uint64_t ws_bytes, double* d_out, void* stream) {
  if (!d_out) return fail(SLIM_EINVAL, "d_out is NULL");
  if (!d_row_off_p || !d_row_off_q) return fail(SLIM_EINVAL, "row offsets are NULL");
  if (n > 0xffffffffull) return fail(SLIM_EINVAL, "n = %llu exceeds 2^32-1", (unsigned long long)n);
  const KlLayout L = kl_layout(n);
  if (ws_bytes < L.total)
    return fail(SLIM_ENOMEM, "workspace has %llu bytes, %llu needed", (unsigned long long)ws_bytes,
                (unsigned long long)L.total);
  if (!d_ws) return fail(SLIM_EINVAL, "d_ws is NULL");
  if (reinterpret_cast<uintptr_t>(d_ws) % 256) return fail(SLIM_EINVAL, "d_ws must be 256-byte aligned");
  hipStream_t s = static_cast<hipStream_t>(stream);
  (void)hipGetLastError();
  char* ws = static_cast<char*>(d_ws);
  double* part = reinterpret_cast<double*>(ws + L.part);
  const uint64_t bins = n + 1;
  uint32_t nb = 0;
  if (n > 0) {
    KlArgs a{{d_row_off_p, d_row_off_q},
             {reinterpret_cast<uint64_t*>(ws + L.hp), reinterpret_cast<uint64_t*>(ws + L.hq)},
             n};
    uint64_t g = (n + kBlock - 1) / kBlock;
    const unsigned all = (unsigned)(g < 2048 ? g : 2048);
    if (g > (uint64_t)kHistBlocks) g = kHistBlocks;
    hipLaunchKernelGGL(k_kl_clear, dim3(kHistLds / kBlock), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(k_deg_hist, dim3((unsigned)g, 2), dim3(kBlock), 0, s, a);
    if (n >= (uint64_t)kHistLds) {
      hipLaunchKernelGGL(k_kl_clear_high, dim3(all), dim3(kBlock), 0, s, a);
      hipLaunchKernelGGL(k_deg_hist_high, dim3(all, 2), dim3(kBlock), 0, s, a);
    }
    uint64_t b = (bins + kBlock - 1) / kBlock;
    if (b > (uint64_t)kKlBlocks) b = kKlBlocks;
    nb = (uint32_t)b;
    hipLaunchKernelGGL(k_kl_partial, dim3(nb), dim3(kBlock), 0, s, a, 1.0 / (double)n, part);
  }
  hipLaunchKernelGGL(k_kl_final, dim3(1), dim3(kBlock), 0, s, part, nb, d_out);
  return hip_check("slim_degree_kl");
}

}  // extern "C"
