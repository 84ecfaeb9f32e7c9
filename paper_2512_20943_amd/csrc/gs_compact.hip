// Low-opacity culling for keyframe reconstruction (AirGS Sec. III-B: the
// Gaussians whose opacity has fallen below a threshold are discarded during
// training) as an order-preserving stream compaction, and the gather that
// applies the resulting index list to parameter or optimizer-state planes.
//
// Compaction over chunks of 1024 Gaussians: count the kept ones per chunk,
// then rank inside each chunk with wave ballots and write the kept indices in
// their original order.  Up to kSumChunks chunks every workgroup of the
// second launch adds up the counts before its own; beyond, a launch in
// between scans them.  4 B are read twice and at most 4 B written per
// Gaussian, so at ordinary sizes the launches are what it costs.
#include <algorithm>
#include <cmath>

#include "gs_internal.h"

namespace gs {
namespace {

constexpr int kChunk = 1024;  // Gaussians per workgroup (256 threads x 4)

__device__ __forceinline__ bool kept(const float* logit, int i, int n, double thr) {
  return i < n && (double)logit[i] >= thr;
}

__global__ __launch_bounds__(256) void k_keep_count(const float* __restrict__ logit, int n,
                                                    double thr, uint32_t* __restrict__ counts) {
  const int base = blockIdx.x * kChunk;
  int c = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) c += kept(logit, base + k * 256 + threadIdx.x, n, thr) ? 1 : 0;
  for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off, 64);
  __shared__ int s[4];
  if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) counts[blockIdx.x] = (uint32_t)(s[0] + s[1] + s[2] + s[3]);
}

// Exclusive scan of nb chunk counts in one workgroup of 1024 threads.
__global__ __launch_bounds__(1024) void k_keep_scan(uint32_t* __restrict__ counts, int nb) {
  __shared__ uint32_t s_wave[16];
  __shared__ uint32_t s_carry;
  if (threadIdx.x == 0) s_carry = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int base = 0; base < nb; base += 1024) {
    const int i = base + threadIdx.x;
    const uint32_t v = i < nb ? counts[i] : 0u;
    uint32_t x = v;  // inclusive scan inside the wave
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t y = __shfl_up(x, off, 64);
      if (lane >= off) x += y;
    }
    if (lane == 63) s_wave[wave] = x;
    __syncthreads();
    uint32_t before = s_carry;
    for (int w = 0; w < wave; ++w) before += s_wave[w];
    if (i < nb) counts[i] = before + x - v;
    __syncthreads();
    if (threadIdx.x == 1023) s_carry = before + x;
    __syncthreads();
  }
}

// SUM: offsets holds the chunk counts, else their scan.  The last workgroup
// writes the number kept to host memory, for a host that waits for the stream:
// the other workgroups may still be reading the counts and writing indices.
template <bool SUM>
__global__ __launch_bounds__(256) void k_keep_write(const float* __restrict__ logit, int n,
                                                    double thr,
                                                    const uint32_t* __restrict__ offsets,
                                                    int32_t* __restrict__ index,
                                                    uint32_t* __restrict__ total) {
  __shared__ uint32_t s_cnt[16];
  __shared__ uint32_t s_sum[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int base = blockIdx.x * kChunk;
  // pass k covers Gaussians base + k*256 + [0, 256): 4 waves of 64, so the
  // rank of a lane is (waves of earlier passes) + (earlier waves of this
  // pass) + (earlier lanes of its own wave)
  bool f[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    f[k] = kept(logit, base + k * 256 + threadIdx.x, n, thr);
    const uint64_t b = __ballot(f[k]);
    if (lane == 0) s_cnt[k * 4 + wave] = (uint32_t)__popcll(b);
  }
  if constexpr (SUM) {
    uint32_t x = 0;
    for (uint32_t c = threadIdx.x; c < blockIdx.x; c += 256) x += offsets[c];
    for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
    if (lane == 0) s_sum[wave] = x;
  }
  __syncthreads();
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
  uint32_t run = SUM ? (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]) : offsets[blockIdx.x];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint64_t b = __ballot(f[k]);
    uint32_t pre = run;
    for (int w = 0; w < wave; ++w) pre += s_cnt[k * 4 + w];
    if (f[k]) index[pre + (uint32_t)__popcll(b & below)] = base + k * 256 + threadIdx.x;
    for (int w = 0; w < 4; ++w) run += s_cnt[k * 4 + w];
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total = run;
}

// Planes per thread of the gather: their loads are in flight together, and
// the planes' groups are the grid's second dimension.  59 planes of 270 k
// kept Gaussians (135 MB, 28 us at the copy rate): 28.9 us, 37.8 with one
// thread for all planes.
constexpr int kGatherPlanes = 8;

__global__ __launch_bounds__(256) void k_gather(const float* __restrict__ src, int64_t src_ld,
                                                int planes, const int32_t* __restrict__ index,
                                                int m, float* __restrict__ dst, int64_t dst_ld) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= m) return;
  const int64_t i = index[j];
  const int p0 = (int)blockIdx.y * kGatherPlanes;
  const int count = min(kGatherPlanes, planes - p0);
  src += (int64_t)p0 * src_ld + i;
  dst += (int64_t)p0 * dst_ld + j;
  float x[kGatherPlanes];
#pragma unroll
  for (int p = 0; p < kGatherPlanes; ++p)
    if (p < count) x[p] = src[p * src_ld];
#pragma unroll
  for (int p = 0; p < kGatherPlanes; ++p)
    if (p < count) dst[p * dst_ld] = x[p];
}

// Chunks up to which the second launch adds the counts up itself, in us with
// and without the scan: 0.3 M Gaussians 21.4 / 19.6, 4 M 30.8 / 28.5, 8 M
// 45.6 / 46.8 (the additions grow with the square).
constexpr int kSumChunks = 4096;

}  // namespace

size_t keep_workspace_bytes(int n) {
  const size_t nb = ((size_t)n + kChunk - 1) / kChunk;
  return (nb + 1) * sizeof(uint32_t);
}

double opacity_logit_threshold(float min_opacity) {
  const double m = (double)min_opacity;
  return std::log(m / (1.0 - m));
}

void launch_keep_low_opacity(const float* logit, int n, double thr, int32_t* index, void* ws,
                             uint32_t* total, hipStream_t s) {
  const int nb = (n + kChunk - 1) / kChunk;
  if (nb == 0) return;
  uint32_t* counts = static_cast<uint32_t*>(ws);
  StageScope scope(kStCompact, s);
  hipLaunchKernelGGL(k_keep_count, dim3(nb), dim3(256), 0, s, logit, n, thr, counts);
  const bool sum = nb <= kSumChunks;
  if (!sum) hipLaunchKernelGGL(k_keep_scan, dim3(1), dim3(1024), 0, s, counts, nb);
  hipLaunchKernelGGL(sum ? k_keep_write<true> : k_keep_write<false>, dim3(nb), dim3(256), 0, s,
                     logit, n, thr, (const uint32_t*)counts, index, total);
}

void launch_gather(const float* src, int64_t src_ld, int planes, const int32_t* index, int m,
                   float* dst, int64_t dst_ld, hipStream_t s) {
  if (m <= 0 || planes <= 0) return;
  StageScope scope(kStCompact, s);
  // a grid's second dimension holds 65,535 groups of planes
  constexpr int64_t kMost = 65535 * kGatherPlanes;
  for (int64_t p = 0; p < planes; p += kMost) {
    const int count = (int)std::min<int64_t>(kMost, planes - p);
    const dim3 grid((m + 255) / 256, (count + kGatherPlanes - 1) / kGatherPlanes);
    hipLaunchKernelGGL(k_gather, grid, dim3(256), 0, s, src + p * src_ld, src_ld, count, index, m,
                       dst + p * dst_ld, dst_ld);
  }
}

}  // namespace gs
