// Residual bookkeeping of sent updates and their quantised planes (AirGS
// Sec. III-C, Eq. (11), (12)).
//
// The server keeps the true accumulated delta D_t of the frame and the sum
// D'_(t-1) of what the client has already received.  The update sent for
// frame t is the pruning mask applied to the residual D_t - D'_(t-1), so the
// motion of a pruned Gaussian is not lost but sent with a later frame.  Sent
// updates travel as signed 8- or 16-bit codes with one scale per channel
// (symmetric, so a pruned texel stays exactly zero); both ends add the
// dequantised update to D' so that they hold bit-identical sums, and the
// client applies D'_t to the anchor in the same pass.
//
// Elementwise, HBM-bound, FP32 planes, one IEEE operation per step and
// contraction off so that every step rounds the way it is written.
#include "gs_internal.h"

namespace gs {
namespace {

#pragma clang fp contract(off)

constexpr int kChannels = 8;

// N consecutive values as one access (N = 4: 16-B aligned floats, 4- or 8-B
// aligned codes).
template <int N, typename T>
struct alignas(N * sizeof(T)) Pack {
  T x[N];
};
template <int N, typename T>
__device__ __forceinline__ Pack<N, T> load_pack(const T* p) {
  return *reinterpret_cast<const Pack<N, T>*>(p);
}
template <int N, typename T>
__device__ __forceinline__ void store_pack(T* p, const Pack<N, T>& v) {
  *reinterpret_cast<Pack<N, T>*>(p) = v;
}

// The kernels move about 100 B per texel and compute next to nothing with
// it, so what counts at a frame's 300 k texels is the loads in flight.  The
// residual and the quantisation take four consecutive texels per thread (N =
// 4, 16 B a load; N = 1 serves planes and buffers that do not keep that
// alignment) of some of the channels.

// d = mask ? D - P : 0 for texels i < n, 0 elsewhere; per-channel max |d|
// over i < n accumulated as the bits of a non-negative float.  One atomic
// instruction per workgroup raises the eight maxima; they share a cache line
// where those serialise (11 ns each), so a workgroup is large: half of its
// threads take channels 0-3, the others 4-7 of the same texels.  21 -> 8 us
// for 300 k texels; one workgroup per channel and 1,024 texels took 60.
constexpr int kResidualThreads = 1024;

template <int N>
__global__ __launch_bounds__(kResidualThreads) void k_residual(
    const float* __restrict__ D, const float* __restrict__ P, const uint8_t* __restrict__ mask,
    int n, size_t plane, float* __restrict__ d, uint32_t* __restrict__ absmax_bits) {
  constexpr int kHalf = kResidualThreads / 2, kOwn = kChannels / 2;
  const int half = threadIdx.x / kHalf;
  const size_t t = ((size_t)blockIdx.x * kHalf + threadIdx.x % kHalf) * N;
  const size_t first = (size_t)half * kOwn * plane + t;
  uint32_t most[kOwn] = {0u, 0u, 0u, 0u};
  if (t + N <= plane) {
    Pack<N, float> a[kOwn], b[kOwn];
#pragma unroll
    for (int c = 0; c < kOwn; ++c) {
      a[c] = load_pack<N>(D + first + c * plane);
      b[c] = load_pack<N>(P + first + c * plane);
    }
    // the mask counts at texels i < n only, and may end there
    Pack<N, uint8_t> m{};
    if (t + N <= (size_t)n) {
      m = load_pack<N>(mask + t);
    } else {
#pragma unroll
      for (int k = 0; k < N; ++k)
        if (t + k < (size_t)n) m.x[k] = mask[t + k];
    }
#pragma unroll
    for (int c = 0; c < kOwn; ++c) {
      Pack<N, float> v;
#pragma unroll
      for (int k = 0; k < N; ++k) {
        v.x[k] = t + k < (size_t)n && m.x[k] != 0 ? a[c].x[k] - b[c].x[k] : 0.f;
        most[c] = max(most[c], __float_as_uint(fabsf(v.x[k])));
      }
      store_pack<N>(d + first + c * plane, v);
    }
  }
  constexpr int kWaves = kResidualThreads / 64;
  __shared__ uint32_t s_max[kWaves][kOwn];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int c = 0; c < kOwn; ++c) {
    uint32_t m = most[c];
    for (int off = 32; off >= 1; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, 64));
    if (lane == 0) s_max[wave][c] = m;
  }
  __syncthreads();
  if (threadIdx.x < kChannels) {
    const int c = threadIdx.x;
    uint32_t m = 0u;
    for (int w = 0; w < kWaves / 2; ++w) m = max(m, s_max[c / kOwn * (kWaves / 2) + w][c % kOwn]);
    if (m) atomicMax(absmax_bits + c, m);
  }
}

// 9.3 -> 6.0 us for 300 k texels against a thread per texel that walked the
// eight channels.
template <int N, typename Q>
__global__ __launch_bounds__(256) void k_quantize(const float* __restrict__ d,
                                                  const float* __restrict__ absmax, float qmax,
                                                  int n, size_t plane, Q* __restrict__ q,
                                                  float* __restrict__ scale_out,
                                                  float* __restrict__ P) {
  const size_t t = ((size_t)blockIdx.x * 256 + threadIdx.x) * N;
  if (t + N > plane) return;
  const int c = blockIdx.y;
  const Pack<N, float> v = load_pack<N>(d + c * plane + t);
  Pack<N, float> p{};
  if (P) p = load_pack<N>(P + c * plane + t);
  const float a = absmax[c];
  const float sc = a > 0.f ? a / qmax : 0.f;
  if (t == 0) scale_out[c] = sc;
  Pack<N, Q> out;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    float code = 0.f;
    const bool in = t + k < (size_t)n;
    if (in && sc > 0.f) code = fminf(fmaxf(rintf(v.x[k] / sc), -qmax), qmax);
    out.x[k] = (Q)code;
    if (in) p.x[k] = p.x[k] + code * sc;
  }
  store_pack<N>(q + c * plane + t, out);
  if (P) store_pack<N>(P + c * plane + t, p);
}

// Client side: P += code * scale at texels i < n, then the frame is the
// anchor with P applied (all texels, as the frame-update apply with a full
// mask; FP64 arithmetic rounded once to FP32).
// All loads go out before the first store; four texels per thread were
// slower (8.1 against 7.6 us for 300 k).
template <typename Q>
__global__ __launch_bounds__(256) void k_apply_quantized(
    int n, int ld, size_t plane, const Q* __restrict__ q, const float* __restrict__ scale,
    float* __restrict__ P, const float* __restrict__ mean, const float* __restrict__ quat,
    const float* __restrict__ opac, float* __restrict__ mean_o, float* __restrict__ quat_o,
    float* __restrict__ opac_o) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const size_t L = (size_t)ld;
  Q code[kChannels];
  float u[kChannels];
#pragma unroll
  for (int c = 0; c < kChannels; ++c) {
    code[c] = q[c * plane + i];
    u[c] = P[c * plane + i];
  }
  const float m[3] = {mean[i], mean[L + i], mean[2 * L + i]};
  const double bw = quat[i], bx = quat[L + i], by = quat[2 * L + i], bz = quat[3 * L + i];
  const float o = opac[i];
#pragma unroll
  for (int c = 0; c < kChannels; ++c) {
    u[c] = u[c] + (float)code[c] * scale[c];
    P[c * plane + i] = u[c];
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) mean_o[c * L + i] = (float)((double)m[c] + (double)u[c]);
  const double aw = u[3], ax = u[4], ay = u[5], az = u[6];
  quat_o[i] = (float)(((aw * bw - ax * bx) - ay * by) - az * bz);
  quat_o[L + i] = (float)(((aw * bx + ax * bw) + ay * bz) - az * by);
  quat_o[2 * L + i] = (float)(((aw * by - ax * bz) + ay * bw) + az * bx);
  quat_o[3 * L + i] = (float)(((aw * bz + ax * by) - ay * bx) + az * bw);
  opac_o[i] = (float)((double)o + (double)u[7]);
}

// Whether the pointers allow accesses of `bytes` bytes.
template <typename... T>
bool aligned_to(size_t bytes, const T*... p) {
  return ((reinterpret_cast<uintptr_t>(p) % bytes == 0) && ...);
}

}  // namespace

void launch_residual(const float* D, const float* P, const uint8_t* mask, int n, int gw, int gh,
                     float* d, float* absmax, hipStream_t s) {
  const size_t plane = (size_t)gw * (size_t)gh;
  if (plane == 0) return;
  StageScope scope(kStResidual, s);
  const bool four = plane % 4 == 0 && aligned_to(16, D, P, d) && aligned_to(4, mask);
  const size_t groups = four ? plane / 4 : plane;
  constexpr size_t kPer = kResidualThreads / 2;
  hipLaunchKernelGGL(four ? k_residual<4> : k_residual<1>,
                     dim3((unsigned)((groups + kPer - 1) / kPer)), dim3(kResidualThreads), 0, s, D,
                     P, mask, n, plane, d, reinterpret_cast<uint32_t*>(absmax));
}

namespace {
template <typename Q>
void quantize(const float* d, const float* absmax, float qmax, int n, size_t plane, Q* q,
              float* scale, float* P, hipStream_t s) {
  const bool four = plane % 4 == 0 && aligned_to(16, d, P) && aligned_to(4 * sizeof(Q), q);
  const size_t groups = four ? plane / 4 : plane;
  hipLaunchKernelGGL((four ? k_quantize<4, Q> : k_quantize<1, Q>),
                     dim3((unsigned)((groups + 255) / 256), kChannels), dim3(256), 0, s, d,
                     absmax, qmax, n, plane, q, scale, P);
}
}  // namespace

void launch_quantize(const float* d, const float* absmax, int bits, int n, int gw, int gh,
                     void* q, float* scale, float* P, hipStream_t s) {
  const size_t plane = (size_t)gw * (size_t)gh;
  if (plane == 0) return;
  StageScope scope(kStResidual, s);
  const float qmax = (float)((1 << (bits - 1)) - 1);
  if (bits == 8)
    quantize(d, absmax, qmax, n, plane, static_cast<int8_t*>(q), scale, P, s);
  else
    quantize(d, absmax, qmax, n, plane, static_cast<int16_t*>(q), scale, P, s);
}

void launch_apply_quantized(const gs_gaussians& a, const void* q, int bits, const float* scale,
                            float* P, int gw, int gh, gs_gaussians& f, hipStream_t s) {
  const size_t plane = (size_t)gw * (size_t)gh;
  const int blocks = (a.n + 255) / 256;
  if (blocks == 0) return;
  StageScope scope(kStResidual, s);
  if (bits == 8)
    hipLaunchKernelGGL(k_apply_quantized<int8_t>, dim3(blocks), dim3(256), 0, s, a.n, a.ld, plane,
                       static_cast<const int8_t*>(q), scale, P, a.mean, a.quat, a.opacity, f.mean,
                       f.quat, f.opacity);
  else
    hipLaunchKernelGGL(k_apply_quantized<int16_t>, dim3(blocks), dim3(256), 0, s, a.n, a.ld,
                       plane, static_cast<const int16_t*>(q), scale, P, a.mean, a.quat, a.opacity,
                       f.mean, f.quat, f.opacity);
}

}  // namespace gs
