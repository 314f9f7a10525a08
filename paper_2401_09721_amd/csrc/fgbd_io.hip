// Steps on either side of the per-frame path.
//
// Quantisation (Sec. 2.2 takes integer voxel coordinates; a capture with float
// coordinates is first brought onto a 2^b grid): one isotropic scale for the
// three axes so the shape is not distorted,
//   lo_c = min_i x_ic,  ext = max_c (max_i x_ic - lo_c),  s = 2^b / ext,
//   g_ic = min(floor((x_ic - lo_c) s), 2^b - 1),
// in FP64 with IEEE division, so the result is fixed to the bit.  Points that
// fall on one voxel are all kept (the scan-line graph handles equal
// coordinates as neighbours at distance 0).  Bounds: per-block minima and
// maxima of order-preserving 32-bit keys, combined with integer atomics (exact
// and order-free); NaN coordinates take no part in the bounds and map to 0.
//
// Geometry as the signal: the integer coordinates as float32, which the
// filter then smooths like colours.
//
// Output rounding: colours to uint8 by round-half-to-even and clipping to
// 0..255 (NaN to 0).
#include "fgbd_internal.h"

namespace fgbd {

namespace {

// Monotone map of float onto uint32: a < b (as floats, not NaN) iff key(a) < key(b).
__device__ __forceinline__ uint32_t order_key(float x) {
  const uint32_t u = __float_as_uint(x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_value(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

__global__ void k_bounds_init(uint32_t *__restrict__ keys) {
  const int t = threadIdx.x;
  if (t < 6) keys[t] = t < 3 ? 0xffffffffu : 0u;  // minima start high, maxima low
}

// Bound by the atomics, all on six words of one line (about 5 ns each): few,
// large blocks, and a block adds its bound only where it is past the one it
// reads there (a value read early only costs an atomic).  700k points: 17 us
// with six atomics from each of 512 blocks of 256 threads, 7.6 with this.
constexpr int kBoundsThreads = 1024;
constexpr int kBoundsGrid = 128;
__global__ __launch_bounds__(kBoundsThreads) void k_bounds(const float *__restrict__ xyz, int64_t n, uint32_t *keys) {
  __shared__ uint32_t s_k[kBoundsThreads / kWave][6];
  uint32_t mn[3] = {0xffffffffu, 0xffffffffu, 0xffffffffu}, mx[3] = {0u, 0u, 0u};
  constexpr int U = 4;  // points in flight per thread
  const int64_t stride = (int64_t)gridDim.x * kBoundsThreads;
  for (int64_t i0 = (int64_t)blockIdx.x * kBoundsThreads + threadIdx.x; i0 < n; i0 += U * stride) {
    float x[U][3];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = min(i0 + u * stride, n - 1);  // (the last point again changes nothing)
#pragma unroll
      for (int c = 0; c < 3; ++c) x[u][c] = xyz[3 * i + c];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const bool num = x[u][c] == x[u][c];
        const uint32_t k = order_key(x[u][c]);
        mn[c] = min(mn[c], num ? k : 0xffffffffu);
        mx[c] = max(mx[c], num ? k : 0u);
      }
    }
  }
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      mn[c] = min(mn[c], (uint32_t)__shfl_xor((int)mn[c], o, kWave));
      mx[c] = max(mx[c], (uint32_t)__shfl_xor((int)mx[c], o, kWave));
    }
  }
  const int t = threadIdx.x;
  if (lane_id() == 0) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      s_k[t / kWave][c] = mn[c];
      s_k[t / kWave][3 + c] = mx[c];
    }
  }
  __syncthreads();
  if (t < 6) {
    uint32_t k = s_k[0][t];
    for (int w = 1; w < kBoundsThreads / kWave; ++w) k = t < 3 ? min(k, s_k[w][t]) : max(k, s_k[w][t]);
    const uint32_t now = __hip_atomic_load(&keys[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (t < 3) {
      if (k < now) atomicMin(&keys[t], k);
    } else if (k > now) {
      atomicMax(&keys[t], k);
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_quantize(const float *__restrict__ xyz, int64_t n, int bits,
                                                     const uint32_t *__restrict__ keys, int32_t *__restrict__ out,
                                                     double *__restrict__ frame) {
  double lo[3], ext = 0.0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    lo[c] = (double)key_value(keys[c]);
    const double e = (double)key_value(keys[3 + c]) - lo[c];
    ext = e > ext ? e : ext;  // NaN (no finite value on an axis) never wins
  }
  const double cells = (double)(1 << bits);
  const double s = ext > 0.0 ? cells / ext : 0.0;
  const int32_t top = (1 << bits) - 1;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    frame[0] = lo[0];
    frame[1] = lo[1];
    frame[2] = lo[2];
    frame[3] = s;
  }
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double v = ((double)xyz[3 * i + c] - lo[c]) * s;
      int32_t g = 0;
      if (v >= 0.0) g = v < cells ? (int32_t)floor(v) : top;  // NaN fails the test: 0
      out[3 * i + c] = g < top ? g : top;
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_round_u8(const float *__restrict__ x, int64_t m,
                                                     uint8_t *__restrict__ out) {
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  for (int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x; e < m; e += stride) {
    const float v = rintf(x[e]);
    out[e] = v >= 0.0f ? (v < 255.0f ? (uint8_t)v : (uint8_t)255) : (uint8_t)0;
  }
}

__global__ __launch_bounds__(kBlock) void k_coords_f32(const int32_t *__restrict__ g, int64_t m,
                                                       float *__restrict__ out) {
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  for (int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x; e < m; e += stride) out[e] = (float)g[e];
}

int grid_for(int64_t items) {
  const int64_t b = (items + kBlock - 1) / kBlock;
  return (int)(b < 1 ? 1 : (b > 4096 ? 4096 : b));
}

}  // namespace

hipError_t launch_quantize(const float *xyz, int64_t n, int32_t bits, int32_t *out, double *frame, uint32_t *keys,
                           hipStream_t st) {
  k_bounds_init<<<1, 64, 0, st>>>(keys);
  if (n > 0) {
    const int64_t gb = (n + kBoundsThreads - 1) / kBoundsThreads;
    k_bounds<<<(int)(gb < kBoundsGrid ? gb : kBoundsGrid), kBoundsThreads, 0, st>>>(xyz, n, keys);
  }
  k_quantize<<<grid_for(n), kBlock, 0, st>>>(xyz, n, bits, keys, out, frame);
  return hipGetLastError();
}

hipError_t launch_coords_f32(const int32_t *g, int64_t m, float *out, hipStream_t st) {
  if (m <= 0) return hipSuccess;
  k_coords_f32<<<grid_for(m), kBlock, 0, st>>>(g, m, out);
  return hipGetLastError();
}

hipError_t launch_round_u8(const float *x, int64_t m, uint8_t *out, hipStream_t st) {
  if (m <= 0) return hipSuccess;
  k_round_u8<<<grid_for(m), kBlock, 0, st>>>(x, m, out);
  return hipGetLastError();
}

}  // namespace fgbd
