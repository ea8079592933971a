// The norm of one row, shared by the norm kernel and by the slice reduction that norms the rows it completes.
#pragma once
#include "qzo_device.hpp"
#include "qzo_kernels.hpp"
#include "qzo_nibble.hpp"

namespace qzo {

// Sum over the first 256 threads of a workgroup (every thread takes part in the barriers): wavefront-shuffle
// reduction, fixed order across the four wavefronts.
__device__ __forceinline__ float block_sum(float v, float* red) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0 && threadIdx.x < 256) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// Row `row` of `rows`, d features, to its place in y; chunk(i, c): 16-byte chunk c = thread + 256 i of the row (any value beyond it).
// fp32 statistics by the first 256 threads; the others only take part in the barriers.
// CACHED: the row fits four chunks per thread.  xsum_t (nullable): block sums of the output, [d/128][rows].  pack: both as
// the few-token kernel takes them.
template <bool LAYERNORM, bool CACHED, class Chunk>
__device__ __forceinline__ void norm_row(const Chunk& chunk, const bf16_t* __restrict__ gain, const bf16_t* __restrict__ bias,
                                         uint32_t d, float eps, bf16_t* __restrict__ y, float* __restrict__ xsum_t,
                                         uint32_t row, uint32_t rows, const XPack& pack, float* red) {
  const uint32_t cpr = threadIdx.x < 256 ? d >> 3 : 0u;
  constexpr int NC = 4;
  const uint32_t passes = CACHED ? NC : ((d >> 3) + 255) / 256;
  float mu = 0.0f;
  if (LAYERNORM) {
    float acc = 0.0f;
#pragma unroll
    for (uint32_t i = 0; i < passes; ++i) {
      const uint32_t c = threadIdx.x + 256u * i;
      if (c < cpr) {
        const uint4 v = chunk(i, c);
        const uint32_t a[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) acc += __uint_as_float(a[j] << 16) + __uint_as_float(a[j] & 0xffff0000u);
      }
    }
    mu = block_sum(acc, red) / (float)d;
  }
  float ss = 0.0f;
#pragma unroll
  for (uint32_t i = 0; i < passes; ++i) {
    const uint32_t c = threadIdx.x + 256u * i;
    if (c < cpr) {
      const uint4 v = chunk(i, c);
      const uint32_t a[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float lo = __uint_as_float(a[j] << 16) - mu, hi = __uint_as_float(a[j] & 0xffff0000u) - mu;
        ss = __builtin_fmaf(lo, lo, ss);
        ss = __builtin_fmaf(hi, hi, ss);
      }
    }
  }
  const float var = block_sum(ss, red) / (float)d;
  const float inv = 1.0f / sqrtf(var + eps);
#pragma unroll
  for (uint32_t i = 0; i < passes; ++i) {
    const uint32_t c = threadIdx.x + 256u * i;
    uint32_t o[4] = {0, 0, 0, 0};
    if (c < cpr) {
      const uint4 v = chunk(i, c);
      uint4 gq = *reinterpret_cast<const uint4*>(gain + c * 8);
      uint32_t a[4] = {v.x, v.y, v.z, v.w}, g[4] = {gq.x, gq.y, gq.z, gq.w}, b[4] = {0, 0, 0, 0};
      if (LAYERNORM) {
        uint4 bq = *reinterpret_cast<const uint4*>(bias + c * 8);
        b[0] = bq.x; b[1] = bq.y; b[2] = bq.z; b[3] = bq.w;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float lo = (__uint_as_float(a[j] << 16) - mu) * inv * __uint_as_float(g[j] << 16);
        float hi = (__uint_as_float(a[j] & 0xffff0000u) - mu) * inv * __uint_as_float(g[j] & 0xffff0000u);
        if (LAYERNORM) {
          lo += __uint_as_float(b[j] << 16);
          hi += __uint_as_float(b[j] & 0xffff0000u);
        }
        o[j] = pack_bf16x2(lo, hi);
      }
      if (pack.rows) *reinterpret_cast<u32x4*>((unsigned char*)y + pack.chunk(row, c)) = permute8(u32x4{o[0], o[1], o[2], o[3]});
      else *reinterpret_cast<uint4*>(y + (uint64_t)row * d + c * 8) = make_uint4(o[0], o[1], o[2], o[3]);
    }
    if (xsum_t) {
      // block sums of the row's output for a few-token linear that reads it: the 16 chunks of 128 features
      // sit in 16 consecutive lanes (every lane takes part: lanes beyond the row add zero)
      float lo = 0.0f, hi = 0.0f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        lo += __uint_as_float(o[j] << 16);
        hi += __uint_as_float(o[j] & 0xffff0000u);
      }
      float sx = lo + hi;
      sx += __shfl_xor(sx, 1, 64); sx += __shfl_xor(sx, 2, 64);
      sx += __shfl_xor(sx, 4, 64); sx += __shfl_xor(sx, 8, 64);
      if (c < cpr && (c & 15u) == 0u)
        xsum_t[(uint64_t)(c >> 4) * (pack.rows ? pack.rows : rows) + (pack.rows ? pack.tile_row(row) : row)] = sx;
    }
  }
}

}  // namespace qzo
