// quantize.hip -- input conversion for the precision forms.
//
// FP32 -> BF16 / F16: round to nearest even per element (the hardware
// conversions, which round to nearest even in the default mode).
// FP32 -> FP8 E4M3FN: per token, the scale s = 2^k with k the smallest
// integer such that max|x| <= 448 * 2^k (s = 1 for an all-zero token); the
// codes are E4M3FN(x * 2^-k), rounded to nearest even. Multiplying by 2^-k is
// exact, and |x * 2^-k| <= 448 so no code saturates.
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace {

__global__ __launch_bounds__(256) void copy_f32_kernel(const u32x4* __restrict__ src,
                                                       u32x4* __restrict__ dst, int64_t n16) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n16;
       i += (int64_t)gridDim.x * 256)
    dst[i] = src[i];
}

// 8 elements per thread: 32 bytes in, 16 bytes out.
template <bool BF>
__global__ __launch_bounds__(256) void to_half_kernel(const float4* __restrict__ src,
                                                      u32x4* __restrict__ dst, int64_t n8) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n8;
       i += (int64_t)gridDim.x * 256) {
    float4 a = src[2 * i], b = src[2 * i + 1];
    float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    uint32_t w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint16_t lo, hi;
      if constexpr (BF) {
        lo = __builtin_bit_cast(uint16_t, (__bf16)v[2 * j]);
        hi = __builtin_bit_cast(uint16_t, (__bf16)v[2 * j + 1]);
      } else {
        lo = __builtin_bit_cast(uint16_t, (_Float16)v[2 * j]);
        hi = __builtin_bit_cast(uint16_t, (_Float16)v[2 * j + 1]);
      }
      w[j] = (uint32_t)lo | ((uint32_t)hi << 16);
    }
    dst[i] = u32x4{w[0], w[1], w[2], w[3]};
  }
}

// Exponent k of the per-token scale, from the bits of amax (> 0, finite).
__device__ __forceinline__ int fp8_scale_exponent(float amax) {
  int bias = 0;
  if (amax < 1.17549435e-38f) {  // subnormal: renormalise exactly
    amax *= 18446744073709551616.0f;  // 2^64
    bias = 64;
  }
  uint32_t u = __float_as_uint(amax);
  int e = (int)((u >> 23) & 0xFF) - 127;
  uint32_t mant = u & 0x7FFFFF;
  // amax = 1.m * 2^e; 448 * 2^k = 1.75 * 2^(8 + k): k = e - 8 suffices iff 1.m <= 1.75
  return e - 8 + (mant > 0x600000u ? 1 : 0) - bias;
}

// Max over the G lanes of a token's lane group (G a power of two), left in
// each of them: lanes i ^ 1 and i ^ 2 by quad permutes, the other four of
// eight by a half-row mirror, the other eight of a row by a rotation, then
// the row and half-wave swaps. No LDS round trip; the whole wave executes it.
template <int G>
__device__ __forceinline__ float group_max(float v) {
  auto dpp = [](float x, auto ctrl) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x),
                                                                 decltype(ctrl)::value, 0xF, 0xF,
                                                                 false));
  };
  if constexpr (G >= 2) v = fmaxf(v, dpp(v, std::integral_constant<int, 0xB1>{}));
  if constexpr (G >= 4) v = fmaxf(v, dpp(v, std::integral_constant<int, 0x4E>{}));
  if constexpr (G >= 8) v = fmaxf(v, dpp(v, std::integral_constant<int, 0x141>{}));
  if constexpr (G >= 16) v = fmaxf(v, dpp(v, std::integral_constant<int, 0x128>{}));
  if constexpr (G >= 32) v = max_row_pairs(v);
  if constexpr (G >= 64) v = max_half_waves(v);
  return v;
}

// A token is dim / 4 pieces of four elements: lane j of its group of G lanes
// takes pieces j, j + G, ... (NP of them), so every load instruction reads 16
// consecutive bytes per lane and every store writes 4. U token groups are
// loaded before the first is converted.
// Bound: HBM (4 bytes read and 1 written per element). One token per wave,
// 4-byte loads and single-byte stores took 234 us for 1M tokens of 128
// elements (2.7 TB/s); 16-byte non-temporal loads, four in flight per lane,
// and 4-byte stores take 101 us (6.4 TB/s).
template <int G, int NP, int U>
__global__ __launch_bounds__(256) void to_fp8_kernel(const float* __restrict__ src,
                                                     uint8_t* __restrict__ dst,
                                                     float* __restrict__ scales,
                                                     int64_t n_tokens, int dim) {
  constexpr int TPW = 64 / G;         // tokens per wave and load round
  constexpr int TPB = 4 * TPW * U;    // tokens per workgroup step
  const int j = threadIdx.x % G;
  const int slot = threadIdx.x / G;   // token of a round within the workgroup
  const int pieces = dim >> 2;
  for (int64_t t0 = (int64_t)blockIdx.x * TPB; t0 < n_tokens; t0 += (int64_t)gridDim.x * TPB) {
    f32x4 v[U][NP];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t t = t0 + u * (4 * TPW) + slot;
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        v[u][p] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (t < n_tokens && j + p * G < pieces)
          v[u][p] = __builtin_nontemporal_load((const f32x4*)(src + t * dim) + j + p * G);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t t = t0 + u * (4 * TPW) + slot;
      float amax = 0.f;
#pragma unroll
      for (int p = 0; p < NP; ++p)
        amax = fmaxf(amax, fmaxf(fmaxf(fabsf(v[u][p].x), fabsf(v[u][p].y)),
                                 fmaxf(fabsf(v[u][p].z), fabsf(v[u][p].w))));
      amax = group_max<G>(amax);
      const int k = amax > 0.f ? fp8_scale_exponent(amax) : 0;
      const float inv = __uint_as_float((uint32_t)(127 - k) << 23);  // 2^-k
      if (t < n_tokens) {
        if (j == 0) scales[t] = __uint_as_float((uint32_t)(127 + k) << 23);
        uint32_t* out = (uint32_t*)(dst + t * dim);
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          if (j + p * G < pieces) {
            int w = __builtin_amdgcn_cvt_pk_fp8_f32(v[u][p].x * inv, v[u][p].y * inv, 0, false);
            w = __builtin_amdgcn_cvt_pk_fp8_f32(v[u][p].z * inv, v[u][p].w * inv, w, true);
            out[j + p * G] = (uint32_t)w;
          }
        }
      }
    }
  }
}

int grid_for(int64_t work, int per_block) {
  int64_t g = (work + per_block - 1) / per_block;
  if (g > 65536) g = 65536;
  if (g < 1) g = 1;
  return (int)g;
}

template <int G, int NP>
void launch_fp8(const float* src, uint8_t* dst, float* scales, int64_t n_tokens, int dim,
                hipStream_t s) {
  constexpr int U = 4 / NP;  // about four loads in flight per lane
  hipLaunchKernelGGL((to_fp8_kernel<G, NP, U>), dim3(grid_for(n_tokens, 4 * (64 / G) * U)),
                     dim3(256), 0, s, src, dst, scales, n_tokens, dim);
}

}  // namespace

hipError_t launch_quantize(const float* src, int64_t n_tokens, int dim, int dt, void* dst,
                           float* scales, hipStream_t s) {
  const int64_t n = n_tokens * dim;
  if (n == 0) return hipSuccess;
  switch (dt) {
    case DT_F32:
      hipLaunchKernelGGL(copy_f32_kernel, dim3(grid_for(n / 4, 256)), dim3(256), 0, s,
                         (const u32x4*)src, (u32x4*)dst, n / 4);
      break;
    case DT_BF16:
      hipLaunchKernelGGL(to_half_kernel<true>, dim3(grid_for(n / 8, 256)), dim3(256), 0, s,
                         (const float4*)src, (u32x4*)dst, n / 8);
      break;
    case DT_F16:
      hipLaunchKernelGGL(to_half_kernel<false>, dim3(grid_for(n / 8, 256)), dim3(256), 0, s,
                         (const float4*)src, (u32x4*)dst, n / 8);
      break;
    default: {
      // the smallest power-of-two lane group that holds a token in one piece
      // per lane, up to a wave; wider tokens take more pieces per lane
      const int pieces = dim / 4;
      uint8_t* d = (uint8_t*)dst;
      if (pieces <= 4)
        launch_fp8<4, 1>(src, d, scales, n_tokens, dim, s);
      else if (pieces <= 8)
        launch_fp8<8, 1>(src, d, scales, n_tokens, dim, s);
      else if (pieces <= 16)
        launch_fp8<16, 1>(src, d, scales, n_tokens, dim, s);
      else if (pieces <= 32)
        launch_fp8<32, 1>(src, d, scales, n_tokens, dim, s);
      else if (pieces <= 64)
        launch_fp8<64, 1>(src, d, scales, n_tokens, dim, s);
      else if (pieces <= 128)
        launch_fp8<64, 2>(src, d, scales, n_tokens, dim, s);
      else if (pieces <= 192)
        launch_fp8<64, 3>(src, d, scales, n_tokens, dim, s);
      else
        launch_fp8<64, 4>(src, d, scales, n_tokens, dim, s);
    }
      break;
  }
  return hipGetLastError();
}
