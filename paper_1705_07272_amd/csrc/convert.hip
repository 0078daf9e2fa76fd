// Storage conversion of coefficient values for the reduced-precision forms:
// binary16 and bfloat16 (round to nearest even), OCP FP8 E4M3FN, int16 and
// packed 11-bit fixed point, the last three with one float32 scale per
// block of 64 values of a row (scale = max|x| / 448, / 32767, / 1023).
#include <hip/hip_fp16.h>

#include "rrt_internal.h"

namespace rrt {
namespace {

__device__ __forceinline__ uint16_t to_bf16(float x) {
  const unsigned b = __float_as_uint(x);
  if ((b & 0x7fffffffu) > 0x7f800000u) return uint16_t((b >> 16) | 0x40u);  // quiet NaN
  return uint16_t((b + 0x7fffu + ((b >> 16) & 1u)) >> 16);
}

// E4M3FN code of y (|y| <= 448 expected; larger magnitudes saturate to 448).
__device__ __forceinline__ uint8_t to_e4m3(float y) {
  const unsigned b = __float_as_uint(y);
  const unsigned sign = (b >> 24) & 0x80u;
  const float a = fabsf(y);
  unsigned code;
  if (!(a == a)) return uint8_t(sign | 0x7fu);
  if (a < 0x1p-6f) {
    code = unsigned(rintf(a * 512.0f));  // subnormal step 2^-9; 8 carries into 2^-6
  } else {
    const unsigned ab = __float_as_uint(a);
    const int eb = int(ab >> 23) - 127 + 7;  // >= 1 here
    const unsigned m23 = ab & 0x7fffffu;
    const unsigned m = (m23 + 0x7ffffu + ((m23 >> 20) & 1u)) >> 20;  // 0..8, RNE
    code = eb >= 16 ? 0x7fu : (unsigned(eb) << 3) + m;
  }
  if (code > 0x7eu) code = 0x7eu;  // saturate at 448 (0x7f is NaN)
  return uint8_t(sign | code);
}

__global__ void convert_f16(const float* __restrict__ src, __half* __restrict__ dst,
                            int64_t total) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < total) dst[i] = __float2half_rn(src[i]);
}

__global__ void convert_bf16(const float* __restrict__ src, uint16_t* __restrict__ dst,
                             int64_t total) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < total) dst[i] = to_bf16(src[i]);
}

__device__ __forceinline__ int16_t to_s16(float y) {
  const float r = rintf(fminf(fmaxf(y, -32767.0f), 32767.0f));
  return int16_t(r == r ? r : 0.0f);
}

// Block-scaled forms: one wave per (row, block of 64), one value per lane; the
// scale from a maximum over the wave; codes = round(x * M / max|x|).  (One thread per block
// read its 64 values one after the other, 256 bytes apart from its
// neighbours': 512 rows of 256 packed to 11 bits 23 -> 12 us, launch included;
// 200,000 rows 1.82 -> 0.22 ms, to 16 bits 2.18 -> 0.17 ms.)
__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, 64));
  return x;
}

constexpr int kConvThreads = 256;

template <int FORM>
__global__ __launch_bounds__(kConvThreads) void convert_blocks(const float* __restrict__ src,
                                                               void* __restrict__ dst,
                                                               float* __restrict__ scale,
                                                               int64_t rows, int cols) {
  constexpr float M = FORM == RRT_E4M3 ? 448.0f : (FORM == RRT_S11 ? 1023.0f : 32767.0f);
  const int nblk = (cols + RRT_BLOCK - 1) / RRT_BLOCK;
  const int lane = threadIdx.x & 63;
  const int64_t nt = rows * nblk;
  const int64_t waves = int64_t(gridDim.x) * (kConvThreads / 64);
  for (int64_t t = int64_t(blockIdx.x) * (kConvThreads / 64) + (threadIdx.x >> 6); t < nt;
       t += waves) {
    const int64_t row = t / nblk;
    const int blk = int(t - row * nblk);
    const int c = blk * RRT_BLOCK + lane;
    const float v = c < cols ? src[row * cols + c] : 0.0f;
    const float amax = wave_max(fabsf(v));
    const float sc = amax > 0.0f ? __fdiv_rn(amax, M) : 1.0f;
    const float inv = amax > 0.0f ? __fdiv_rn(M, amax) : 1.0f;
    const float y = v * inv;
    if constexpr (FORM == RRT_E4M3) {
      if (c < cols) static_cast<uint8_t*>(dst)[row * cols + c] = to_e4m3(y);
    } else if constexpr (FORM == RRT_S16) {
      if (c < cols) static_cast<int16_t*>(dst)[row * cols + c] = to_s16(y);
    } else {
      // the block's 64 codes fill exactly 22 words of the row's bit stream (a
      // shorter last block ends inside a word whose remaining bits stay zero);
      // lane w < 22 puts word w together from the four codes that reach into it
      const float r = rintf(fminf(fmaxf(y, -1023.0f), 1023.0f));
      const unsigned code = c < cols ? unsigned(int(r == r ? r : 0.0f)) & 0x7ffu : 0u;
      const int first = 32 * lane / 11;
      unsigned word = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const unsigned x = unsigned(__shfl(int(code), (first + j) & 63, 64));
        const int sh = 11 * (first + j) - 32 * lane;
        if (first + j < RRT_BLOCK && sh < 32) word |= sh >= 0 ? x << sh : x >> -sh;
      }
      const int64_t words = RRT_S11_WORDS(cols), w = int64_t(blk) * 22 + lane;
      if (lane < 22 && w < words) static_cast<uint32_t*>(dst)[row * words + w] = word;
    }
    if (lane == 0) scale[t] = sc;
  }
}

}  // namespace

int launch_convert(const float* src, int64_t rows, int cols, int dtype, void* dst, float* scale,
                   hipStream_t s) {
  const int64_t total = rows * cols;
  if (total == 0) return RRT_OK;
  if (dtype == RRT_F16) {
    hipLaunchKernelGGL(convert_f16, dim3(unsigned((total + 255) / 256)), dim3(256), 0, s, src,
                       static_cast<__half*>(dst), total);
  } else if (dtype == RRT_BF16) {
    hipLaunchKernelGGL(convert_bf16, dim3(unsigned((total + 255) / 256)), dim3(256), 0, s, src,
                       static_cast<uint16_t*>(dst), total);
  } else {
    const int64_t nt = rows * ((cols + RRT_BLOCK - 1) / RRT_BLOCK);
    const int64_t wanted = (nt + kConvThreads / 64 - 1) / (kConvThreads / 64);
    const dim3 grid(unsigned(wanted < (1 << 20) ? wanted : (1 << 20)));
    if (dtype == RRT_E4M3) {
      hipLaunchKernelGGL(convert_blocks<RRT_E4M3>, grid, dim3(kConvThreads), 0, s, src, dst, scale,
                         rows, cols);
    } else if (dtype == RRT_S11) {
      hipLaunchKernelGGL(convert_blocks<RRT_S11>, grid, dim3(kConvThreads), 0, s, src, dst, scale,
                         rows, cols);
    } else {
      hipLaunchKernelGGL(convert_blocks<RRT_S16>, grid, dim3(kConvThreads), 0, s, src, dst, scale,
                         rows, cols);
    }
  }
  return check_launch("convert");
}

}  // namespace rrt
