// Learned transport decoder (not part of the paper): positional encoding, the
// network for inference (decode_kernel) and for training (forward_kernel,
// back_kernel, grad_kernel), MSE loss and Adam.
//
// Weights and the layers' inputs are bfloat16, products are summed in FP32 by
// the matrix cores (v_mfma_f32_32x32x16_bf16, wave64) in steps of 16 of the
// inner index, in order: the same value is the same bits in every kernel.
#include <hip/hip_fp16.h>

#include "rrt_internal.h"

namespace rrt {
namespace {

constexpr float kSqrt2OverPi = 0.7978845608028654f;
constexpr float kGeluC = 0.044715f;

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef float float16_t __attribute__((ext_vector_type(16)));

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float float2_t __attribute__((ext_vector_type(2)));

// Two values rounded to bfloat16 (nearest, ties to even) by one
// v_cvt_pk_bf16_f32: a in the low half, b in the high half.
__device__ __forceinline__ unsigned bf16x2_bits(float a, float b) {
  return __builtin_bit_cast(unsigned, __builtin_convertvector((float2_t){a, b}, bf16x2_t));
}
__device__ __forceinline__ uint16_t bf16_bits(float x) { return uint16_t(bf16x2_bits(x, 0.0f)); }
__device__ __forceinline__ float bf16_value(uint16_t h) { return __uint_as_float(unsigned(h) << 16); }

// GELU with the tanh approximation, written with the identity
// (1 + tanh u) / 2 = 1 / (1 + exp(-2u)): gelu(z) = z sigma(2u),
// u = sqrt(2/pi) (z + 0.044715 z^3); its derivative is
// sigma + 2 z sigma (1 - sigma) du/dz.  exp(-2u) is evaluated as
// 2^(t kGeluExp2), t = z + 0.044715 z^3, with the three constant factors
// folded into one (one product and the hardware 2^x).
constexpr float kGeluExp2 = -2.302208198144325f;  // -2 sqrt(2/pi) log2(e)
__device__ __forceinline__ float gelu_sigma(float z) {
  const float t = z + kGeluC * z * z * z;
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(t * kGeluExp2));
}
__device__ __forceinline__ float gelu_f(float z) { return z * gelu_sigma(z); }
__device__ __forceinline__ float gelu_grad_f(float z) {
  const float sg = gelu_sigma(z);
  const float du = kSqrt2OverPi * (1.0f + 3.0f * kGeluC * z * z);
  return sg + 2.0f * z * sg * (1.0f - sg) * du;
}

// Band q of gamma(x) = (x, sin(2^k pi x), cos(2^k pi x), k = 0..7) of the 6
// inputs at `in`, rounded to bfloat16 into the feature row `row`: the six
// sines (features 6 + 12 q + i) and cosines (6 + 12 q + 6 + i), band 0 also
// the inputs themselves (features 0..5); band q writes the zero padding of
// features 102 + 4 q .. 102 + 4 q + 3 below 128.  The six inputs are loaded
// together.  2^q pi x is r = 2^(q-1) x revolutions (an exact power-of-two
// product); r - rint(r) is exact and within half a revolution, and the
// hardware sine and cosine of revolutions take it from there (absolute
// error far below the bfloat16 rounding of the features).
constexpr int kEncBands = 8;
static_assert(6 + 12 * kEncBands + 4 * (kEncBands - 1) >= RRT_MLP_IN, "padding per band");

__device__ __forceinline__ void encode_band(const float* __restrict__ in, int q,
                                            uint16_t* __restrict__ row) {
  float x[6];
#pragma unroll
  for (int i = 0; i < 6; ++i) x[i] = in[i];
  const float rev = 0.5f * float(1 << q);
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    const float r = x[i] * rev;
    const float f = r - __builtin_rintf(r);
    row[6 + 12 * q + i] = bf16_bits(__builtin_amdgcn_sinf(f));
    row[6 + 12 * q + 6 + i] = bf16_bits(__builtin_amdgcn_cosf(f));
  }
  if (q == 0) {
#pragma unroll
    for (int i = 0; i < 6; ++i) row[i] = bf16_bits(x[i]);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int f = 6 + 12 * kEncBands + 4 * q + e;
    if (f < RRT_MLP_IN) row[f] = 0;
  }
}

// One thread per (row, band).
__global__ void encode_kernel(const float* __restrict__ in, uint16_t* __restrict__ out,
                              int64_t B) {
  const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= B * kEncBands) return;
  const int64_t r = t / kEncBands;
  encode_band(in + r * 6, int(t - r * kEncBands), out + r * RRT_MLP_IN);
}

// Decoder weight layout (rrt_mlp_pack): layer l keeps its offset and size
// of the row-major packing (256 rows of K = 128 or 256 inputs); inside it
// the MFMA operand of feature tile t (rows 32 t .. 32 t + 31) at k-step s
// (k = 16 s .. 16 s + 15) is 512 values at (t * K / 16 + s) * 512, lane
// m + 32 h of the 64 holding W[32 t + m][16 s + 8 h + e], e = 0..7, at
// 8 (m + 32 h) + e.  One thread per 8-value piece (16-byte copies).
__global__ void pack_kernel(const uint16_t* __restrict__ w, uint16_t* __restrict__ out) {
  int64_t p = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (p >= RRT_MLP_WEIGHT_COUNT / 8) return;
  int64_t base = 0;
  int K = RRT_MLP_IN;
  for (int l = 0; l < RRT_MLP_WEIGHTS; ++l) {
    K = l == 0 ? RRT_MLP_IN : RRT_MLP_HIDDEN;
    const int64_t pieces = int64_t(RRT_MLP_HIDDEN) * K / 8;
    if (p < pieces) break;
    p -= pieces;
    base += int64_t(RRT_MLP_HIDDEN) * K;
  }
  const int S = K / 16;
  const int lane = int(p % 64), s = int((p / 64) % S), t = int(p / 64 / S);
  const int m = lane & 31, h = lane >> 5;
  const uint4 v = *reinterpret_cast<const uint4*>(w + base + int64_t(32 * t + m) * K + 16 * s + 8 * h);
  *reinterpret_cast<uint4*>(out + base + p * 8) = v;
}

// The whole decoder for a tile of kDecRows = 64 vertices in one 512-thread
// workgroup (8 waves): encoding, the four hidden layers and the output
// layer, with the tile's activations kept in LDS (one bfloat16 buffer of
// k-contiguous rows, 33.8 KB, rewritten in place between two barriers after
// each layer's products, so that three workgroups share a CU) and the
// weights read from global memory in the decoder layout (592 KB shared by
// every tile: an L2-resident stream).
// Wave w computes output features [32 w, 32 w + 32) of every layer for the
// tile's 64 vertices as the transposed product W A^T: 1 x 2 tiles of
// 32 x 32 MFMAs with the weights as the first operand, so that each lane
// ends with four consecutive features of one vertex per register group and
// stores them with one 8-byte LDS write.  The output layer goes through
// LDS as float rows, 32 vertices at a time, so that each wave writes whole
// 1 KiB rows of the result.  The k steps, the products and their order are those of forward_kernel
// (a product of two operands is the same either way round), and so are
// the epilogues (bias + GELU rounded to bfloat16; bias, then the per-slot
// scale of the vertex's cluster for the output): the values are
// bit-identical to encode + forward_kernel + the per-slot scaling
// in binary32.
constexpr int kDecRows = 64;
constexpr int kDecTiles = kDecRows / 32;  // 32-vertex MFMA tiles per workgroup
constexpr int kDecWaves = 8;                // waves per workgroup
constexpr int kDecFeat = RRT_MLP_HIDDEN / 32 / kDecWaves;  // 32-feature tiles per wave
constexpr int kActStride = RRT_MLP_HIDDEN + 8;  // bf16 per LDS row (staggered banks)
constexpr int kOutStride = RRT_MLP_OUT + 4;      // float per LDS output row (staggered banks)
static_assert(32 * kOutStride * 4 <= kDecRows * kActStride * 2,
              "a 32-vertex output tile fits the activation buffer");
static_assert(RRT_MLP_OUT == 4 * 64, "one float4 per lane and output row");

// One layer's products for the tile: acc[i][j] = W rows [n0 + 32 i, +32) x
// the tile's activations of vertices [32 j, +32), over k = 0..K-1 in steps of
// 16.  The weights come from L2 in the decoder layout (one 16-byte load per
// lane, feature tile and step: 1 KiB contiguous per wave, eight whole cache
// lines); they are loaded kDecAhead steps ahead into a register ring, so
// that that many loads are in flight while the products run instead of
// each step waiting for its own.  K is a compile-time constant so that the
// loop and the ring unroll.
constexpr int kDecAhead = 2;

template <int K>
__device__ __forceinline__ void decode_products(const uint16_t* __restrict__ act,
                                                const uint16_t* __restrict__ Wl, int n0, int lane,
                                                float16_t (&acc)[kDecFeat][kDecTiles]) {
  constexpr int kSteps = K / 16;
  constexpr int kAhead = kDecAhead < kSteps ? kDecAhead : kSteps;
  const int ml = lane & 31;
#pragma unroll
  for (int i = 0; i < kDecFeat; ++i)
#pragma unroll
    for (int j = 0; j < kDecTiles; ++j) acc[i][j] = float16_t{};
  const uint16_t* a_base = act + ml * kActStride + 8 * (lane >> 5);
  // fragment (tile n0 / 32 + i, step s) of this lane: 8 values at
  // ((tile * kSteps + s) * 64 + lane) * 8 of the layer's decoder layout
  const uint16_t* w_base = Wl + (int64_t(n0 / 32) * kSteps * 64 + lane) * 8;
  bf16x8_t ring[kAhead][kDecFeat];
#pragma unroll
  for (int s = 0; s < kAhead; ++s)
#pragma unroll
    for (int i = 0; i < kDecFeat; ++i)
      ring[s][i] = *reinterpret_cast<const bf16x8_t*>(w_base + (int64_t(i) * kSteps + s) * 512);
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    // keep each step's loads in their step (the scheduler would otherwise
    // sink them next to their use to save registers)
    __builtin_amdgcn_sched_barrier(0);
    bf16x8_t w[kDecFeat], a[kDecTiles];
#pragma unroll
    for (int i = 0; i < kDecFeat; ++i) w[i] = ring[s % kAhead][i];
    if (s + kAhead < kSteps) {
#pragma unroll
      for (int i = 0; i < kDecFeat; ++i)
        ring[s % kAhead][i] = *reinterpret_cast<const bf16x8_t*>(
            w_base + (int64_t(i) * kSteps + s + kAhead) * 512);
    }
#pragma unroll
    for (int j = 0; j < kDecTiles; ++j)
      a[j] = *reinterpret_cast<const bf16x8_t*>(a_base + 32 * j * kActStride + 16 * s);
#pragma unroll
    for (int i = 0; i < kDecFeat; ++i)
#pragma unroll
      for (int j = 0; j < kDecTiles; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[i], a[j], acc[i][j], 0, 0, 0);
  }
}

__global__ __launch_bounds__(64 * kDecWaves, 6) void decode_kernel(const float* __restrict__ pos_nrm, int64_t B,
                                                     const uint16_t* __restrict__ W,
                                                     const float* __restrict__ bias,
                                                     const int32_t* __restrict__ cluster,
                                                     const float* __restrict__ scale, int C,
                                                     float* __restrict__ out) {
  __shared__ __align__(16) uint16_t act[kDecRows * kActStride];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t r0 = int64_t(blockIdx.x) * kDecRows;
  static_assert(kDecRows * kEncBands == 64 * kDecWaves, "one thread per (row, band)");
  {
    const int row = threadIdx.x / kEncBands, q = threadIdx.x % kEncBands;
    uint16_t* dst = act + row * kActStride;
    if (r0 + row < B) {
      encode_band(pos_nrm + (r0 + row) * 6, q, dst);
    } else {
      for (int f = q; f < RRT_MLP_IN; f += kEncBands) dst[f] = 0;
    }
  }
  __syncthreads();
  const int n0 = 32 * kDecFeat * wave;
  // register r of tile (i, j): feature n0 + 32 i + 8 (r / 4) + 4 (lane / 32) + r % 4,
  // vertex 32 j + lane % 32
  const int fl = 4 * (lane >> 5), ml = lane & 31;
  const uint16_t* Wl = W;
  const float* bl = bias;
#pragma unroll 1
  for (int l = 0; l < RRT_MLP_WEIGHTS; ++l) {
    const int K = l == 0 ? RRT_MLP_IN : RRT_MLP_HIDDEN;
    float16_t acc[kDecFeat][kDecTiles];
    if (l == 0)
      decode_products<RRT_MLP_IN>(act, Wl, n0, lane, acc);
    else
      decode_products<RRT_MLP_HIDDEN>(act, Wl, n0, lane, acc);
    __syncthreads();  // every wave has read its operands: the buffer is free
    if (l < RRT_MLP_WEIGHTS - 1) {
#pragma unroll
      for (int i = 0; i < kDecFeat; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int n = n0 + 32 * i + 8 * g + fl;
          const float4 b4 = *reinterpret_cast<const float4*>(bl + n);
#pragma unroll
          for (int j = 0; j < kDecTiles; ++j) {
            const int m = 32 * j + ml;
            uint2 v;
            v.x = bf16x2_bits(gelu_f(acc[i][j][4 * g] + b4.x), gelu_f(acc[i][j][4 * g + 1] + b4.y));
            v.y = bf16x2_bits(gelu_f(acc[i][j][4 * g + 2] + b4.z),
                              gelu_f(acc[i][j][4 * g + 3] + b4.w));
            *reinterpret_cast<uint2*>(act + m * kActStride + n) = v;
          }
        }
      __syncthreads();
    } else {
      // output layer, one 32-vertex tile at a time: acc + bias into LDS
      // (float rows of kOutStride), then each wave writes whole 1 KiB rows,
      // scaled by the row's cluster (one cluster per row: a uniform load)
      float* outl = reinterpret_cast<float*>(act);
#pragma unroll
      for (int j = 0; j < kDecTiles; ++j) {
#pragma unroll
        for (int i = 0; i < kDecFeat; ++i)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int n = n0 + 32 * i + 8 * g + fl;
            const float4 b4 = *reinterpret_cast<const float4*>(bl + n);
            *reinterpret_cast<float4*>(outl + ml * kOutStride + n) =
                make_float4(acc[i][j][4 * g] + b4.x, acc[i][j][4 * g + 1] + b4.y,
                            acc[i][j][4 * g + 2] + b4.z, acc[i][j][4 * g + 3] + b4.w);
          }
        __syncthreads();
        const int64_t rj = r0 + 32 * j;
        for (int row = wave; row < 32 && rj + row < B; row += kDecWaves) {
          const int c = cluster[rj + row];
          const float4 v = *reinterpret_cast<const float4*>(outl + row * kOutStride + 4 * lane);
          float4 o = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
          if (c >= 0 && c < C) {
            const float4 s4 = *reinterpret_cast<const float4*>(scale + int64_t(c) * RRT_MLP_OUT + 4 * lane);
            o = make_float4(v.x * s4.x, v.y * s4.y, v.z * s4.z, v.w * s4.w);
          }
          *reinterpret_cast<float4*>(out + (rj + row) * RRT_MLP_OUT + 4 * lane) = o;
        }
        if (j + 1 < kDecTiles) __syncthreads();
      }
    }
    Wl += int64_t(K) * RRT_MLP_HIDDEN;
    bl += RRT_MLP_HIDDEN;
  }
}

// Weight and bias gradients of up to three layers: dW_l[m][n] = sum_b dz_l[b][m]
// a_l[b][n] and db_l[m] = sum_b dz_l[b][m], over the batch rows b, which both
// operands store row by row.  The batch is cut into at most 16 ranges of
// g.rows rows whose sums are added in order of the range, the bias in ranges of
// 64 rows, so the result does not depend on the launch.  A workgroup takes a
// 32 x 32 tile of one dW, each of its waves one range: a lane loads an 8 x 8
// block of one operand (eight 16-byte loads, the next 64 rows' under way while
// the matrix cores consume these), transposes it in registers (32 byte
// permutes) and stores it as eight rows of 8 consecutive k in the wave's own
// part of LDS, which is how the MFMA reads them; no wave waits for another
// until their tiles are added up.  Eight more workgroups per layer add up the
// columns of dz, a range of 64 rows and two columns per thread.
//
// Layer li is blockIdx.y.  A chip's eight L2s get the workgroups in turn
// (blockIdx.x % 8): each takes a part of 128 x 64 of dW, so that it reads half
// of dz and a quarter of the activations.
//
// What bounds it: the latency of a range's four slices, at 72 workgroups a
// layer, so the layers whose operands are ready share a launch.  4,096 rows: a
// GEMM that stored transposed slices two bytes at a time, with its partial sums
// in memory and the column sums in launches of their own, took 177 us for all
// five layers and the training step 287 us; 64 x 64 tiles with partial sums in
// memory 38 us and 114 us; this way the step takes 110 us, with the sums of the
// first to the bit (training carries a last place of a weight gradient into the
// weights' BF16 roundings).
constexpr int kGradRows = 64;               // rows of a wave's slice
constexpr int kGradStride = kGradRows + 8;  // bf16 per LDS row (16-byte rows, staggered banks)
constexpr int kGradLayers = 3;
constexpr int kGradTiles = 64;              // 32 x 32 tiles of a 256 x 256 dW
constexpr int kGradBias = RRT_MLP_HIDDEN / 32;
constexpr int kMaxSplits = 16;
constexpr int kBiasPass = 64;               // bias ranges added up at a time

struct GradLayer {
  const uint16_t* dz;  // [B][256]
  const uint16_t* a;   // [B][n]
  int n;
  float* dw;           // [256][n]
  float* db;           // [256]
};
struct GradArgs {
  GradLayer layer[kGradLayers];
  int64_t B;
  int64_t rows;        // rows of a range (a multiple of 32); one wave each
};

__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Columns 32 cb .. of one layer's bias gradient.
__device__ void bias_gradient(const GradLayer& L, int64_t B, int cb, float* red) {
  const int tid = threadIdx.x, pair = tid & 15, slots = int(blockDim.x) >> 4;
  const uint16_t* col = L.dz + 32 * cb + 2 * pair;
  const int64_t ranges = (B + 63) / 64;
  float total = 0.0f;
  for (int64_t c0 = 0; c0 < ranges; c0 += kBiasPass) {
    const int nc = int(ranges - c0 < kBiasPass ? ranges - c0 : kBiasPass);
    for (int c = tid >> 4; c < nc; c += slots) {
      const int64_t r0 = (c0 + c) * 64;
      const int64_t left = B - r0;
      float s0 = 0.0f, s1 = 0.0f;
      for (int r = 0; r < 64 && r < left; r += 16) {
        unsigned v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i)
          v[i] = r + i < left ? *reinterpret_cast<const unsigned*>(col + (r0 + r + i) * RRT_MLP_HIDDEN) : 0u;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          s0 += __uint_as_float(v[i] << 16);
          s1 += __uint_as_float(v[i] & 0xffff0000u);
        }
      }
      red[c * 32 + 2 * pair] = s0;
      red[c * 32 + 2 * pair + 1] = s1;
    }
    __syncthreads();
    if (tid < 32) {
      float s = 0.0f;
      for (int c = 0; c < nc; ++c) s += red[c * 32 + tid];
      total = c0 == 0 ? s : total + s;
    }
    __syncthreads();
  }
  if (tid < 32) L.db[32 * cb + tid] = total;
}

__global__ __launch_bounds__(64 * kMaxSplits) void grad_kernel(GradArgs g) {
  __shared__ __align__(16) uint16_t lds[kMaxSplits][2][32 * kGradStride];
  static_assert(sizeof(lds) >= kMaxSplits * 1024 * sizeof(float), "the waves' tiles");
  static_assert(sizeof(lds) >= kBiasPass * 32 * sizeof(float), "a pass of bias ranges");
  float* red = reinterpret_cast<float*>(&lds[0][0][0]);
  const GradLayer L = g.layer[blockIdx.y];
  const int t = blockIdx.x;
  if (t >= kGradTiles) {
    bias_gradient(L, g.B, t - kGradTiles, red);
    return;
  }
  const int part = t & 7, in = t >> 3;
  const int m0 = 128 * (part & 1) + 32 * (in & 3);
  const int n0 = 64 * (part >> 1) + 32 * (in >> 2);
  if (n0 >= L.n) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t b0 = int64_t(wave) * g.rows;
  const int64_t b1 = b0 + g.rows < g.B ? b0 + g.rows : g.B;
  // lanes 0..31 load dz, 32..63 the activations: block kb (8 rows) x mb (8
  // columns) of the 64 x 32 slice
  const bool acts = lane >= 32;
  const int kb = (lane & 31) >> 2, mb = lane & 3;
  const int width = acts ? L.n : RRT_MLP_HIDDEN;
  const uint16_t* from = (acts ? L.a + n0 : L.dz + m0) + 8 * mb;
  uint16_t* to = lds[wave][acts ? 1 : 0] + 8 * mb * kGradStride + 8 * kb;
  u32x4_t v[8];
  auto load = [&](int64_t b) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int64_t r = b + 8 * kb + i;
      v[i] = u32x4_t{0u, 0u, 0u, 0u};
      if (r < b1) v[i] = *reinterpret_cast<const u32x4_t*>(from + r * width);
    }
  };
  float16_t acc = {};
  const uint16_t* ar = lds[wave][0] + (lane & 31) * kGradStride + 8 * (lane >> 5);
  const uint16_t* br = lds[wave][1] + (lane & 31) * kGradStride + 8 * (lane >> 5);
  load(b0);
  for (int64_t b = b0; b < b1; b += kGradRows) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      u32x4_t w;
#pragma unroll
      for (int p = 0; p < 4; ++p)
        w[p] = __builtin_amdgcn_perm(v[2 * p + 1][j / 2], v[2 * p][j / 2],
                                     (j & 1) ? 0x07060302u : 0x05040100u);
      *reinterpret_cast<u32x4_t*>(to + j * kGradStride) = w;
    }
    wave_lds_order();
    if (b + kGradRows < b1) load(b + kGradRows);
#pragma unroll
    for (int s = 0; s < kGradRows / 16; ++s)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
          *reinterpret_cast<const bf16x8_t*>(ar + 16 * s),
          *reinterpret_cast<const bf16x8_t*>(br + 16 * s), acc, 0, 0, 0);
    wave_lds_order();
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r)
    red[wave * 1024 + (8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * 32 + (lane & 31)] = acc[r];
  __syncthreads();
  const int waves = int(blockDim.x) >> 6;
  for (int e = threadIdx.x; e < 1024; e += int(blockDim.x)) {
    float s = 0.0f;
    for (int z = 0; z < waves; ++z) s += red[z * 1024 + e];
    L.dw[int64_t(m0 + (e >> 5)) * L.n + n0 + (e & 31)] = s;
  }
}

// The layers of a training step for 32 rows of the batch in one 512-thread
// workgroup: wave w computes the features [32 w, 32 w + 32) of every layer as
// the transposed product W A^T, like the decoder, with the rows' values in LDS
// from layer to layer.  Its 32 rows of the weights (row by row in memory) come
// in whole cache lines through its own part of LDS; loaded as the matrix cores'
// operands, 32 rows of 32 bytes at a time, they went through the L1 four times
// (forward 27.8 us for 4,096 rows, this way 19.5).
//
// What bounds it: a layer's chain of weight load, LDS, products and barrier,
// 4 us, with 128 workgroups for 4,096 rows.  A GEMM launch per layer, its
// operands through memory, took 37.4 us forward and 63.8 back (55.1 now); for
// 65,536 rows 216 and 657 (154 and 600), for 64 rows 29.9 and 37.3 (16.5 and
// 30.7), so that way has no size left.  A training step at 4,096 rows 110 -> 86 us.
constexpr int kRowTile = 32;
// four floats of a caller's array, which need not start on 16 bytes
typedef float float4_u __attribute__((ext_vector_type(4), aligned(4)));

struct ForwardArgs {
  const uint16_t* x;  // [B][128]
  const uint16_t* W;  // row-major layers
  const float* bias;
  int64_t B;
  float* z[4];
  uint16_t* a[4];
  float* out;
};

// The tile's rows of 256 bfloat16 from LDS to rows r0.. of a [B][256] array.
__device__ __forceinline__ void store_rows(const uint16_t* act, int64_t r0, int64_t B,
                                           uint16_t* __restrict__ to) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int e = int(threadIdx.x) + 512 * i, row = e >> 5, c = (e & 31) * 8;
    if (r0 + row < B)
      *reinterpret_cast<u32x4_t*>(to + (r0 + row) * RRT_MLP_HIDDEN + c) =
          *reinterpret_cast<const u32x4_t*>(act + row * kActStride + c);
  }
}

__global__ __launch_bounds__(512) void forward_kernel(ForwardArgs g) {
  __shared__ __align__(16) uint16_t wt[8][32 * kActStride];
  __shared__ __align__(16) uint16_t act[kRowTile * kActStride];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n0 = 32 * wave, fl = 4 * (lane >> 5), ml = lane & 31;
  const int64_t r0 = int64_t(blockIdx.x) * kRowTile, m = r0 + ml;
  const uint16_t* Wl = g.W;
  const float* bl = g.bias;
  uint16_t* own = wt[wave];
  // the wave's 32 rows of a layer, 1 KiB per load (4 rows of 128 or 2 of 256)
  u32x4_t v[16];
  constexpr int kIn8 = RRT_MLP_IN / 8, kHid8 = RRT_MLP_HIDDEN / 8;
#pragma unroll
  for (int i = 0; i < kIn8 / 2; ++i)
    v[i] = *reinterpret_cast<const u32x4_t*>(Wl + n0 * RRT_MLP_IN + (64 * i + lane) * 8);
  {
    const int row = threadIdx.x >> 4, c = (threadIdx.x & 15) * 8;
    u32x4_t t = {0u, 0u, 0u, 0u};
    if (r0 + row < g.B) t = *reinterpret_cast<const u32x4_t*>(g.x + (r0 + row) * RRT_MLP_IN + c);
    *reinterpret_cast<u32x4_t*>(act + row * kActStride + c) = t;
  }
  __syncthreads();
  const uint16_t* wr = own + ml * kActStride + 8 * (lane >> 5);
  const uint16_t* ar = act + ml * kActStride + 8 * (lane >> 5);
#pragma unroll
  for (int l = 0; l < RRT_MLP_WEIGHTS; ++l) {
    const int K = l == 0 ? RRT_MLP_IN : RRT_MLP_HIDDEN, k8 = K / 8;
#pragma unroll
    for (int i = 0; i < k8 / 2; ++i) {
      const int e = 64 * i + lane;
      *reinterpret_cast<u32x4_t*>(own + e / k8 * kActStride + e % k8 * 8) = v[i];
    }
    wave_lds_order();
    // the next layer's weights are under way during this one's products
    Wl += int64_t(K) * RRT_MLP_HIDDEN;
    if (l + 1 < RRT_MLP_WEIGHTS) {
#pragma unroll
      for (int i = 0; i < kHid8 / 2; ++i)
        v[i] = *reinterpret_cast<const u32x4_t*>(Wl + n0 * RRT_MLP_HIDDEN + (64 * i + lane) * 8);
    }
    float16_t acc = {};
#pragma unroll
    for (int s = 0; s < K / 16; ++s)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
          *reinterpret_cast<const bf16x8_t*>(wr + 16 * s),
          *reinterpret_cast<const bf16x8_t*>(ar + 16 * s), acc, 0, 0, 0);
    __syncthreads();  // every wave has read its operands: the buffer is free
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int n = n0 + 8 * q + fl;
      const float4_u x = {acc[4 * q] + bl[n], acc[4 * q + 1] + bl[n + 1],
                          acc[4 * q + 2] + bl[n + 2], acc[4 * q + 3] + bl[n + 3]};
      float* to = l + 1 < RRT_MLP_WEIGHTS ? g.z[l < 4 ? l : 0] : g.out;
      if (m < g.B) *reinterpret_cast<float4_u*>(to + m * RRT_MLP_HIDDEN + n) = x;
      if (l + 1 < RRT_MLP_WEIGHTS) {
        uint2 o;
        o.x = bf16x2_bits(gelu_f(x[0]), gelu_f(x[1]));
        o.y = bf16x2_bits(gelu_f(x[2]), gelu_f(x[3]));
        *reinterpret_cast<uint2*>(act + ml * kActStride + n) = o;
      }
    }
    bl += RRT_MLP_HIDDEN;
    if (l + 1 < RRT_MLP_WEIGHTS) {
      __syncthreads();
      store_rows(act, r0, g.B, g.a[l < 4 ? l : 0]);
    }
  }
}

// Two layers back: dz_{l-1} = (dz_l W_l) * gelu'(z_{l-1}), from dout (also
// stored as bfloat16) or from a dz.  The weights are needed with 8 consecutive
// rows per lane: a wave loads its 32 columns in 8 x 8 blocks, two per lane,
// transposes them in registers and puts them into its own part of LDS.
struct BackArgs {
  const float* dout;      // [B][256], or null: dz_in
  const uint16_t* dz_in;
  uint16_t* dz_top;       // bfloat16 dout
  const uint16_t* W[2];
  const float* z[2];
  uint16_t* dz[2];
  int64_t B;
};

__global__ __launch_bounds__(512) void back_kernel(BackArgs g) {
  __shared__ __align__(16) uint16_t wt[8][32 * kActStride];
  __shared__ __align__(16) uint16_t act[kRowTile * kActStride];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n0 = 32 * wave, fl = 4 * (lane >> 5), ml = lane & 31;
  const int64_t r0 = int64_t(blockIdx.x) * kRowTile, m = r0 + ml;
  const int kb = lane >> 2, nb = lane & 3;
  u32x4_t v[2][8];
  auto load = [&](const uint16_t* W) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 8; ++i)
        v[h][i] = *reinterpret_cast<const u32x4_t*>(
            W + (8 * (kb + 16 * h) + i) * RRT_MLP_HIDDEN + n0 + 8 * nb);
  };
  load(g.W[0]);
  {
    const int row = threadIdx.x >> 4, c = (threadIdx.x & 15) * 8;
    const int64_t at = (r0 + row) * RRT_MLP_HIDDEN + c;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      u32x4_t t = {0u, 0u, 0u, 0u};
      if (r0 + row < g.B) {
        if (g.dout) {
          const float4_u a = *reinterpret_cast<const float4_u*>(g.dout + at + 128 * i);
          const float4_u b = *reinterpret_cast<const float4_u*>(g.dout + at + 128 * i + 4);
          t = u32x4_t{bf16x2_bits(a[0], a[1]), bf16x2_bits(a[2], a[3]), bf16x2_bits(b[0], b[1]),
                      bf16x2_bits(b[2], b[3])};
          *reinterpret_cast<u32x4_t*>(g.dz_top + at + 128 * i) = t;
        } else {
          t = *reinterpret_cast<const u32x4_t*>(g.dz_in + at + 128 * i);
        }
      }
      *reinterpret_cast<u32x4_t*>(act + row * kActStride + c + 128 * i) = t;
    }
  }
  __syncthreads();
  const int64_t mz = m < g.B ? m : g.B - 1;
  uint16_t* own = wt[wave];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    float4 z[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      z[q] = *reinterpret_cast<const float4*>(g.z[t] + mz * RRT_MLP_HIDDEN + n0 + 8 * q + fl);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        u32x4_t x;
#pragma unroll
        for (int p = 0; p < 4; ++p)
          x[p] = __builtin_amdgcn_perm(v[h][2 * p + 1][j / 2], v[h][2 * p][j / 2],
                                       (j & 1) ? 0x07060302u : 0x05040100u);
        *reinterpret_cast<u32x4_t*>(own + (8 * nb + j) * kActStride + 8 * (kb + 16 * h)) = x;
      }
    wave_lds_order();
    if (t == 0) load(g.W[1]);
    const uint16_t* wr = own + ml * kActStride + 8 * (lane >> 5);
    const uint16_t* ar = act + ml * kActStride + 8 * (lane >> 5);
    float16_t acc = {};
#pragma unroll
    for (int s = 0; s < RRT_MLP_HIDDEN / 16; ++s)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
          *reinterpret_cast<const bf16x8_t*>(wr + 16 * s),
          *reinterpret_cast<const bf16x8_t*>(ar + 16 * s), acc, 0, 0, 0);
    __syncthreads();  // every wave has read its operands: the buffers are free
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint2 o;
      o.x = bf16x2_bits(acc[4 * q] * gelu_grad_f(z[q].x), acc[4 * q + 1] * gelu_grad_f(z[q].y));
      o.y = bf16x2_bits(acc[4 * q + 2] * gelu_grad_f(z[q].z), acc[4 * q + 3] * gelu_grad_f(z[q].w));
      *reinterpret_cast<uint2*>(act + ml * kActStride + n0 + 8 * q + fl) = o;
    }
    __syncthreads();
    store_rows(act, r0, g.B, g.dz[t]);
  }
}

// dout = 2 (out - target) / count; loss += sum (out - target)^2 / count (FP64).
// A grid-stride loop over at most 256 workgroups: one FP64 atomic each.
__global__ void mse_kernel(const float* __restrict__ out, const float* __restrict__ tgt,
                           int64_t count, float* __restrict__ dout, double* __restrict__ loss) {
  __shared__ double part[256];
  double sq = 0.0;
  const int64_t first = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t step = int64_t(gridDim.x) * blockDim.x;
  int64_t done = 0;
  // four values at a time where the three arrays allow 16-byte accesses (a
  // thread's rounds follow one another: 16 of them took 10.9 us for 1,048,576
  // values, these 4 7.5)
  if (((reinterpret_cast<uintptr_t>(out) | reinterpret_cast<uintptr_t>(tgt) |
        reinterpret_cast<uintptr_t>(dout)) & 15u) == 0) {
    const int64_t n4 = count >> 2;
    for (int64_t t = first; t < n4; t += step) {
      const float4 o = reinterpret_cast<const float4*>(out)[t];
      const float4 g = reinterpret_cast<const float4*>(tgt)[t];
      const float d0 = o.x - g.x, d1 = o.y - g.y, d2 = o.z - g.z, d3 = o.w - g.w;
      const float c = float(count);
      reinterpret_cast<float4*>(dout)[t] =
          make_float4(2.0f * d0 / c, 2.0f * d1 / c, 2.0f * d2 / c, 2.0f * d3 / c);
      sq += (double(d0) * double(d0) + double(d1) * double(d1)) +
            (double(d2) * double(d2) + double(d3) * double(d3));
    }
    done = 4 * n4;
  }
  for (int64_t t = done + first; t < count; t += step) {
    const float d = out[t] - tgt[t];
    dout[t] = 2.0f * d / float(count);
    sq += double(d) * double(d);
  }
  part[threadIdx.x] = sq;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) part[threadIdx.x] += part[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) atomicAdd(loss, part[0] / double(count));
}

__global__ void adam_kernel(float* __restrict__ p, uint16_t* __restrict__ p_bf16,
                            float* __restrict__ m, float* __restrict__ v,
                            const float* __restrict__ g, int64_t n, float lr, float b1, float b2,
                            float eps, float c1, float c2) {
  const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const float gt = g[t];
  const float mt = b1 * m[t] + (1.0f - b1) * gt;
  const float vt = b2 * v[t] + (1.0f - b2) * gt * gt;
  m[t] = mt;
  v[t] = vt;
  const float pt = p[t] - lr * (mt / c1) / (sqrtf(vt / c2) + eps);
  p[t] = pt;
  if (p_bf16) p_bf16[t] = bf16_bits(pt);
}

inline unsigned blocks(int64_t n, int per = 256) { return unsigned((n + per - 1) / per); }

// Row ranges of the weight gradients' sums over a batch of B rows: one per 256
// rows, at most kMaxSplits.
inline int dw_splits(int64_t B) {
  const int64_t s = (B + 255) / 256;
  return int(s < 1 ? 1 : (s > kMaxSplits ? kMaxSplits : s));
}

// Gradients of `layers` layers over the batch.
int launch_grads(GradArgs g, int layers, hipStream_t s) {
  const int64_t splits = dw_splits(g.B);
  g.rows = ((g.B + splits - 1) / splits + 31) / 32 * 32;
  const int waves = int((g.B + g.rows - 1) / g.rows);
  hipLaunchKernelGGL(grad_kernel, dim3(kGradTiles + kGradBias, unsigned(layers)), dim3(64 * waves), 0,
                     s, g);
  return check_launch("grad");
}

}  // namespace

// Layer geometry: W_l is [out_l][in_l] (row-major), packed in order.
static const int kIn[RRT_MLP_WEIGHTS] = {RRT_MLP_IN, RRT_MLP_HIDDEN, RRT_MLP_HIDDEN,
                                         RRT_MLP_HIDDEN, RRT_MLP_HIDDEN};
static const int kOut[RRT_MLP_WEIGHTS] = {RRT_MLP_HIDDEN, RRT_MLP_HIDDEN, RRT_MLP_HIDDEN,
                                          RRT_MLP_HIDDEN, RRT_MLP_OUT};

int64_t mlp_weight_offset(int l) {
  int64_t o = 0;
  for (int i = 0; i < l; ++i) o += int64_t(kIn[i]) * kOut[i];
  return o;
}
int64_t mlp_bias_offset(int l) {
  int64_t o = 0;
  for (int i = 0; i < l; ++i) o += kOut[i];
  return o;
}

// Activation workspace for a batch of B rows:
//   z_l  FP32 [B][256] for the 4 hidden layers,
//   a_l  BF16 [B][256] for the 4 hidden layers,
//   dz   BF16 [B][256] x 2 (ping-pong, backward only),
//   dout BF16 [B][256] (backward only),
//   256 KiB per row range (FP32 [S][256][256]), which callers provide and the
//   gradients no longer need.
size_t mlp_workspace_bytes(int64_t B) {
  const size_t rows = size_t(B) * RRT_MLP_HIDDEN;
  return align256(rows * 4) * 4 + align256(rows * 2) * 4 + align256(rows * 2) * 2 +
         align256(size_t(B) * RRT_MLP_OUT * 2) +
         align256(size_t(dw_splits(B)) * RRT_MLP_HIDDEN * RRT_MLP_HIDDEN * 4);
}

struct MlpWs {
  float* z[4];
  uint16_t* a[4];
  uint16_t* dz[2];
  uint16_t* dout_bf16;
};

static MlpWs carve(void* ws, int64_t B) {
  const size_t rows = size_t(B) * RRT_MLP_HIDDEN;
  char* p = static_cast<char*>(ws);
  MlpWs w;
  for (int l = 0; l < 4; ++l) {
    w.z[l] = reinterpret_cast<float*>(p);
    p += align256(rows * 4);
  }
  for (int l = 0; l < 4; ++l) {
    w.a[l] = reinterpret_cast<uint16_t*>(p);
    p += align256(rows * 2);
  }
  for (int l = 0; l < 2; ++l) {
    w.dz[l] = reinterpret_cast<uint16_t*>(p);
    p += align256(rows * 2);
  }
  w.dout_bf16 = reinterpret_cast<uint16_t*>(p);
  return w;
}

int launch_mlp_decode(const void* w, const float* b, const float* scale, int C,
                      const float* pos_nrm, const int32_t* cluster, int64_t B, float* out,
                      hipStream_t s) {
  if (B == 0) return RRT_OK;
  hipLaunchKernelGGL(decode_kernel, dim3(unsigned((B + kDecRows - 1) / kDecRows)),
                     dim3(64 * kDecWaves), 0, s,
                     pos_nrm, B, static_cast<const uint16_t*>(w), b, cluster, scale, C, out);
  return check_launch("decode");
}

int launch_mlp_pack(const void* w, void* out, hipStream_t s) {
  hipLaunchKernelGGL(pack_kernel, dim3(blocks(RRT_MLP_WEIGHT_COUNT / 8)), dim3(256), 0, s,
                     static_cast<const uint16_t*>(w), static_cast<uint16_t*>(out));
  return check_launch("mlp_pack");
}

int launch_mlp_encode(const float* in, int64_t B, void* out, hipStream_t s) {
  hipLaunchKernelGGL(encode_kernel, dim3(blocks(B * kEncBands)), dim3(256), 0, s, in,
                     static_cast<uint16_t*>(out), B);
  return check_launch("encode");
}

int launch_mlp_forward(const void* w, const float* b, const void* x, int64_t B, float* out,
                       void* ws, hipStream_t s) {
  MlpWs k = carve(ws, B);
  ForwardArgs f = {};
  f.x = static_cast<const uint16_t*>(x);
  f.W = static_cast<const uint16_t*>(w);
  f.bias = b;
  f.B = B;
  for (int l = 0; l < 4; ++l) {
    f.z[l] = k.z[l];
    f.a[l] = k.a[l];
  }
  f.out = out;
  // the launch reads x while it writes out: an x inside out is copied first, to
  // the space of a gradient
  const size_t xbytes = size_t(B) * RRT_MLP_IN * 2, obytes = size_t(B) * RRT_MLP_OUT * 4;
  const uintptr_t xa = reinterpret_cast<uintptr_t>(x), oa = reinterpret_cast<uintptr_t>(out);
  if (xa < oa + obytes && oa < xa + xbytes) {
    const hipError_t e = hipMemcpyAsync(k.dz[0], x, xbytes, hipMemcpyDeviceToDevice, s);
    if (e != hipSuccess) return fail(RRT_ERR_DEVICE, "forward: %s", hipGetErrorString(e));
    f.x = k.dz[0];
  }
  hipLaunchKernelGGL(forward_kernel, dim3(unsigned((B + kRowTile - 1) / kRowTile)), dim3(512), 0, s, f);
  return check_launch("forward");
}

int launch_mlp_backward(const void* w, const void* x, int64_t B, const float* dout, float* dw,
                        float* db, void* ws, hipStream_t s) {
  const uint16_t* W = static_cast<const uint16_t*>(w);
  MlpWs k = carve(ws, B);
  // dz_{l-1} = (dz_l W_l) * gelu'(z_{l-1}): the buffers of dz hold three layers'
  // at a time, so the gradients are taken in two launches
  const uint16_t* dz[RRT_MLP_WEIGHTS];
  dz[4] = k.dout_bf16;
  // layers l and l - 1
  auto two_back = [&](int l, uint16_t* next, uint16_t* last) {
    BackArgs a = {};
    if (l == RRT_MLP_WEIGHTS - 1) {
      a.dout = dout;
      a.dz_top = k.dout_bf16;
    } else {
      a.dz_in = dz[l];
    }
    for (int i = 0; i < 2; ++i) {
      a.W[i] = W + mlp_weight_offset(l - i);
      a.z[i] = k.z[l - 1 - i];
    }
    dz[l - 1] = a.dz[0] = next;
    dz[l - 2] = a.dz[1] = last;
    a.B = B;
    hipLaunchKernelGGL(back_kernel, dim3(unsigned((B + kRowTile - 1) / kRowTile)), dim3(512), 0, s, a);
    return check_launch("back");
  };
  auto grads = [&](int top, int layers) {
    GradArgs g = {};
    g.B = B;
    for (int i = 0; i < layers; ++i) {
      const int l = top - i;
      g.layer[i] = {dz[l], l == 0 ? static_cast<const uint16_t*>(x) : k.a[l - 1], kIn[l],
                    dw + mlp_weight_offset(l), db + mlp_bias_offset(l)};
    }
    return launch_grads(g, layers, s);
  };
  int st;
  if ((st = two_back(4, k.dz[0], k.dz[1]))) return st;
  if ((st = grads(4, 3))) return st;
  if ((st = two_back(2, k.dout_bf16, k.dz[0]))) return st;
  return grads(1, 2);
}

int launch_mse(const float* out, const float* tgt, int64_t count, float* dout, double* loss,
               hipStream_t s) {
  const int64_t nb = (count + 255) / 256;
  hipLaunchKernelGGL(mse_kernel, dim3(unsigned(nb < 256 ? nb : 256)), dim3(256), 0, s, out, tgt,
                     count, dout, loss);
  return check_launch("mse");
}

int launch_adam(float* p, void* p_bf16, float* m, float* v, const float* g, int64_t n, float lr,
                float b1, float b2, float eps, int step, hipStream_t s) {
  const float c1 = 1.0f - powf(b1, float(step));
  const float c2 = 1.0f - powf(b2, float(step));
  hipLaunchKernelGGL(adam_kernel, dim3(blocks(n)), dim3(256), 0, s, p,
                     static_cast<uint16_t*>(p_bf16), m, v, g, n, lr, b1, b2, eps, c1, c2);
  return check_launch("adam");
}

}  // namespace rrt
