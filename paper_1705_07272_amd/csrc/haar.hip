// Orthonormal non-standard 2-D Haar transform of cube faces (Sec. V.B: the
// H/V/D coefficients of every scale are finite differences of 2x2 block
// averages of the next finer scale; Mallat quadrant layout per face).
//
// Each face is cut into Q x Q tiles (Q = min(n, 64)), one 256-thread
// workgroup per tile: the tile is staged in LDS (16 KiB, small enough to run
// beside relight waves that hold most of a CU's LDS), the levels of block
// side 2..Q are computed in place there (S stays at the block's corner), and
// the H/V/D outputs of every level go straight to their Mallat positions,
// which for one tile form contiguous row segments.  For n > 64 the (n/64)^2
// tile sums are combined by a second, tiny launch; the tile sums travel between
// the launches through the top-left corner of the output (forward) or the
// first texel of each output tile (inverse), positions no other coefficient
// or texel of the first launch uses.

#include "geometry.h"
#include "rrt_internal.h"

namespace rrt {
namespace {

constexpr int kThreads = 256;
constexpr int kTile = 64;
constexpr int kMaxGrid = 1024 / kTile;  // tiles per face side at n = 1024

__device__ __forceinline__ void butterfly(float a, float b, float c, float d, float& S, float& H,
                                          float& V, float& D) {
  S = 0.5f * ((a + b) + (c + d));
  H = 0.5f * ((a - b) + (c - d));
  V = 0.5f * ((a + b) - (c + d));
  D = 0.5f * ((a - b) - (c - d));
}

__device__ __forceinline__ void inverse_butterfly(float S, float H, float V, float D, float& a,
                                                  float& b, float& c, float& d) {
  a = 0.5f * ((S + H) + (V + D));
  b = 0.5f * ((S - H) + (V - D));
  c = 0.5f * ((S + H) - (V + D));
  d = 0.5f * ((S - H) - (V - D));
}

// Tile of a rotated map: destination texel (row, col) of a face takes the
// source texel of its direction; in patches of 8 x 8 texels with the lanes in
// Morton order and the map in strips of eight columns (n >= 8) as the relight
// gathers them, a wave of the workgroup taking every fourth patch.
__device__ __forceinline__ void rotated_tile(const float* __restrict__ map,
                                             const float* __restrict__ rot, int face, int logn,
                                             int logq, int row0, int col0, float* lds) {
  const int n = 1 << logn, Q = 1 << logq;
  const IRot R = frame_vertex_rotation(rot, nullptr, scale_bits(logn));
  const FaceAxes ax = face_axes(R, face);
  const float3 centre = dir_add(ax.mN, float(n), make_float3(0.0f, 0.0f, 0.0f));
  const unsigned last = unsigned(6 << (2 * logn)) - 1u;
  if (n < 8) {
    for (int e = threadIdx.x; e < Q * Q; e += kThreads) {
      const float3 d = dir_mad(ax.mU, float(2 * (col0 + (e & (Q - 1))) + 1 - n), ax.mV,
                               float(2 * (row0 + (e >> logq)) + 1 - n), centre);
      lds[e] = map[min(unsigned(source_texel(d, logn)), last)];
    }
    return;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int gx = morton_x(lane), gy = morton_y(lane);
  const int across = logq - 3;  // log2 patches per tile side
  constexpr int kWaves = kThreads / 64, kAhead = 4;  // patches in flight per wave
  const int patches = 1 << (2 * across);
  for (int k0 = wave; k0 < patches; k0 += kAhead * kWaves) {
    float v[kAhead];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const int k = min(k0 + j * kWaves, patches - 1);
      const int r = 8 * (k >> across) + gy, c = 8 * (k & ((1 << across) - 1)) + gx;
      const float3 d = dir_mad(ax.mU, float(2 * (col0 + c) + 1 - n), ax.mV,
                               float(2 * (row0 + r) + 1 - n), centre);
      // the index stays in the map by construction; the bound keeps this plain
      // pointer read in it whatever the rotation holds
      v[j] = map[min(source_texel_strip(d.x, d.y, d.z, logn) - strip_bias(logn), last)];
    }
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const int k = k0 + j * kWaves;
      if (k < patches)
        lds[((8 * (k >> across) + gy) << logq) + 8 * (k & ((1 << across) - 1)) + gx] = v[j];
    }
  }
}

// grid: count * 6 * G * G workgroups (G = n / Q); LDS: Q * Q floats.
// ROTATE: the squares are the faces of the map `pix` (in strips for n >= 8)
// under the rotations `rot`, gathered here instead of read (the rotated maps
// went through memory in a launch of their own: 64 rotations at n = 128 took
// 25 us for it, of 48 in all, 27.7 now).
template <bool ROTATE>
__global__ __launch_bounds__(kThreads) void haar_fwd_tiles(const float* __restrict__ pix,
                                                           const float* __restrict__ rot,
                                                           float* __restrict__ coef, int n,
                                                           int logq, int G) {
  extern __shared__ float lds[];
  const int Q = 1 << logq;
  const int64_t blk = blockIdx.x;
  const int tile = int(blk % (G * G));
  const int64_t face = blk / (G * G);
  const int ty = tile / G, tx = tile % G;
  float* dst = coef + face * int64_t(n) * n;
  const int row0 = ty * Q, col0 = tx * Q;
  if constexpr (ROTATE) {
    rotated_tile(pix, rot + face / 6 * 9, int(face % 6), __builtin_ctz(unsigned(n)), logq, row0, col0, lds);
  } else {
    const float* src = pix + face * int64_t(n) * n;
    for (int e = threadIdx.x; e < Q * Q; e += kThreads) {
      const int r = e >> logq, c = e & (Q - 1);
      lds[e] = src[int64_t(row0 + r) * n + col0 + c];
    }
  }
  __syncthreads();
  for (int B = 2; B <= Q; B <<= 1) {
    const int nb = Q / B, h = B >> 1, q = n / B;
    for (int e = threadIdx.x; e < nb * nb; e += kThreads) {
      const int br = e / nb, bc = e - br * nb;
      const int r0 = br * B, c0 = bc * B;
      float S, H, V, D;
      butterfly(lds[r0 * Q + c0], lds[r0 * Q + c0 + h], lds[(r0 + h) * Q + c0],
                lds[(r0 + h) * Q + c0 + h], S, H, V, D);
      lds[r0 * Q + c0] = S;
      const int gbr = ty * nb + br, gbc = tx * nb + bc;
      dst[int64_t(gbr) * n + q + gbc] = H;
      dst[int64_t(q + gbr) * n + gbc] = V;
      dst[int64_t(q + gbr) * n + q + gbc] = D;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) dst[int64_t(ty) * n + tx] = lds[0];
}

// Coarse levels above the tiles: the G x G tile sums sit in the top-left
// corner of each face of `coef` (spatial order); they are replaced by their
// own Mallat transform.  grid: count * 6; LDS: G * G floats (G <= kMaxGrid).
__global__ __launch_bounds__(64) void haar_fwd_coarse(float* __restrict__ coef, int n, int G) {
  __shared__ float s[kMaxGrid * kMaxGrid];
  float* f = coef + int64_t(blockIdx.x) * n * n;
  for (int e = threadIdx.x; e < G * G; e += 64) s[e] = f[int64_t(e / G) * n + (e % G)];
  __syncthreads();
  for (int B = 2; B <= G; B <<= 1) {
    const int nb = G / B, h = B >> 1, q = G / B;
    for (int e = threadIdx.x; e < nb * nb; e += 64) {
      const int br = e / nb, bc = e - br * nb;
      const int r0 = br * B, c0 = bc * B;
      float S, H, V, D;
      butterfly(s[r0 * G + c0], s[r0 * G + c0 + h], s[(r0 + h) * G + c0],
                s[(r0 + h) * G + c0 + h], S, H, V, D);
      s[r0 * G + c0] = S;
      f[int64_t(br) * n + q + bc] = H;
      f[int64_t(q + br) * n + bc] = V;
      f[int64_t(q + br) * n + q + bc] = D;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) f[0] = s[0];
}

// Inverse of haar_fwd_coarse: reads the Mallat corner of `coef` and writes
// the tile sum of tile (ty, tx) to stage[face * n * n + ty * rs + tx * cs].
__global__ __launch_bounds__(64) void haar_inv_coarse(const float* coef, float* stage, int n,
                                                      int G, int64_t rs, int64_t cs) {
  __shared__ float s[kMaxGrid * kMaxGrid];
  const float* f = coef + int64_t(blockIdx.x) * n * n;
  float* st = stage + int64_t(blockIdx.x) * n * n;
  if (threadIdx.x == 0) s[0] = f[0];
  __syncthreads();
  for (int B = G; B >= 2; B >>= 1) {
    const int nb = G / B, h = B >> 1, q = G / B;
    for (int e = threadIdx.x; e < nb * nb; e += 64) {
      const int br = e / nb, bc = e - br * nb;
      const int r0 = br * B, c0 = bc * B;
      float a, b, c, d;
      inverse_butterfly(s[r0 * G + c0], f[int64_t(br) * n + q + bc], f[int64_t(q + br) * n + bc],
                        f[int64_t(q + br) * n + q + bc], a, b, c, d);
      s[r0 * G + c0] = a;
      s[r0 * G + c0 + h] = b;
      s[(r0 + h) * G + c0] = c;
      s[(r0 + h) * G + c0 + h] = d;
    }
    __syncthreads();
  }
  for (int e = threadIdx.x; e < G * G; e += 64) st[(e / G) * rs + (e % G) * cs] = s[e];
}

// grid: count * 6 * G * G; the tile sum comes from coef[face][0] when G == 1,
// else from stage[face * n * n + ty * rs + tx * cs].  With `strips` (n >= 8)
// the pixels are written in strips of eight columns, each row by row
// (strip_offset): row r, column c of a square at (c >> 3) 8n + 8 r + (c & 7).
__global__ __launch_bounds__(kThreads) void haar_inv_tiles(const float* coef, const float* stage,
                                                           float* pix, int n, int logq, int G,
                                                           int64_t rs, int64_t cs, bool strips) {
  extern __shared__ float lds[];
  const int Q = 1 << logq;
  const int64_t blk = blockIdx.x;
  const int tile = int(blk % (G * G));
  const int64_t face = blk / (G * G);
  const int ty = tile / G, tx = tile % G;
  const float* f = coef + face * int64_t(n) * n;
  float* dst = pix + face * int64_t(n) * n;
  if (threadIdx.x == 0)
    lds[0] = (G == 1) ? f[0] : stage[face * int64_t(n) * n + ty * rs + tx * cs];
  __syncthreads();
  for (int B = Q; B >= 2; B >>= 1) {
    const int nb = Q / B, h = B >> 1, q = n / B;
    for (int e = threadIdx.x; e < nb * nb; e += kThreads) {
      const int br = e / nb, bc = e - br * nb;
      const int r0 = br * B, c0 = bc * B;
      const int gbr = ty * nb + br, gbc = tx * nb + bc;
      float a, b, c, d;
      inverse_butterfly(lds[r0 * Q + c0], f[int64_t(gbr) * n + q + gbc],
                        f[int64_t(q + gbr) * n + gbc], f[int64_t(q + gbr) * n + q + gbc], a, b,
                        c, d);
      lds[r0 * Q + c0] = a;
      lds[r0 * Q + c0 + h] = b;
      lds[(r0 + h) * Q + c0] = c;
      lds[(r0 + h) * Q + c0 + h] = d;
    }
    __syncthreads();
  }
  const int row0 = ty * Q, col0 = tx * Q;
  if (strips) {
    // consecutive threads write consecutive elements of a strip
    for (int e = threadIdx.x; e < Q * Q; e += kThreads) {
      const int r = (e >> 3) & (Q - 1), c = ((e >> (logq + 3)) << 3) + (e & 7);
      dst[int64_t((col0 + c) >> 3) * 8 * n + 8 * (row0 + r) + (c & 7)] = lds[r * Q + c];
    }
  } else {
    for (int e = threadIdx.x; e < Q * Q; e += kThreads) {
      const int r = e >> logq, c = e & (Q - 1);
      dst[int64_t(row0 + r) * n + col0 + c] = lds[e];
    }
  }
}

// Source map of a sparse lighting in one launch: a workgroup per 32 x 32 tile
// (the whole square below) looks through all entries, keeps those of its own
// levels and of its square's levels above the tiles in LDS and inverts both,
// with the arithmetic of the kernels above (the same values bit for bit).
// Of a repeated index the last entry counts: the tiles of a square each keep
// the square's coarse coefficients and have to keep the same ones, so a cell
// holds (entry number + 1, value) as 64 bits and takes the largest.
//
// What bounds it: latency (one round of loads, about 5 + log2 of the tiles
// per side barriers); the staged way clears, scatters and inverts a dense map in
// three or four launches.  13 KiB of LDS and few registers, to run beside relight waves.
// The call that prepares a lighting of 1,024 entries at n = 128 takes 7.2 us
// (the host's time; 4.8 us in a graph) instead of 18.7, at n = 16 7.2 instead of
// 14.9.  (Plain stores without the entry number and no flags: 4.6 us in a graph,
// 11.3 for 16,384 entries at n = 64 against 11.6.)
constexpr int kMapTile = 32;
constexpr int kMapMost = 16384;                    // entries
constexpr int64_t kMapEntries = int64_t(1) << 22;  // tiles x entries of the one-launch way

// The flag of a tile, a byte from each of the workgroup's four waves (without a
// barrier, which takes 0.6 us here); most: the largest magnitude bits of the
// thread's texels.
__device__ __forceinline__ void flag_tile(unsigned* flag, unsigned most) {
  static_assert(kThreads == 256, "four waves");
  const bool all = __ballot(most >= 0x7f800000u) == 0;
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0)
    reinterpret_cast<uint8_t*>(flag)[wave] = all ? uint8_t(kMapFinite >> (8 * wave)) : uint8_t(0);
}

__global__ __launch_bounds__(kThreads) void source_map_kernel(const int32_t* __restrict__ idx,
                                                              const void* __restrict__ val, int f16,
                                                              int k, int logn, int total,
                                                              float* __restrict__ pix, bool strips,
                                                              unsigned* __restrict__ flags) {
  extern __shared__ __align__(8) float lds[];
  const int n = 1 << logn, Q = n < kMapTile ? n : kMapTile, logq = __builtin_ctz(Q);
  const int G = n >> logq;
  // cells (value, entry number + 1): the tile's own levels, then G x G of the
  // levels above, each in Mallat layout
  unsigned long long* cells = reinterpret_cast<unsigned long long*>(lds);
  const float* coef = lds;
  const float* top = lds + 2 * Q * Q;
  float* tile = lds + 2 * (Q * Q + G * G);  // Q x Q
  float* sums = tile + Q * Q;               // G x G: tile sums
  const int blk = blockIdx.x;
  const int face = blk / (G * G), t = blk % (G * G);
  const int ty = t / G, tx = t % G;
  for (int e = threadIdx.x; e < Q * Q + G * G; e += kThreads) cells[e] = 0;
  __syncthreads();
  auto place = [&](int v, int i) {
    if (v < 0 || v >= total || (v >> (2 * logn)) != face) return;
    const int r = (v >> logn) & (n - 1), c = v & (n - 1);
    int to;
    if (r < G && c < G) {
      to = Q * Q + r * G + c;
    } else {
      const int q = 1 << (31 - __builtin_clz(unsigned(r | c)));  // blocks per side of the level
      const int nb = q >> (logn - logq);                         // those of a tile
      const int br = r & (q - 1), bc = c & (q - 1);
      if (br / nb != ty || bc / nb != tx) return;
      to = ((r >= q ? nb : 0) + (br & (nb - 1))) * Q + (c >= q ? nb : 0) + (bc & (nb - 1));
    }
    const float x = f16 ? __half2float(static_cast<const __half*>(val)[i])
                        : static_cast<const float*>(val)[i];
    atomicMax(cells + to, static_cast<unsigned long long>(i + 1) << 32 | __float_as_uint(x));
  };
  for (int i = threadIdx.x; i < k; i += 4 * kThreads) {
    int v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = i + j * kThreads < k ? idx[i + j * kThreads] : -1;
#pragma unroll
    for (int j = 0; j < 4; ++j) place(v[j], i + j * kThreads);
  }
  __syncthreads();
  // one inverse level of block side B of an S x S grid, in place (m: cells)
  auto level = [&](float* g, const float* m, int S, int B) {
    const int nb = S / B, h = B >> 1;
    for (int e = threadIdx.x; e < nb * nb; e += kThreads) {
      const int br = e / nb, bc = e - br * nb;
      const int at = br * B * S + bc * B;
      float a, b, c, d;
      inverse_butterfly(g[at], m[2 * (br * S + nb + bc)], m[2 * ((nb + br) * S + bc)],
                        m[2 * ((nb + br) * S + nb + bc)], a, b, c, d);
      g[at] = a;
      g[at + h] = b;
      g[at + h * S] = c;
      g[at + h * S + h] = d;
    }
    __syncthreads();
  };
  if (threadIdx.x == 0) sums[0] = top[0];
  __syncthreads();
  for (int B = G; B >= 2; B >>= 1) level(sums, top, G, B);
  if (threadIdx.x == 0) tile[0] = sums[ty * G + tx];
  __syncthreads();
  for (int B = Q; B >= 2; B >>= 1) level(tile, coef, Q, B);
  float* dst = pix + (int64_t(face) << (2 * logn));
  const int row0 = ty * Q, col0 = tx * Q;
  unsigned most = 0;
  for (int e = threadIdx.x; e < Q * Q; e += kThreads) {
    const int r = strips ? (e >> 3) & (Q - 1) : e >> logq;
    const int c = strips ? ((e >> (logq + 3)) << 3) + (e & 7) : e & (Q - 1);
    const float x = tile[r * Q + c];
    most = max(most, __float_as_uint(x) & 0x7fffffffu);
    dst[strips ? int64_t((col0 + c) >> 3) * 8 * n + 8 * (row0 + r) + (c & 7)
               : int64_t(row0 + r) * n + col0 + c] = x;
  }
  flag_tile(flags + blk, most);
}

// The flags of a finished map (its layout does not matter: a tile is that many
// consecutive texels), in a launch after those that read dense: 2.7 us of the
// 13.6 that 24,576 entries at n = 64 take.  grid: tiles.
__global__ __launch_bounds__(kThreads) void map_flags_kernel(const float* __restrict__ pix, int texels,
                                                             unsigned* __restrict__ flags) {
  const float* t = pix + int64_t(blockIdx.x) * texels;
  unsigned most = 0;
  for (int e = threadIdx.x; e < texels; e += kThreads) most = max(most, __float_as_uint(t[e]) & 0x7fffffffu);
  flag_tile(flags + blockIdx.x, most);
}

}  // namespace

int launch_source_map(const int32_t* idx, const void* val, int dtype, int k, int n, int squares,
                      float* dense, float* pix, hipStream_t s, bool strips) {
  const int Q = n < kMapTile ? n : kMapTile;
  const int G = n / Q;
  const int64_t grid = int64_t(squares) * G * G;
  // Every tile reads every index, at 0.6 us per 1,024 of them: past 16,384 the
  // dense way is as fast (24,576 entries at n = 64: 15.2 against 16.4 us), and
  // the tiles' reads together are bounded, too.
  if (k <= kMapMost && grid * k <= kMapEntries) {
    if (n < 8) strips = false;
    const size_t lds = 3 * (size_t(Q) * Q + size_t(G) * G) * sizeof(float);
    hipLaunchKernelGGL(source_map_kernel, dim3(unsigned(grid)), dim3(kThreads), lds, s, idx, val,
                       dtype == RRT_F16 ? 1 : 0, k, ilog2(n), squares * n * n, pix, strips,
                       reinterpret_cast<unsigned*>(dense));
    return check_launch("source_map");
  }
  int st = launch_scatter_light(idx, val, dtype, k, n, squares, dense, s);
  if (st) return st;
  if ((st = launch_haar_inverse(dense, pix, n, squares, s, strips))) return st;
  hipLaunchKernelGGL(map_flags_kernel, dim3(unsigned(grid)), dim3(kThreads), 0, s, pix, Q * Q,
                     reinterpret_cast<unsigned*>(dense));
  return check_launch("map_flags");
}

static int launch_forward(const float* pix, const float* rot, float* coef, int n, int64_t squares,
                          hipStream_t s) {
  if (squares == 0) return RRT_OK;
  const int Q = n < kTile ? n : kTile;
  const int G = n / Q;
  const int64_t grid = squares * G * G;
  const size_t lds = size_t(Q) * Q * sizeof(float);
  if (rot) {
    hipLaunchKernelGGL(haar_fwd_tiles<true>, dim3(unsigned(grid)), dim3(kThreads), lds, s, pix, rot,
                       coef, n, ilog2(Q), G);
  } else {
    hipLaunchKernelGGL(haar_fwd_tiles<false>, dim3(unsigned(grid)), dim3(kThreads), lds, s, pix, rot,
                       coef, n, ilog2(Q), G);
  }
  int st = check_launch("haar_fwd_tiles");
  if (st || G == 1) return st;
  hipLaunchKernelGGL(haar_fwd_coarse, dim3(unsigned(squares)), dim3(64), 0, s, coef, n, G);
  return check_launch("haar_fwd_coarse");
}

int launch_haar_forward(const float* pix, float* coef, int n, int64_t squares, hipStream_t s) {
  return launch_forward(pix, nullptr, coef, n, squares, s);
}

int launch_haar_rotated(const float* map, const float* rot, int nrot, int n, float* coef,
                        hipStream_t s) {
  return launch_forward(map, rot, coef, n, int64_t(6) * nrot, s);
}

int launch_haar_inverse(const float* coef, float* pix, int n, int64_t squares, hipStream_t s,
                        bool strips) {
  if (squares == 0) return RRT_OK;
  if (n < 8) strips = false;
  const int Q = n < kTile ? n : kTile;
  const int G = n / Q;
  // first texel of each output tile (row and column multiples of Q)
  const int64_t rs = strips ? 8 * Q : int64_t(Q) * n, cs = strips ? int64_t(Q) * n : Q;
  if (G > 1) {
    hipLaunchKernelGGL(haar_inv_coarse, dim3(unsigned(squares)), dim3(64), 0, s, coef, pix, n,
                       G, rs, cs);
    int st = check_launch("haar_inv_coarse");
    if (st) return st;
  }
  const int64_t grid = squares * G * G;
  hipLaunchKernelGGL(haar_inv_tiles, dim3(unsigned(grid)), dim3(kThreads),
                     size_t(Q) * Q * sizeof(float), s, coef, (const float*)pix, pix, n, ilog2(Q),
                     G, rs, cs, strips);
  return check_launch("haar_inv_tiles");
}

}  // namespace rrt
