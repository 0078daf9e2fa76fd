// Non-linear approximation (Sec. III, Haar-domain methods): keep the k
// entries of largest magnitude of each row, ties to the lower position,
// output in ascending position order.
//
// One workgroup per row.  The k-th largest key (|x| orders like its bit
// pattern) is found from one histogram of the top 11 magnitude bits: the keys
// of the bin that holds it are candidates, ranked against each other in LDS.
// A bit per position collects what is kept; the output follows from a prefix
// sum over the bits in position order.  Three other ways remain: rows longer
// than the bits' LDS (a radix select and an ordered compaction), a few long
// rows (several workgroups per row) and k = len (a copy).
#include "rrt_internal.h"

namespace rrt {
namespace {

constexpr int kItems = 4;

// Exclusive prefix sum over the workgroup; *total gets the sum.
template <int kWaves>
__device__ __forceinline__ int block_scan(int x, int* total, int* sh) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  int v = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(v, o, 64);
    if (lane >= o) v += t;
  }
  if (lane == 63) sh[wid] = v;
  __syncthreads();
  int base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const int s = sh[w];
    base += (w < wid) ? s : 0;
    tot += s;
  }
  *total = tot;
  __syncthreads();
  return base + v - x;
}

__device__ __forceinline__ unsigned key_of(float x) { return __float_as_uint(x) & 0x7fffffffu; }

template <int kThreads>
__global__ __launch_bounds__(kThreads) void topk_rows(const float* __restrict__ x, int64_t len,
                                                      int k, int32_t* __restrict__ oidx,
                                                      float* __restrict__ oval) {
  constexpr int kWaves = kThreads / 64;
  __shared__ unsigned hist[kWaves][256];
  __shared__ unsigned s_prefix, s_need;
  __shared__ int sh[kWaves];
  const int tid = threadIdx.x;
  const int wave = tid >> 6;
  const float* row = x + int64_t(blockIdx.x) * len;
  int32_t* ri = oidx + int64_t(blockIdx.x) * k;
  float* rv = oval + int64_t(blockIdx.x) * k;

  unsigned prefix = 0, mask = 0, need = unsigned(k);
  const bool all = int64_t(k) >= len;
  if (!all) {
    for (int pass = 0; pass < 4; ++pass) {
      const int shift = 24 - 8 * pass;
      for (int b = tid; b < kWaves * 256; b += kThreads) (&hist[0][0])[b] = 0;
      __syncthreads();
      int64_t i = tid;
      for (; i + 3 * kThreads < len; i += 4 * kThreads) {
        float v4[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v4[j] = row[i + j * kThreads];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const unsigned u = key_of(v4[j]);
          if ((u & mask) == prefix) atomicAdd(&hist[wave][(u >> shift) & 255u], 1u);
        }
      }
      for (; i < len; i += kThreads) {
        const unsigned u = key_of(row[i]);
        if ((u & mask) == prefix) atomicAdd(&hist[wave][(u >> shift) & 255u], 1u);
      }
      __syncthreads();
      for (int b = tid; b < 256; b += kThreads) {
        unsigned t = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) t += hist[w][b];
        hist[0][b] = t;
      }
      __syncthreads();
      if (tid == 0) {
        unsigned cum = 0;
        int b = 255;
        for (; b > 0; --b) {
          const unsigned c = hist[0][b];
          if (cum + c >= need) break;
          cum += c;
        }
        s_prefix = prefix | (unsigned(b) << shift);
        s_need = need - cum;
      }
      __syncthreads();
      prefix = s_prefix;
      need = s_need;
      mask |= 255u << shift;
    }
  }
  const unsigned thr = prefix;

  int out_base = 0, eq_base = 0;
  for (int64_t c0 = 0; c0 < len; c0 += int64_t(kThreads) * kItems) {
    unsigned gt = 0, eq = 0;
    float v[kItems];
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      const int64_t i = c0 + int64_t(tid) * kItems + j;
      v[j] = i < len ? row[i] : 0.0f;
      if (i < len) {
        const unsigned u = key_of(v[j]);
        if (all || u > thr) gt |= 1u << j;
        else if (u == thr) eq |= 1u << j;
      }
    }
    int eq_total;
    const int eq_off = block_scan<kWaves>(__popc(eq), &eq_total, sh);
    // the first `need` equal keys (in position order) are kept
    unsigned sel = gt;
    int rank = eq_base + eq_off;
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      if (eq & (1u << j)) {
        if (unsigned(rank) < need) sel |= 1u << j;
        ++rank;
      }
    }
    int sel_total;
    int pos = out_base + block_scan<kWaves>(__popc(sel), &sel_total, sh);
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      if (sel & (1u << j)) {
        if (pos < k) {
          ri[pos] = int32_t(c0 + int64_t(tid) * kItems + j);
          rv[pos] = v[j];
        }
        ++pos;
      }
    }
    out_base += sel_total;
    eq_base += eq_total;
  }
}

// ---------------------------------------------------------------------------
// One workgroup per row, the row read twice.
//
// What bounds it: reading the row.  The radix select above reads it five
// times, adds every value to a histogram of 256 bins in LDS (the zeros that
// fill most of a transport row all into one) and has one thread look through
// each; here zeros are counted by difference, and a bin of 11 bits (an eighth
// of a power of two) leaves a few hundred candidates.  512 rows of 98,304, k =
// 256: 446 -> 80 us, 2.5 TB/s of the row once (it is read twice); 1,024 threads
// per row, two rows per CU; 256 threads for rows up to 8,192.
// ---------------------------------------------------------------------------
constexpr int kSelBits = 11;
constexpr int kSelBins = 1 << kSelBits;
constexpr int kSelShift = 31 - kSelBits;
// Candidates (key, position) listed in the bins' place and ranked against each
// other: more take ten more bits first (936 zeros around the threshold of short
// rows took 400 us to rank).
constexpr int kSelCand = 384;
static_assert(2 * kSelCand <= kSelBins, "the list fits the bins");
constexpr int64_t kSelMaxLen = 6 * 256 * 256;  // 48 KiB of bits

// f(position, value) for every value of the row, 16 bytes at a time where its
// start and length allow; the same thread takes the same positions each time.
template <int kThreads, typename F>
__device__ __forceinline__ void for_row(const float* __restrict__ row, int len, bool wide, F f) {
  const int tid = threadIdx.x;
  if (wide) {
    const float4* r4 = reinterpret_cast<const float4*>(row);
    const int n4 = len >> 2;
    int i = tid;
    for (; i + 3 * kThreads < n4; i += 4 * kThreads) {
      float4 v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = r4[i + j * kThreads];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int at = 4 * (i + j * kThreads);
        f(at, v[j].x);
        f(at + 1, v[j].y);
        f(at + 2, v[j].z);
        f(at + 3, v[j].w);
      }
    }
    for (; i < n4; i += kThreads) {
      const float4 v = r4[i];
      f(4 * i, v.x);
      f(4 * i + 1, v.y);
      f(4 * i + 2, v.z);
      f(4 * i + 3, v.w);
    }
  } else {
    for (int i = tid; i < len; i += kThreads) f(i, row[i]);
  }
}

// The bin of `nb` (a multiple of kThreads, at most kSelBins) that holds the
// need-th largest key, with zeros added to bin 0: bin and the number needed
// from it, through s_bin and s_need.
template <int kThreads>
__device__ __forceinline__ void find_bin(const unsigned* hist, int nb, unsigned zeros, unsigned need,
                                         int* s_bin, int* s_need, int* sh) {
  const int tid = threadIdx.x;
  const int per = nb / kThreads > 0 ? nb / kThreads : 1;
  const bool mine_ok = per * tid < nb;
  unsigned mine = 0;
  for (int j = 0; mine_ok && j < per; ++j) mine += hist[per * tid + j];
  if (tid == 0) mine += zeros;
  int total;
  const int before = block_scan<kThreads / 64>(int(mine), &total, sh);
  unsigned above = unsigned(total) - unsigned(before) - mine;
  for (int j = per - 1; mine_ok && j >= 0; --j) {
    unsigned c = hist[per * tid + j];
    if (tid == 0 && j == 0) c += zeros;
    if (above < need && above + c >= need) {
      *s_bin = per * tid + j;
      *s_need = int(need - above);
    }
    above += c;
  }
  __syncthreads();
}

template <int kThreads>
__global__ __launch_bounds__(kThreads) void topk_select(const float* __restrict__ x, int len, int k,
                                                        int32_t* __restrict__ oidx,
                                                        float* __restrict__ oval) {
  constexpr int kWaves = kThreads / 64;
  extern __shared__ __align__(8) unsigned lds[];
  unsigned* hist = lds;             // kSelBins; later the candidates
  unsigned* bits = lds + kSelBins;  // one bit per position
  __shared__ int sh[kWaves];
  __shared__ int s_bin, s_need, s_count;
  const int tid = threadIdx.x;
  const int words = (len + 31) >> 5;
  const float* row = x + int64_t(blockIdx.x) * len;
  int32_t* ri = oidx + int64_t(blockIdx.x) * k;
  float* rv = oval + int64_t(blockIdx.x) * k;
  const bool wide = ((reinterpret_cast<uintptr_t>(row) | unsigned(len * 4)) & 15u) == 0;
  for (int b = tid; b < kSelBins + words; b += kThreads) lds[b] = 0u;
  if (tid == 0) s_count = 0;
  __syncthreads();
  // histogram of the nonzero keys; zeros are the rest
  int nonzero = 0;
  for_row<kThreads>(row, len, wide, [&](int, float v) {
    const unsigned u = key_of(v);
    if (u) {
      atomicAdd(&hist[u >> kSelShift], 1u);
      ++nonzero;
    }
  });
  __syncthreads();
  int total;
  block_scan<kWaves>(nonzero, &total, sh);
  const unsigned zeros = unsigned(len - total);
  find_bin<kThreads>(hist, kSelBins, zeros, unsigned(k), &s_bin, &s_need, sh);
  unsigned need = unsigned(s_need);
  // the bits above `shift` of the keys in the bin
  int shift = kSelShift;
  unsigned bin = unsigned(s_bin);
  unsigned in_bin = hist[bin] + (bin == 0 ? zeros : 0u);
  __syncthreads();
  // more candidates than the list holds: ten more bits (at most twice)
  while (in_bin > unsigned(kSelCand) && shift > 0) {
    for (int b = tid; b < 1024; b += kThreads) hist[b] = 0u;
    __syncthreads();
    for_row<kThreads>(row, len, wide, [&](int, float v) {
      const unsigned u = key_of(v);
      if (u && u >> shift == bin) atomicAdd(&hist[(u >> (shift - 10)) & 1023u], 1u);
    });
    __syncthreads();
    const unsigned extra = bin == 0 ? zeros : 0u;
    find_bin<kThreads>(hist, 1024, extra, need, &s_bin, &s_need, sh);
    need = unsigned(s_need);
    in_bin = hist[s_bin] + (s_bin == 0 ? extra : 0u);
    bin = bin << 10 | unsigned(s_bin);
    shift -= 10;
    __syncthreads();
  }
  if (in_bin <= unsigned(kSelCand)) {
    // keys above the bin are kept, the bin's are listed ...
    for_row<kThreads>(row, len, wide, [&](int i, float v) {
      const unsigned u = key_of(v), b = u >> shift;
      if (b > bin) {
        atomicOr(&bits[i >> 5], 1u << (i & 31));
      } else if (b == bin) {
        const int at = atomicAdd(&s_count, 1);
        hist[2 * at] = u;
        hist[2 * at + 1] = unsigned(i);
      }
    });
    __syncthreads();
    // ... and those of a rank (larger key, then lower position) below `need` kept
    const int m = int(in_bin);
    const uint2* list = reinterpret_cast<const uint2*>(hist);
    for (int c = tid; c < m; c += kThreads) {
      const unsigned u = list[c].x, i = list[c].y;
      unsigned rank = 0;
#pragma unroll 8
      for (int j = 0; j < m; ++j) {
        const uint2 o = list[j];
        rank += (o.x > u || (o.x == u && o.y < i)) ? 1u : 0u;
      }
      if (rank < need) atomicOr(&bits[i >> 5], 1u << (i & 31));
    }
  } else {
    // many equal keys: the first `need` of them in position order
    const unsigned prefix = bin;
    int base = 0;
    for (int c0 = 0; c0 < len; c0 += kThreads * kItems) {
      unsigned keep = 0, eq = 0;
#pragma unroll
      for (int j = 0; j < kItems; ++j) {
        const int i = c0 + tid * kItems + j;
        const unsigned u = i < len ? key_of(row[i]) : 0u;
        if (i < len && u > prefix) keep |= 1u << j;
        if (i < len && u == prefix) eq |= 1u << j;
      }
      int eqs;
      int rank = base + block_scan<kWaves>(__popc(eq), &eqs, sh);
#pragma unroll
      for (int j = 0; j < kItems; ++j) {
        if (eq & (1u << j)) {
          if (rank < int(need)) keep |= 1u << j;
          ++rank;
        }
      }
      base += eqs;
      const int i = c0 + tid * kItems;  // kItems positions share a word
      if (keep) atomicOr(&bits[i >> 5], keep << (i & 31));
    }
  }
  __syncthreads();
  // emission: each thread's words follow those of the threads before it
  const int per = (words + kThreads - 1) / kThreads;
  const int w0 = tid * per, w1 = w0 + per < words ? w0 + per : words;
  int count = 0;
  for (int w = w0; w < w1; ++w) count += __popc(bits[w]);
  int kept;
  int pos = block_scan<kWaves>(count, &kept, sh);
  for (int w = w0; w < w1; ++w) {
    unsigned m = bits[w];
    while (m) {
      const int i = 32 * w + __builtin_ctz(m);
      m &= m - 1;
      if (pos < k) {
        ri[pos] = i;
        rv[pos] = row[i];
      }
      ++pos;
    }
  }
}

// k = len: every value in place.
__global__ void topk_all(const float* __restrict__ x, int64_t total, int64_t len,
                         int32_t* __restrict__ oidx, float* __restrict__ oval) {
  const int64_t step = int64_t(gridDim.x) * blockDim.x;
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < total; i += step) {
    oidx[i] = int32_t(i % len);
    oval[i] = x[i];
  }
}

// ---------------------------------------------------------------------------
// A few long rows (one environment map): the row is split into chunks
// processed by many workgroups.
//   1. per-chunk histograms of the top 12 key bits, added up over the chunks
//      (in the candidate list's space, cleared first);
//   2. per row: the bin holding the k-th largest key and, per chunk, the
//      start of that bin's keys in a candidate list;
//   3. per chunk: the candidates, compacted in position order;
//   4. per row: radix select over the candidates' remaining 19 bits gives the
//      exact threshold key t and how many keys equal to t are kept; the
//      position of the last kept one is the cut;
//   5. per chunk: the number of kept entries (key > t, or key == t at a
//      position up to the cut);
//   6. per chunk: ordered emission at the sum of the preceding chunks' counts.
// ---------------------------------------------------------------------------
constexpr int kBinBits = 12;
constexpr int kBins = 1 << kBinBits;
constexpr int kLowBits = 31 - kBinBits;  // key bits below the bin
constexpr int kMaxChunks = 64;
constexpr int kMinChunk = 4096;
constexpr int kChunkThreads = 256;

// Per-row parameters in the workspace.
enum { P_BIN, P_NEED, P_CAND, P_THR, P_CUT, P_COUNT };

struct ChunkPlan {
  int chunks;
  int64_t chunk_len;
};

ChunkPlan chunk_plan(int64_t len) {
  int64_t chunks = (len + kMinChunk - 1) / kMinChunk;
  if (chunks > kMaxChunks) chunks = kMaxChunks;
  ChunkPlan c;
  c.chunks = int(chunks);
  c.chunk_len = (len + chunks - 1) / chunks;
  return c;
}

struct TopkWs {
  uint32_t* hist;     // [rows][chunks][kBins]
  uint32_t* eq_base;  // [rows][chunks]
  uint32_t* sel_cnt;  // [rows][chunks]
  uint32_t* par;      // [rows][P_COUNT]
  uint32_t* ckey;     // [rows][len]
  int32_t* cidx;      // [rows][len]
};

size_t carve(void* base, int64_t rows, int64_t len, TopkWs* w) {
  const ChunkPlan cp = chunk_plan(len);
  char* p = static_cast<char*>(base);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* q = p ? p + off : nullptr;
    off += align256(bytes);
    return q;
  };
  TopkWs t;
  t.hist = reinterpret_cast<uint32_t*>(take(size_t(rows) * cp.chunks * kBins * 4));
  t.eq_base = reinterpret_cast<uint32_t*>(take(size_t(rows) * cp.chunks * 4));
  t.sel_cnt = reinterpret_cast<uint32_t*>(take(size_t(rows) * cp.chunks * 4));
  t.par = reinterpret_cast<uint32_t*>(take(size_t(rows) * P_COUNT * 4));
  t.ckey = reinterpret_cast<uint32_t*>(take(size_t(rows) * len * 4));
  t.cidx = reinterpret_cast<int32_t*>(take(size_t(rows) * len * 4));
  if (w) *w = t;
  return off;
}

// Sum over the workgroup; every thread gets the total.
template <int kWaves>
__device__ __forceinline__ int block_sum(int x, int* sh) {
  int total;
  block_scan<kWaves>(x, &total, sh);
  return total;
}

__global__ __launch_bounds__(kChunkThreads) void tk_clear(uint32_t* __restrict__ tot, int64_t len) {
  tot[int64_t(blockIdx.y) * len + blockIdx.x * kChunkThreads + threadIdx.x] = 0u;
}

// tot: the row's histogram, at the start of its candidate list.  (The bin
// search read it from the chunks' own before, one after the other: 32 us of the
// 57 that one row of 98,304 took.)
__global__ __launch_bounds__(kChunkThreads) void tk_hist(const float* __restrict__ x, int64_t len,
                                                         int64_t chunk_len, int chunks,
                                                         uint32_t* __restrict__ hist,
                                                         uint32_t* __restrict__ tot) {
  __shared__ unsigned h[kBins];
  const int tid = threadIdx.x, c = blockIdx.x, row = blockIdx.y;
  for (int b = tid; b < kBins; b += kChunkThreads) h[b] = 0;
  __syncthreads();
  const float* r = x + int64_t(row) * len;
  const int64_t lo = int64_t(c) * chunk_len;
  const int64_t hi = lo + chunk_len < len ? lo + chunk_len : len;
  int64_t i = lo + tid;
  for (; i + 3 * kChunkThreads < hi; i += 4 * kChunkThreads) {
    float v4[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v4[j] = r[i + j * kChunkThreads];
#pragma unroll
    for (int j = 0; j < 4; ++j) atomicAdd(&h[key_of(v4[j]) >> kLowBits], 1u);
  }
  for (; i < hi; i += kChunkThreads) atomicAdd(&h[key_of(r[i]) >> kLowBits], 1u);
  __syncthreads();
  uint32_t* out = hist + (int64_t(row) * chunks + c) * kBins;
  uint32_t* sum = tot + int64_t(row) * len;
  for (int b = tid; b < kBins; b += kChunkThreads) {
    const unsigned c = h[b];
    out[b] = c;
    if (c) atomicAdd(&sum[b], c);
  }
}

// The single-workgroup steps of a long row run as four waves (one per SIMD)
// of at most 32 VGPRs with dynamic LDS, so that they find room on a CU next
// to other work (a relight kernel holding 5 waves of 96 VGPRs per SIMD
// leaves 32 per SIMD).
constexpr int kSmallThreads = 256;
#define RRT_SMALL_STEP __global__ __launch_bounds__(kSmallThreads)

RRT_SMALL_STEP void tk_bin(const uint32_t* __restrict__ hist, const uint32_t* __restrict__ sums,
                           int64_t len, int chunks, int k,
                           uint32_t* __restrict__ eq_base, uint32_t* __restrict__ par) {
  constexpr int kWaves = kSmallThreads / 64;
  constexpr int kPer = kBins / kSmallThreads;
  // per-bin totals in dynamic LDS (kBins words): with a static array the
  // compiler pads the register allocation to the occupancy the LDS allows,
  // which keeps the wave from running beside other kernels
  extern __shared__ unsigned tot[];
  __shared__ int sh[kWaves];
  __shared__ int s_bin, s_need;
  const int tid = threadIdx.x, row = blockIdx.x;
  if (tid == 0) {
    s_bin = 0;
    s_need = 0;
  }
  const uint32_t* h = hist + int64_t(row) * chunks * kBins;
#pragma unroll 4
  for (int b = tid; b < kBins; b += kSmallThreads) tot[b] = sums[int64_t(row) * len + b];
  __syncthreads();
  // this thread's bins kPer tid .. kPer tid + kPer - 1
  const unsigned* mt = tot + kPer * tid;
  int mine = 0;
#pragma unroll 4
  for (int j = 0; j < kPer; ++j) mine += int(mt[j]);
  int total;
  const int before = block_scan<kWaves>(mine, &total, sh);
  // keys in bins above this thread's bins
  unsigned above = unsigned(total - before - mine);
#pragma unroll 4
  for (int j = kPer - 1; j >= 0; --j) {
    const unsigned c = mt[j];
    if (above < unsigned(k) && above + c >= unsigned(k)) {
      s_bin = kPer * tid + j;
      s_need = int(unsigned(k) - above);
    }
    above += c;
  }
  __syncthreads();
  const int bin = s_bin;
  // start of each chunk's candidates (keys in the bin), in chunk order
  if (tid < 64) {
    int run = 0;
    for (int c0 = 0; c0 < chunks; c0 += 64) {
      const int c = c0 + tid;
      const int cnt = c < chunks ? int(h[int64_t(c) * kBins + bin]) : 0;
      int v = cnt;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(v, o, 64);
        if (tid >= o) v += t;
      }
      if (c < chunks) eq_base[int64_t(row) * chunks + c] = unsigned(run + v - cnt);
      run += __shfl(v, 63, 64);
    }
    if (tid == 0) {
      uint32_t* pr = par + int64_t(row) * P_COUNT;
      pr[P_BIN] = unsigned(bin);
      pr[P_NEED] = unsigned(s_need);
      pr[P_CAND] = unsigned(run);
    }
  }
}

// Ordered compaction helper: the keep flags of kItems consecutive positions
// per thread become positions base + rank in position order.
template <int kThreads, typename Pred, typename Emit>
__device__ __forceinline__ int ordered_pass(int64_t lo, int64_t hi, int base, int* sh, Pred keep,
                                            Emit emit) {
  constexpr int kWaves = kThreads / 64;
  for (int64_t c0 = lo; c0 < hi; c0 += int64_t(kThreads) * kItems) {
    unsigned sel = 0;
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      const int64_t i = c0 + int64_t(threadIdx.x) * kItems + j;
      if (i < hi && keep(i)) sel |= 1u << j;
    }
    int total;
    int pos = base + block_scan<kWaves>(__popc(sel), &total, sh);
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      if (sel & (1u << j)) emit(c0 + int64_t(threadIdx.x) * kItems + j, pos++);
    }
    base += total;
  }
  return base;
}

__global__ __launch_bounds__(kChunkThreads) void tk_cand(const float* __restrict__ x, int64_t len,
                                                         int64_t chunk_len, int chunks,
                                                         const uint32_t* __restrict__ eq_base,
                                                         const uint32_t* __restrict__ par,
                                                         uint32_t* __restrict__ ckey,
                                                         int32_t* __restrict__ cidx) {
  __shared__ int sh[kChunkThreads / 64];
  const int c = blockIdx.x, row = blockIdx.y;
  const float* r = x + int64_t(row) * len;
  const unsigned bin = par[int64_t(row) * P_COUNT + P_BIN];
  const int64_t lo = int64_t(c) * chunk_len;
  const int64_t hi = lo + chunk_len < len ? lo + chunk_len : len;
  uint32_t* kk = ckey + int64_t(row) * len;
  int32_t* ki = cidx + int64_t(row) * len;
  ordered_pass<kChunkThreads>(
      lo, hi, int(eq_base[int64_t(row) * chunks + c]), sh,
      [&](int64_t i) { return (key_of(r[i]) >> kLowBits) == bin; },
      [&](int64_t i, int pos) {
        kk[pos] = key_of(r[i]);
        ki[pos] = int32_t(i);
      });
}

RRT_SMALL_STEP void tk_resolve(int64_t len,
                                                            const uint32_t* __restrict__ ckey,
                                                            const int32_t* __restrict__ cidx,
                                                            uint32_t* __restrict__ par) {
  constexpr int kWaves = kSmallThreads / 64;
  __shared__ unsigned h[1024];
  __shared__ int sh[kWaves];
  __shared__ unsigned s_prefix, s_need;
  __shared__ int s_cut;
  const int tid = threadIdx.x, row = blockIdx.x;
  uint32_t* pr = par + int64_t(row) * P_COUNT;
  const int m = int(pr[P_CAND]);
  const uint32_t* kk = ckey + int64_t(row) * len;
  const int32_t* ki = cidx + int64_t(row) * len;
  unsigned prefix = pr[P_BIN] << kLowBits;
  unsigned mask = ~((1u << kLowBits) - 1u) & 0x7fffffffu;
  unsigned need = pr[P_NEED];
  // two passes: bits 18..9 (1024 bins), then bits 8..0 (512 bins)
  for (int pass = 0; pass < 2; ++pass) {
    const int shift = pass == 0 ? 9 : 0;
    const int nb = pass == 0 ? 1024 : 512;
    if (tid == 0) {
      s_prefix = prefix;
      s_need = need;
    }
    for (int b = tid; b < nb; b += kSmallThreads) h[b] = 0;
    __syncthreads();
    for (int i = tid; i < m; i += kSmallThreads) {
      const unsigned u = kk[i];
      if ((u & mask) == prefix) atomicAdd(&h[(u >> shift) & unsigned(nb - 1)], 1u);
    }
    __syncthreads();
    // bins per * tid .. per * tid + per - 1 of this thread: keys above them,
    // then each bin from the top
    const int per = nb / kSmallThreads;
    int mine = 0;
    for (int j = 0; j < per; ++j) mine += int(h[per * tid + j]);
    int total;
    const int before = block_scan<kWaves>(mine, &total, sh);
    unsigned above = unsigned(total - before - mine);
    for (int j = per - 1; j >= 0; --j) {
      const unsigned c = h[per * tid + j];
      if (above < need && above + c >= need) {
        s_prefix = prefix | (unsigned(per * tid + j) << shift);
        s_need = need - above;
      }
      above += c;
    }
    __syncthreads();
    prefix = s_prefix;
    need = s_need;
    mask |= unsigned(nb - 1) << shift;
    __syncthreads();
  }
  // the need-th key equal to the threshold, in position order
  if (tid == 0) s_cut = -1;
  __syncthreads();
  int base = 0;
  for (int c0 = 0; c0 < m && base < int(need); c0 += kSmallThreads) {
    const int i = c0 + tid;
    const int eq = (i < m && kk[i] == prefix) ? 1 : 0;
    int total;
    const int rank = base + block_scan<kWaves>(eq, &total, sh);
    if (eq && rank == int(need) - 1) s_cut = ki[i];
    base += total;
  }
  __syncthreads();
  if (tid == 0) {
    pr[P_THR] = prefix;
    pr[P_CUT] = unsigned(s_cut);
  }
}

__device__ __forceinline__ bool kept(float v, int64_t i, unsigned thr, int cut) {
  const unsigned u = key_of(v);
  return u > thr || (u == thr && i <= int64_t(cut));
}

__global__ __launch_bounds__(kChunkThreads) void tk_count(const float* __restrict__ x, int64_t len,
                                                          int64_t chunk_len, int chunks,
                                                          const uint32_t* __restrict__ par,
                                                          uint32_t* __restrict__ sel_cnt) {
  __shared__ int sh[kChunkThreads / 64];
  const int c = blockIdx.x, row = blockIdx.y;
  const float* r = x + int64_t(row) * len;
  const unsigned thr = par[int64_t(row) * P_COUNT + P_THR];
  const int cut = int(par[int64_t(row) * P_COUNT + P_CUT]);
  const int64_t lo = int64_t(c) * chunk_len;
  const int64_t hi = lo + chunk_len < len ? lo + chunk_len : len;
  int n = 0;
  for (int64_t i = lo + threadIdx.x; i < hi; i += kChunkThreads) n += kept(r[i], i, thr, cut);
  n = block_sum<kChunkThreads / 64>(n, sh);
  if (threadIdx.x == 0) sel_cnt[int64_t(row) * chunks + c] = unsigned(n);
}

__global__ __launch_bounds__(kChunkThreads) void tk_emit(const float* __restrict__ x, int64_t len,
                                                         int64_t chunk_len, int chunks, int k,
                                                         const uint32_t* __restrict__ par,
                                                         const uint32_t* __restrict__ sel_cnt,
                                                         int32_t* __restrict__ oidx,
                                                         float* __restrict__ oval) {
  __shared__ int sh[kChunkThreads / 64];
  const int c = blockIdx.x, row = blockIdx.y;
  const float* r = x + int64_t(row) * len;
  const unsigned thr = par[int64_t(row) * P_COUNT + P_THR];
  const int cut = int(par[int64_t(row) * P_COUNT + P_CUT]);
  const int64_t lo = int64_t(c) * chunk_len;
  const int64_t hi = lo + chunk_len < len ? lo + chunk_len : len;
  int before = 0;
  for (int c2 = threadIdx.x; c2 < c; c2 += kChunkThreads)
    before += int(sel_cnt[int64_t(row) * chunks + c2]);
  before = block_sum<kChunkThreads / 64>(before, sh);
  int32_t* ri = oidx + int64_t(row) * k;
  float* rv = oval + int64_t(row) * k;
  ordered_pass<kChunkThreads>(
      lo, hi, before, sh, [&](int64_t i) { return kept(r[i], i, thr, cut); },
      [&](int64_t i, int pos) {
        if (pos < k) {
          ri[pos] = int32_t(i);
          rv[pos] = r[i];
        }
      });
}

bool few_long_rows(int64_t rows, int64_t len, int k) {
  return rows <= 8 && len >= 16384 && int64_t(k) < len;
}

}  // namespace

size_t topk_workspace_bytes(int64_t rows, int64_t len, int k) {
  return few_long_rows(rows, len, k) ? carve(nullptr, rows, len, nullptr) : 0;
}

int launch_topk(const float* x, int64_t rows, int64_t len, int k, int32_t* idx, float* val,
                void* ws, hipStream_t s) {
  if (rows == 0 || k == 0) return RRT_OK;
  const int64_t total = rows * len;
  // (a launch has fewer than 2^32 threads: the grid ends at 2^30 and goes on from
  // there, and so many long rows take the smaller workgroup)
  if (int64_t(k) == len) {
    const int64_t grid = (total + 255) / 256, most = int64_t(1) << 22;
    hipLaunchKernelGGL(topk_all, dim3(unsigned(grid < most ? grid : most)), dim3(256), 0, s, x, total,
                       len, idx, val);
    return check_launch("topk_all");
  }
  // One workgroup for a row of a map's coefficients: 80 us for 512 rows of
  // 98,304 (radix select 446), 26 us for 9 (192), 26 us for 2,048 rows of 6,144
  // (108); a few long rows would leave most CUs idle (92 us for one row of
  // 98,304 log-normal values against 33).
  if (len <= kSelMaxLen && !few_long_rows(rows, len, k)) {
    const size_t lds = (kSelBins + size_t((len + 31) >> 5)) * sizeof(unsigned);
    if (len > 8192 && rows < (int64_t(1) << 22)) {
      hipLaunchKernelGGL(topk_select<1024>, dim3(unsigned(rows)), dim3(1024), lds, s, x, int(len), k,
                         idx, val);
    } else {
      hipLaunchKernelGGL(topk_select<256>, dim3(unsigned(rows)), dim3(256), lds, s, x, int(len), k,
                         idx, val);
    }
    return check_launch("topk_select");
  }
  if (few_long_rows(rows, len, k)) {
    TopkWs w;
    carve(ws, rows, len, &w);
    const ChunkPlan cp = chunk_plan(len);
    const dim3 grid(unsigned(cp.chunks), unsigned(rows));
    hipLaunchKernelGGL(tk_clear, dim3(kBins / kChunkThreads, unsigned(rows)), dim3(kChunkThreads), 0, s,
                       w.ckey, len);
    hipLaunchKernelGGL(tk_hist, grid, dim3(kChunkThreads), 0, s, x, len, cp.chunk_len, cp.chunks,
                       w.hist, w.ckey);
    hipLaunchKernelGGL(tk_bin, dim3(unsigned(rows)), dim3(kSmallThreads), kBins * sizeof(unsigned), s,
                       w.hist, w.ckey, len, cp.chunks, k,
                       w.eq_base, w.par);
    hipLaunchKernelGGL(tk_cand, grid, dim3(kChunkThreads), 0, s, x, len, cp.chunk_len, cp.chunks,
                       w.eq_base, w.par, w.ckey, w.cidx);
    hipLaunchKernelGGL(tk_resolve, dim3(unsigned(rows)), dim3(kSmallThreads), 0, s, len, w.ckey,
                       w.cidx, w.par);
    hipLaunchKernelGGL(tk_count, grid, dim3(kChunkThreads), 0, s, x, len, cp.chunk_len, cp.chunks,
                       w.par, w.sel_cnt);
    hipLaunchKernelGGL(tk_emit, grid, dim3(kChunkThreads), 0, s, x, len, cp.chunk_len, cp.chunks,
                       k, w.par, w.sel_cnt, idx, val);
    return check_launch("topk chunks");
  }
  if (rows < 64 && len >= 16384) {
    hipLaunchKernelGGL(topk_rows<1024>, dim3(unsigned(rows)), dim3(1024), 0, s, x, len, k, idx,
                       val);
  } else {
    hipLaunchKernelGGL(topk_rows<256>, dim3(unsigned(rows)), dim3(256), 0, s, x, len, k, idx, val);
  }
  return check_launch("topk_rows");
}

}  // namespace rrt
