// Device kernels of the SELL-C-sigma construction (Sects. 3.3 and 3.4 of
// Kreutzer et al., arXiv:1307.6209): row lengths and CRS validation, the
// sigma-window sort, chunk widths (Eq. (max)), chunk offsets (prefix sum of
// C * cl[i]) and the padded column-major fill.
#include "sell_internal.h"

#include <hip/hip_bf16.h>

namespace sell {

namespace {

constexpr int kBlock = 256;

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

template <typename T>
__device__ __forceinline__ T wave_max(T v) {
  for (int off = 32; off > 0; off >>= 1) {
    T o = __shfl_xor(v, off);
    v = o > v ? o : v;
  }
  return v;
}

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// Orders the LDS accesses of a wave's lanes among each other.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Validation flag bits.
constexpr uint32_t F_RPT0 = 1u, F_DECR = 2u, F_COL = 4u, F_RPTN = 8u, F_LONG = 16u;

// len[i] = rpt[i+1] - rpt[i]; flags for a malformed rpt; sum of squared
// lengths (for the coefficient of variation) and the longest row. A fixed
// grid strides over the rows, U of a thread's loads in flight, and reduces per
// block; the blocks' atomics on the three totals take turns (10 ns each: with
// 1,024 blocks they made 20 of the 31 us that it took on 1M to 2M rows, now 11 to 13).
constexpr int kStrideBlock = 1024;
constexpr int kStrideGrid = 256;

__global__ void __launch_bounds__(kStrideBlock) k_rowlen(const int64_t *__restrict__ rpt, int64_t n, int64_t nnz,
                                                         int32_t *__restrict__ len, uint32_t *flags,
                                                         unsigned long long *sumsq, int32_t *maxlen) {
  constexpr int U = 4;
  __shared__ unsigned long long s_sq[kStrideBlock / 64];
  __shared__ int32_t s_mx[kStrideBlock / 64];
  __shared__ uint32_t s_f[kStrideBlock / 64];
  uint32_t f = 0;
  int32_t mx = 0;
  unsigned long long sq = 0;
  const int64_t stride = (int64_t)gridDim.x * kStrideBlock;
  for (int64_t i0 = (int64_t)blockIdx.x * kStrideBlock + threadIdx.x; i0 < n; i0 += U * stride) {
    int64_t d[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + u * stride;
      d[u] = i < n ? rpt[i + 1] - rpt[i] : 0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = i0 + u * stride;
      if (i >= n) continue;
      if (d[u] < 0) f |= F_DECR;
      if (d[u] > 0x7fffffffLL) f |= F_LONG;
      const int32_t l = (d[u] < 0 || d[u] > 0x7fffffffLL) ? 0 : (int32_t)d[u];
      len[i] = l;
      sq += (unsigned long long)l * (unsigned long long)l;
      mx = l > mx ? l : mx;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (rpt[0] != 0) f |= F_RPT0;
    if (rpt[n] != nnz) f |= F_RPTN;
  }
  sq = wave_sum_u64(sq);
  mx = wave_max(mx);
  for (int off = 32; off > 0; off >>= 1) f |= __shfl_xor(f, off);
  const int w = threadIdx.x >> 6;
  if (lane_id() == 0) {
    s_sq[w] = sq;
    s_mx[w] = mx;
    s_f[w] = f;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < kStrideBlock / 64; ++k) {
      sq += s_sq[k];
      mx = s_mx[k] > mx ? s_mx[k] : mx;
      f |= s_f[k];
    }
    if (sq) atomicAdd(sumsq, sq);
    if (mx) atomicMax(maxlen, mx);
    if (f) atomicOr(flags, f);
  }
}

// Every column index within [0, ncols): 16 bytes an access, four in flight (the
// array may start at any element: the first few and the last ones singly).
__global__ void __launch_bounds__(kBlock) k_colcheck(const int32_t *__restrict__ col, int64_t nnz, int64_t ncols,
                                                     uint32_t *flags) {
  constexpr int U = 4;
  const int64_t head0 = (int64_t)((16 - (reinterpret_cast<uintptr_t>(col) & 15)) & 15) / 4;
  const int64_t head = head0 < nnz ? head0 : nnz, quads = (nnz - head) / 4;
  const int4 *q = reinterpret_cast<const int4 *>(col + head);
  const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x, stride = (int64_t)gridDim.x * kBlock;
  const uint32_t lim = (uint32_t)ncols;  // below 2^31: a negative index is above it unsigned
  bool bad = false;
  for (int64_t j = t; j < quads; j += U * stride) {
    int4 c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) c[u] = j + u * stride < quads ? q[j + u * stride] : q[j];
#pragma unroll
    for (int u = 0; u < U; ++u)
      bad |= ((uint32_t)c[u].x >= lim) | ((uint32_t)c[u].y >= lim) | ((uint32_t)c[u].z >= lim) |
             ((uint32_t)c[u].w >= lim);
  }
  if (t < head) bad |= (uint32_t)col[t] >= lim;
  if (t < nnz - head - 4 * quads) bad |= (uint32_t)col[head + 4 * quads + t] >= lim;
  if (__ballot(bad) != 0ull && lane_id() == 0) atomicOr(flags, F_COL);
}

// ---------------------------------------------------------------------------
// sigma-window sort.
//
// Rows are ordered by descending length inside each window of sigma rows,
// ties by ascending row index.
//
// sigma <= kTile: tiles of whole windows are sorted in LDS (bitonic network)
// by a 64-bit key that is unique and whose ascending order is that order:
// (window in the tile, INT32_MAX - len, index).
//
// sigma > kTile: two stable counting passes over tiles of kTile rows of one
// window, by the low byte of the length and then by the rest of it (255 for all
// of 65,280 or more), longest first: counts per (window, digit, tile), their
// exclusive prefix, ranks inside the tile. Rows of 65,280 entries or more then
// stand in front of their window in the order of their low byte; k_sort_longest
// goes on with the higher ones. (Sorted tiles merged pairwise, log2(sigma /
// kTile) passes of binary searches: 191 us on one window of 1M rows, now 47.)
// ---------------------------------------------------------------------------
constexpr int kTile = 4096;
constexpr int kSortBlock = 512;

__global__ void __launch_bounds__(kSortBlock) k_sort_tiles(const int32_t *__restrict__ len, int64_t n,
                                                           int64_t sigma, int32_t *__restrict__ perm_out) {
  __shared__ uint64_t sk[kTile];
  const int64_t tile_rows = kTile / sigma * sigma;  // whole windows per tile
  const int64_t start = (int64_t)blockIdx.x * tile_rows;
  const int64_t count = n - start < tile_rows ? n - start : tile_rows;
  if (count <= 0) return;  // uniform over the block
  for (int q = threadIdx.x; q < kTile; q += kSortBlock) {
    uint64_t key = ~0ull;
    if (q < count) {
      const uint64_t inv = (uint64_t)(0x7fffffff - len[start + q]), wl = (uint64_t)(q / sigma);
      key = (wl << 44) | (inv << 13) | (uint64_t)q;
    }
    sk[q] = key;
  }
  __syncthreads();
  // bitonic sort, ascending
  for (int size = 2; size <= kTile; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int t = threadIdx.x; t < kTile / 2; t += kSortBlock) {
        int lo = 2 * t - (t & (stride - 1));
        int hi = lo + stride;
        bool asc = (lo & size) == 0;
        uint64_t a = sk[lo], b = sk[hi];
        if ((a > b) == asc) {
          sk[lo] = b;
          sk[hi] = a;
        }
      }
      __syncthreads();
    }
  }
  for (int q = threadIdx.x; q < count; q += kSortBlock)
    perm_out[start + q] = (int32_t)(start + (int64_t)(sk[q] & 0x1fffull));
}

// Tile b of the counting passes: rows [start, start + count) of window w.
struct SortTile {
  int64_t start, w, tw;
  int count;
};
__device__ __forceinline__ SortTile sort_tile(int64_t b, int64_t n, int64_t sigma, int64_t per_window) {
  SortTile t;
  t.w = b / per_window;
  t.tw = b - t.w * per_window;
  t.start = t.w * sigma + t.tw * kTile;
  const int64_t end = (t.w + 1) * sigma < n ? (t.w + 1) * sigma : n;
  t.count = end - t.start < kTile ? (end > t.start ? (int)(end - t.start) : 0) : kTile;
  return t;
}

// Digit of a length, 0 for the longest.
template <int PASS>
__device__ __forceinline__ int sort_digit(uint32_t len) {
  if (PASS == 0) return 255 - (int)(len & 255u);
  return 255 - (int)(len >> 8 < 255u ? len >> 8 : 255u);
}

// Row q of the tile: before pass 0 the rows in order, then what pass 0 left
// ((length, row) in 32 bits each).
template <int PASS>
__device__ __forceinline__ uint64_t sort_item(const int32_t *__restrict__ len, const uint64_t *__restrict__ in,
                                              int64_t i) {
  return PASS == 0 ? (uint64_t)(uint32_t)len[i] << 32 | (uint64_t)i : in[i];
}

template <int PASS>
__global__ void __launch_bounds__(kSortBlock) k_sort_count(const int32_t *__restrict__ len,
                                                           const uint64_t *__restrict__ in, int64_t n, int64_t sigma,
                                                           int64_t per_window, int64_t *__restrict__ counts) {
  __shared__ int32_t hist[256];
  const SortTile t = sort_tile(blockIdx.x, n, sigma, per_window);
  if (threadIdx.x < 256) hist[threadIdx.x] = 0;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kTile / kSortBlock; ++k) {
    const int q = k * kSortBlock + threadIdx.x;
    if (q < t.count) atomicAdd(&hist[sort_digit<PASS>((uint32_t)(sort_item<PASS>(len, in, t.start + q) >> 32))], 1);
  }
  __syncthreads();
  if (threadIdx.x < 256) counts[(t.w * 256 + threadIdx.x) * per_window + t.tw] = hist[threadIdx.x];
}

// Wave v of the block takes the tile's rows [512 v, 512 v + 512) in strips of
// 64: a row's place is its digit's (the prefix of the counts, which covers all
// windows in turn, plus the earlier waves' rows of the digit) plus its rank among
// the digit's rows of the wave so far and of its strip.
template <int PASS>
__global__ void __launch_bounds__(kSortBlock) k_sort_place(const int32_t *__restrict__ len,
                                                           const uint64_t *__restrict__ in, int64_t n, int64_t sigma,
                                                           int64_t per_window, const int64_t *__restrict__ places,
                                                           uint64_t *__restrict__ out, int32_t *__restrict__ perm) {
  constexpr int WAVES = kSortBlock / 64, STRIPS = kTile / kSortBlock;
  __shared__ int32_t next[WAVES][256];
  const SortTile t = sort_tile(blockIdx.x, n, sigma, per_window);
  const int lane = lane_id(), v = threadIdx.x >> 6;
  for (int d = lane; d < 256; d += 64) next[v][d] = 0;
  wave_sync();
  uint64_t item[STRIPS];
#pragma unroll
  for (int k = 0; k < STRIPS; ++k) {
    const int q = (v * STRIPS + k) * 64 + lane;
    item[k] = q < t.count ? sort_item<PASS>(len, in, t.start + q) : 0;
  }
#pragma unroll
  for (int k = 0; k < STRIPS; ++k)
    if ((v * STRIPS + k) * 64 + lane < t.count) atomicAdd(&next[v][sort_digit<PASS>((uint32_t)(item[k] >> 32))], 1);
  __syncthreads();
  if (threadIdx.x < 256) {
    int32_t at = (int32_t)places[(t.w * 256 + threadIdx.x) * per_window + t.tw];
#pragma unroll
    for (int u = 0; u < WAVES; ++u) {
      const int32_t c = next[u][threadIdx.x];
      next[u][threadIdx.x] = at;
      at += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < STRIPS; ++k) {
    const bool real = (v * STRIPS + k) * 64 + lane < t.count;
    const int d = sort_digit<PASS>((uint32_t)(item[k] >> 32));
    unsigned long long same = __ballot(real);  // lanes with this lane's digit
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
      const unsigned long long b = __ballot((d >> bit) & 1);
      same &= (d >> bit) & 1 ? b : ~b;
    }
    const int rank = __popcll(same & ((1ull << lane) - 1ull));
    int32_t at = 0;
    if (real) at = next[v][d] + rank;
    wave_sync();
    if (real && rank == 0) next[v][d] += __popcll(same);
    wave_sync();
    if (real) {
      if (PASS == 0) out[at] = item[k];
      else perm[at] = (int32_t)(uint32_t)item[k];
    }
  }
}

// One workgroup per window: its rows of 65,280 entries or more, which stand in
// front in the order of their low byte, by the bytes above it, one stable counting
// pass each (the longest row says how many). A pass counts the digits, then takes
// the rows kSortBlock at a time: a row's place is its digit's, plus the rows of the
// digit in the turns and waves before, plus its rank in its wave. Linear in their
// number, which is no small one where rows are dense: 1,000 take 5 us, 8,000 take 26
// and 20,000 take 63 (before, each was counted against every other: 256,000 steps of
// two dependent loads a thread for 8,000). Nothing to do where the row pointers are
// malformed: any length may stand there, and no order is needed. tmp: n int32.
__global__ void __launch_bounds__(kSortBlock) k_sort_longest(const int32_t *__restrict__ len,
                                                             const uint32_t *__restrict__ flags,
                                                             const int32_t *__restrict__ maxlen, int64_t sigma,
                                                             int64_t per_window, const int64_t *__restrict__ places,
                                                             int32_t *tmp, int32_t *perm) {
  constexpr int WAVES = kSortBlock / 64;
  __shared__ int32_t place[256];  // where the next row of each digit goes
  __shared__ int32_t next[WAVES][256];
  const int64_t w0 = (int64_t)blockIdx.x * sigma;
  const int64_t m = places[((int64_t)blockIdx.x * 256 + 1) * per_window] - w0;  // rows of digit 0
  if (m <= 1 || *flags != 0) return;  // uniform over the block
  const int lane = lane_id(), v = threadIdx.x >> 6;
  const int32_t longest = *maxlen;
  int32_t *in = perm + w0, *out = tmp + w0;
  for (int shift = 8; shift < 32 && longest >> shift != 0; shift += 8) {
    if (threadIdx.x < 256) place[threadIdx.x] = 0;
    __syncthreads();
    for (int64_t e = threadIdx.x; e < m; e += kSortBlock) atomicAdd(&place[255 - ((len[in[e]] >> shift) & 255)], 1);
    __syncthreads();
    if (v == 0) {  // exclusive prefix, four digits a lane
      int32_t c[4], sum = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        c[k] = place[4 * lane + k];
        sum += c[k];
      }
      int32_t at = sum;
      for (int off = 1; off < 64; off <<= 1) {
        const int32_t o = __shfl_up(at, off);
        if (lane >= off) at += o;
      }
      at -= sum;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        place[4 * lane + k] = at;
        at += c[k];
      }
    }
    for (int64_t t0 = 0; t0 < m; t0 += kSortBlock) {
      const bool real = t0 + threadIdx.x < m;
      const int32_t row = real ? in[t0 + threadIdx.x] : 0;
      const int d = real ? 255 - ((len[row] >> shift) & 255) : 0;
      for (int q = lane; q < 256; q += 64) next[v][q] = 0;
      unsigned long long same = __ballot(real);  // lanes with this lane's digit
#pragma unroll
      for (int bit = 0; bit < 8; ++bit) {
        const unsigned long long b = __ballot((d >> bit) & 1);
        same &= (d >> bit) & 1 ? b : ~b;
      }
      const int rank = __popcll(same & ((1ull << lane) - 1ull));
      wave_sync();
      if (real && rank == 0) next[v][d] = __popcll(same);
      __syncthreads();
      if (threadIdx.x < 256) {
        int32_t at = place[threadIdx.x];
#pragma unroll
        for (int u = 0; u < WAVES; ++u) {
          const int32_t c = next[u][threadIdx.x];
          next[u][threadIdx.x] = at;
          at += c;
        }
        place[threadIdx.x] = at;
      }
      __syncthreads();
      if (real) out[next[v][d] + rank] = row;
      wave_sync();
    }
    __syncthreads();
    int32_t *const t = in;
    in = out;
    out = t;
  }
  if (in != perm + w0)
    for (int64_t e = threadIdx.x; e < m; e += kSortBlock) perm[w0 + e] = in[e];
}

// Chunks up to this width are never split: their few[] is not looked at.
constexpr int32_t kFewMin = 32;

// cl[i] = max length of the chunk's rows in sorted order (Eq. (max));
// csz[i] = C * cl[i] (scanned into cs afterwards); csz[nchunks] = 0. One lane
// per row, so that the permuted lengths of a chunk are one access (one thread
// per chunk took its C accesses in turn: 22 us on 1M rows; now 17.6, few[] found as
// well), a fixed grid striding over the rows, so that the sums cost one atomic per
// block.
__global__ void __launch_bounds__(kStrideBlock) k_chunkwidth(const int32_t *__restrict__ len,
                                                       const int32_t *__restrict__ perm, int64_t n, int C,
                                                       int64_t nchunks, int T, int wpc, int32_t *__restrict__ cl,
                                                       int64_t *__restrict__ csz,
                                                       unsigned long long *__restrict__ padded,
                                                       unsigned long long *__restrict__ total_steps,
                                                       int32_t *__restrict__ max_width,
                                                       int32_t *__restrict__ few) {
  __shared__ unsigned long long s_cols[kStrideBlock / 64];
  __shared__ unsigned long long s_steps[kStrideBlock / 64];
  __shared__ int32_t s_mx[kStrideBlock / 64];
  const int span = C < 64 ? 64 : C;  // rows of a wave's turn: whole chunks
  const int lane = lane_id(), width = C < 64 ? C : 64;
  const int64_t rows = nchunks * C, stride = (int64_t)gridDim.x * (kStrideBlock / 64) * span;
  unsigned long long steps = 0, cols = 0;
  int32_t mx = 0;
  const int nfew = thin_rows(width, T);
  for (int64_t p0 = ((int64_t)blockIdx.x * (kStrideBlock / 64) + (threadIdx.x >> 6)) * span; p0 < rows; p0 += stride) {
    int32_t l = 0;
    for (int64_t p = p0 + lane; p < p0 + span; p += 64) {
      const int32_t v = p < n ? len[perm ? (int64_t)perm[p] : p] : 0;
      if (few && nfew > 0) {
        // the longest row of each item taken out nfew times, then the longest
        // left; kFewMin where all of the wave's rows are that short (half of a
        // wide chunk at C = 128 may be)
        int32_t f = kFewMin, f2 = kFewMin;
        if (__ballot(v > kFewMin) != 0ull) {
          int64_t key = (int64_t)v << 6 | lane;
          for (int t = 0;; ++t) {
            int64_t m = key;
            for (int off = width / 2; off > 0; off >>= 1) {
              const int64_t o = __shfl_xor(m, off);
              m = o > m ? o : m;
            }
            f = (int32_t)(m >> 6);
            if (t == kThinnestRows) f2 = f;
            if (t == nfew) break;
            if (m == key) key = -64;
          }
        }
        if (lane % width == 0 && p < rows) {
          few[2 * (p / width)] = f;
          few[2 * (p / width) + 1] = f2;
        }
      }
      l = v > l ? v : l;
    }
    for (int off = width / 2; off > 0; off >>= 1) {
      const int32_t o = __shfl_xor(l, off);
      l = o > l ? o : l;
    }
    const int64_t i = (p0 + lane) / C;
    if (lane % width == 0 && i < nchunks && p0 + lane < p0 + span) {
      cl[i] = l;
      csz[i] = (int64_t)C * l;
      steps += (unsigned long long)(((int64_t)l + T - 1) / T) * wpc;
      cols += (unsigned long long)l;
      mx = l > mx ? l : mx;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) csz[nchunks] = 0;
  steps = wave_sum_u64(steps);
  cols = wave_sum_u64(cols);
  mx = wave_max(mx);
  if (lane == 0) {
    s_steps[threadIdx.x >> 6] = steps;
    s_cols[threadIdx.x >> 6] = cols;
    s_mx[threadIdx.x >> 6] = mx;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kStrideBlock / 64; ++w) {
      steps += s_steps[w];
      cols += s_cols[w];
      mx = s_mx[w] > mx ? s_mx[w] : mx;
    }
    if (steps) {
      atomicAdd(total_steps, steps);
      atomicAdd(padded, cols * (unsigned long long)C);
    }
    if (mx) atomicMax(max_width, mx);
  }
}

// ---------------------------------------------------------------------------
// Exclusive prefix sum of int64 values: per-block scan of kScanItems
// elements, recursive scan of the block totals, then add the block offsets.
// ---------------------------------------------------------------------------
constexpr int kScanBlock = 256;
constexpr int kScanPer = 4;
constexpr int kScanItems = kScanBlock * kScanPer;

__global__ void __launch_bounds__(kScanBlock) k_scan_block(const int64_t *__restrict__ in, int64_t *__restrict__ out,
                                                           int64_t n, int64_t *__restrict__ totals) {
  __shared__ int64_t wsum[kScanBlock / 64];
  int64_t base = (int64_t)blockIdx.x * kScanItems + (int64_t)threadIdx.x * kScanPer;
  int64_t v[kScanPer];
  int64_t run = 0;
#pragma unroll
  for (int e = 0; e < kScanPer; ++e) {
    int64_t idx = base + e;
    v[e] = idx < n ? in[idx] : 0;
    run += v[e];
  }
  // inclusive scan of the thread totals across the wave
  int lane = lane_id(), wid = threadIdx.x >> 6;
  int64_t incl = run;
  for (int off = 1; off < 64; off <<= 1) {
    int64_t o = __shfl_up(incl, off);
    if (lane >= off) incl += o;
  }
  if (lane == 63) wsum[wid] = incl;
  __syncthreads();
  int64_t wbase = 0;
  for (int w = 0; w < wid; ++w) wbase += wsum[w];
  int64_t excl = wbase + incl - run;
#pragma unroll
  for (int e = 0; e < kScanPer; ++e) {
    int64_t idx = base + e;
    if (idx < n) out[idx] = excl;
    excl += v[e];
  }
  if (threadIdx.x == kScanBlock - 1) {
    int64_t tot = 0;
    for (int w = 0; w < kScanBlock / 64; ++w) tot += wsum[w];
    totals[blockIdx.x] = tot;
  }
}

__global__ void __launch_bounds__(kScanBlock) k_scan_add(int64_t *__restrict__ out, int64_t n,
                                                         const int64_t *__restrict__ offs) {
  int64_t base = (int64_t)blockIdx.x * kScanItems;
  int64_t add = offs[blockIdx.x];
  for (int e = threadIdx.x; e < kScanItems; e += kScanBlock) {
    int64_t idx = base + e;
    if (idx < n) out[idx] += add;
  }
}

// ---------------------------------------------------------------------------
// Fill: slot s of the padded arrays belongs to chunk i with cs[i] <= s <
// cs[i+1]; inside it, column j = (s - cs[i]) / C and lane r = (s - cs[i]) % C
// (the layout val[cs[i] + j*C + r]). The slot receives entry j of row
// perm[i*C + r] in CRS order, or value 0 / column 0 when that row is shorter
// or does not exist.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float f64_to_f32_rne(double d) { return (float)d; }

// Nearest-even rounding of a double to bfloat16 in two steps that cannot
// double-round: round to binary32 with round-to-odd (24 >= 2*8 + 2 bits,
// Boldo and Melquiond, "Emulation of FMA and correctly rounded sums: proved
// algorithms using rounding to odd", IEEE TC 2008), then round that binary32
// to bfloat16 nearest-even on its bit pattern.
__device__ __forceinline__ uint16_t f64_to_bf16_rne(double d) {
  float f = (float)d;
  uint32_t b = __float_as_uint(f);
  double back = (double)f;
  if (back != d && !(d != d)) {
    if (fabs(back) > fabs(d)) b -= 1;  // step toward zero: the truncated value
    b |= 1u;                           // odd last bit marks the inexact result
  }
  if ((b & 0x7f800000u) == 0x7f800000u && (b & 0x007fffffu)) return (uint16_t)((b >> 16) | 0x40u);  // NaN
  uint32_t lsb = (b >> 16) & 1u;
  b += 0x7fffu + lsb;
  return (uint16_t)(b >> 16);
}

template <int VD>
__device__ __forceinline__ void st_val(void *sval, int64_t s, double v) {
  if (VD == SELL_F64) static_cast<double *>(sval)[s] = v;
  else if (VD == SELL_F32) static_cast<float *>(sval)[s] = f64_to_f32_rne(v);
  else static_cast<uint16_t *>(sval)[s] = f64_to_bf16_rne(v);
}

// Last i in [lo, hi) with cs[i] <= s (cs[lo] <= s).
__device__ __forceinline__ int64_t chunk_of(const int64_t *__restrict__ cs, int64_t lo, int64_t hi, int64_t s) {
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (cs[mid] <= s) lo = mid;
    else hi = mid;
  }
  return lo;
}

// One wave per 2^rc <= 64 chunk columns (every chunk starts and ends at a column,
// so no column is cut). The chunks of the range are searched once per
// wave, uniformly. Up to kFillPieces chunks: one after another in tiles of
// kFillTile slots, which are read along the rows (8 rows by 8 entries an
// access, 16 accesses in flight) and turned in LDS. More (short chunks): lane c
// finds the chunk and the place in it of column c, and the slots read theirs
// from that lane, so that the pointer chains of U steps overlap whatever chunks
// they lie in. Wide chunks are bound by memory: 27-point stencil 128^3 in FP64
// (1.34 GB moved) 1,027 us with one slot per thread and a search of its own,
// 508 read down the columns, now 308 (4.4 TB/s; a copy moves 4.9). Short ones by
// the lines that scattered rows fetch: power-law 1M, sigma = n, 79 -> 60 us
// (16 instead of 64 columns per wave: 65).
constexpr int kFillPieces = 8;
constexpr int kFillTile = 1024;

template <int VD, bool TILES>
__global__ void __launch_bounds__(kBlock) k_fill(const int64_t *__restrict__ rpt, const int32_t *__restrict__ col,
                                                 const double *__restrict__ val, int64_t n, int C, int lc, int rc,
                                                 const int32_t *__restrict__ perm, const int64_t *__restrict__ cs,
                                                 int64_t nchunks, int64_t padded, const int32_t *__restrict__ cmap,
                                                 int32_t *__restrict__ scol, void *__restrict__ sval) {
  constexpr int U = 8;
  __shared__ double tile_v[kBlock / 64][TILES ? kFillTile : 1];
  __shared__ int32_t tile_c[kBlock / 64][TILES ? kFillTile : 64];
  const int lane = lane_id();
  double *tv = tile_v[threadIdx.x >> 6];
  int32_t *tc = tile_c[threadIdx.x >> 6];
  // a tile is read 1 << lr rows at a time, 64 >> lr entries of each, 1 << lj
  // times over; column j of it lies rotated by j << lr rows in LDS, so that
  // the lanes of such a read fall on all banks
  constexpr int lr = 3;
  const int lj = 7 - lc > 0 ? 7 - lc : 0;
  const int64_t w = (int64_t)blockIdx.x * (kBlock / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t s0 = w << (rc + lc), range = (int64_t)1 << (rc + lc);
  if (s0 >= padded) return;  // uniform over the wave; no barrier below
  const int64_t s1 = s0 + range < padded ? s0 + range : padded;
  const int64_t i0 = chunk_of(cs, 0, nchunks, s0);
  int64_t step = 1;
  while (i0 + step < nchunks && cs[i0 + step] < s1) step <<= 1;
  const int64_t i1 = chunk_of(cs, i0, i0 + step < nchunks ? i0 + step : nchunks, s1 - 1);  // last chunk of the range

  if (TILES && i1 - i0 < kFillPieces) {
    for (int64_t i = i0; i <= i1; ++i) {
      const int64_t b = cs[i], e = cs[i + 1];
      const int64_t sb = b > s0 ? b : s0, se = e < s1 ? e : s1;
      // lane r keeps where row r (and r + 64 at C = 128) starts and ends
      int64_t src[2] = {0, 0}, end[2] = {0, 0};
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int64_t p = (i << lc) + h * 64 + lane;
        if (h * 64 + lane < C && p < n) {
          const int64_t row = perm ? perm[p] : p;
          src[h] = rpt[row];
          end[h] = rpt[row + 1];
        }
      }
      for (int64_t st = sb; st < se; st += kFillTile) {  // tiles of whole columns
        const int64_t jt = (st - b) >> lc;
        const int slots = se - st < kFillTile ? (int)(se - st) : kFillTile;
        int32_t c[kFillTile / 64];
        double v[kFillTile / 64];
#pragma unroll
        for (int it = 0; it < kFillTile / 64; ++it) {
          const int r = ((it >> lj) << lr) + (lane >> (6 - lr));  // row
          const int j = ((it & ((1 << lj) - 1)) << (6 - lr)) + (lane & ((64 >> lr) - 1));
          int64_t q = __shfl(src[0], r & 63), e = __shfl(end[0], r & 63);
          if (C > 64 && r >= 64) {  // uniform over the wave
            q = __shfl(src[1], r & 63);
            e = __shfl(end[1], r & 63);
          }
          q += jt + j;
          c[it] = 0;
          v[it] = 0.0;
          if ((j << lc) < slots && q < e) {
            c[it] = col[q];
            v[it] = val[q];
            if (cmap) c[it] = cmap[c[it]];
          }
        }
        wave_sync();
#pragma unroll
        for (int it = 0; it < kFillTile / 64; ++it) {
          const int r = ((it >> lj) << lr) + (lane >> (6 - lr));
          const int j = ((it & ((1 << lj) - 1)) << (6 - lr)) + (lane & ((64 >> lr) - 1));
          const int at = (j << lc) + ((r + (j << lr)) & (C - 1));
          tv[at] = v[it];
          tc[at] = c[it];
        }
        wave_sync();
#pragma unroll 4
        for (int o = lane; o < slots; o += 64) {
          const int j = o >> lc;
          const int at = (j << lc) + (((o & (C - 1)) + (j << lr)) & (C - 1));
          scol[st + o] = tc[at];
          st_val<VD>(sval, st + o, tv[at]);
        }
      }
    }
    return;
  }

  // chunk (less i0) of column `lane` of the range, and the column's place in it
  int32_t *mark = tc;
  mark[lane] = 0;
  wave_sync();
  for (int64_t i = i0 + 1 + lane; i <= i1; i += 64) {
    const int64_t b = cs[i];
    if (cs[i + 1] > b) mark[(b - s0) >> lc] = (int32_t)(i - i0);  // empty chunks hold no column
  }
  wave_sync();
  int32_t ci = mark[lane];
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int32_t o = __shfl_up(ci, off);
    if (lane >= off && o > ci) ci = o;
  }
  int64_t j0 = 0;
  if (s0 + ((int64_t)lane << lc) < s1) j0 = (s0 + ((int64_t)lane << lc) - cs[i0 + ci]) >> lc;
  for (int64_t s = s0 + lane; s - lane < s1; s += 64 * U) {
    int64_t q[U], e[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t at = s + 64 * u;
      const int c = (int)((at - s0) >> lc) & 63;
      const int64_t p = ((i0 + __shfl(ci, c)) << lc) + (at & (C - 1));
      const int64_t j = __shfl(j0, c);
      q[u] = e[u] = 0;
      if (at < s1 && p < n) {
        const int64_t row = perm ? perm[p] : p;
        q[u] = rpt[row] + j;
        e[u] = rpt[row + 1];
      }
    }
    int32_t c[U];
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      c[u] = 0;
      v[u] = 0.0;
      if (q[u] < e[u]) {
        c[u] = col[q[u]];
        v[u] = val[q[u]];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t at = s + 64 * u;
      if (at >= s1) continue;
      scol[at] = cmap && q[u] < e[u] ? cmap[c[u]] : c[u];
      st_val<VD>(sval, at, v[u]);
    }
  }
}

// iperm[perm[p]] = p
__global__ void __launch_bounds__(kBlock) k_invert(const int32_t *__restrict__ perm, int64_t n,
                                                   int32_t *__restrict__ iperm) {
  int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (p < n) iperm[perm[p]] = (int32_t)p;
}

// rl[p] = len[perm[p]]: the length of the row in sorted position p, 0 for
// the rows that pad the last chunk (p in [n, np))
__global__ void __launch_bounds__(kBlock) k_sorted_len(const int32_t *__restrict__ len,
                                                       const int32_t *__restrict__ perm, int64_t n, int64_t np,
                                                       int32_t *__restrict__ rl) {
  int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (p < np) rl[p] = p < n ? len[perm ? (int64_t)perm[p] : p] : 0;
}

// One wave per unit: a thin segment's slots in the order that the product's lanes
// take them -- of step t, lane l: column jb + t * (64 / L) + l / L of the (l % L)-th
// row, L the number of rows raised to a power of two; zeros past the rows and the
// columns.
template <typename E>
__global__ void __launch_bounds__(kBlock) k_thin(const Unit1 *__restrict__ units, int64_t nunits, int C,
                                                 const int64_t *__restrict__ cs, const int32_t *__restrict__ col,
                                                 const E *__restrict__ val, int64_t slots, int32_t *__restrict__ tcol,
                                                 E *__restrict__ tval) {
  const int64_t w = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  if (w >= nunits) return;
  const Unit1 u = units[w];
  if (u.rows == 0) return;
  const ThinLane t = thin_lane(u.rows, lane_id());
  const int wpc = C > 64 ? C / 64 : 1, rpw = C < 64 ? C : 64;
  const int64_t chunk = u.item / wpc, off = cs[chunk] + (u.item - chunk * wpc) * rpw;
  int64_t o = u.thin * slots + lane_id();
  for (int32_t j0 = u.jb; j0 < u.je; j0 += t.step, o += 64) {
    const int32_t j = j0 + t.col;
    const bool ok = t.row >= 0 && j < u.je;
    tcol[o] = ok ? col[off + (int64_t)j * C + t.row] : 0;
    tval[o] = ok ? val[off + (int64_t)j * C + t.row] : E{};
  }
}

// out[p] = in[perm[p]] (gather into sorted order) or out[perm[p]] = in[p]
// (scatter back), for elements of ES bytes.
template <typename E, bool SCATTER>
__global__ void __launch_bounds__(kBlock) k_permute(const E *__restrict__ in, E *__restrict__ out,
                                                    const int32_t *__restrict__ perm, int64_t n) {
  int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (p >= n) return;
  const int64_t q = perm ? (int64_t)perm[p] : p;
  if (SCATTER) out[q] = in[p];
  else out[p] = in[q];
}

inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

hipError_t build_sorted_len(const int32_t *len, const int32_t *perm, int64_t n, int64_t np, int32_t *rl,
                            hipStream_t s) {
  if (np <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_sorted_len, dim3(blocks_for(np, kBlock)), dim3(kBlock), 0, s, len, perm, n, np, rl);
  return hipGetLastError();
}

hipError_t build_thin(const Unit1 *units, int64_t nunits, int C, const int64_t *cs, const int32_t *col, const void *val,
                      int esize, int64_t slots, int32_t *tcol, void *tval, hipStream_t s) {
  if (nunits <= 0) return hipSuccess;
  const dim3 nb(blocks_for(nunits, kBlock / 64));
#define SELL_L(SS, EE)                                                                                      \
  if (esize == SS)                                                                                         \
    hipLaunchKernelGGL(k_thin<EE>, nb, dim3(kBlock), 0, s, units, nunits, C, cs, col,                       \
                       static_cast<const EE *>(val), slots, tcol, static_cast<EE *>(tval));
  SELL_L(8, uint64_t) SELL_L(4, uint32_t) SELL_L(2, uint16_t)
#undef SELL_L
  return hipGetLastError();
}

hipError_t build_invert(const int32_t *perm, int64_t n, int32_t *iperm, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_invert, dim3(blocks_for(n, kBlock)), dim3(kBlock), 0, s, perm, n, iperm);
  return hipGetLastError();
}

hipError_t permute_vector(const void *in, void *out, const int32_t *perm, int64_t n, int elem_bytes, bool scatter,
                          hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const unsigned nb = blocks_for(n, kBlock);
  if (elem_bytes == 8) {
    if (scatter)
      hipLaunchKernelGGL((k_permute<uint64_t, true>), dim3(nb), dim3(kBlock), 0, s, static_cast<const uint64_t *>(in),
                         static_cast<uint64_t *>(out), perm, n);
    else
      hipLaunchKernelGGL((k_permute<uint64_t, false>), dim3(nb), dim3(kBlock), 0, s,
                         static_cast<const uint64_t *>(in), static_cast<uint64_t *>(out), perm, n);
  } else {
    if (scatter)
      hipLaunchKernelGGL((k_permute<uint32_t, true>), dim3(nb), dim3(kBlock), 0, s, static_cast<const uint32_t *>(in),
                         static_cast<uint32_t *>(out), perm, n);
    else
      hipLaunchKernelGGL((k_permute<uint32_t, false>), dim3(nb), dim3(kBlock), 0, s,
                         static_cast<const uint32_t *>(in), static_cast<uint32_t *>(out), perm, n);
  }
  return hipGetLastError();
}

hipError_t build_rowlen(const int64_t *rpt, int64_t n, int64_t nnz, int32_t *len, uint32_t *flags,
                        unsigned long long *sumsq, int32_t *maxlen, hipStream_t s) {
  unsigned nb = blocks_for(n > 0 ? n : 1, kStrideBlock);
  if (nb > kStrideGrid) nb = kStrideGrid;
  hipLaunchKernelGGL(k_rowlen, dim3(nb), dim3(kStrideBlock), 0, s, rpt, n, nnz, len, flags, sumsq, maxlen);
  return hipGetLastError();
}

hipError_t build_colcheck(const int32_t *col, int64_t nnz, int64_t ncols, uint32_t *flags, hipStream_t s) {
  if (nnz <= 0) return hipSuccess;
  int64_t nb = blocks_for((nnz + 15) / 16, kBlock);
  if (nb > 4096) nb = 4096;
  hipLaunchKernelGGL(k_colcheck, dim3((unsigned)nb), dim3(kBlock), 0, s, col, nnz, ncols, flags);
  return hipGetLastError();
}

int64_t sort_tmp_elems(int64_t n, int64_t sigma) {
  if (sigma > n) sigma = n;
  if (sigma <= kTile) return 0;
  const int64_t counts = (n + sigma - 1) / sigma * ((sigma + kTile - 1) / kTile) * 256;
  return n + counts + scan_tmp_elems(counts);
}

hipError_t build_sort(const int32_t *len, const uint32_t *flags, const int32_t *maxlen, int64_t n, int64_t sigma,
                      int64_t *tmp, int32_t *perm, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (sigma > n) sigma = n;
  if (sigma <= kTile) {
    const int64_t tile_rows = (kTile / sigma) * sigma;
    hipLaunchKernelGGL(k_sort_tiles, dim3(blocks_for(n, (int)tile_rows)), dim3(kSortBlock), 0, s, len, n, sigma, perm);
    return hipGetLastError();
  }
  const int64_t nwin = (n + sigma - 1) / sigma, per = (sigma + kTile - 1) / kTile, ncounts = nwin * per * 256;
  uint64_t *items = reinterpret_cast<uint64_t *>(tmp);
  int64_t *counts = tmp + n, *stmp = counts + ncounts;
  const dim3 tiles((unsigned)(nwin * per));
  hipError_t e;
  hipLaunchKernelGGL(k_sort_count<0>, tiles, dim3(kSortBlock), 0, s, len, items, n, sigma, per, counts);
  if ((e = hipGetLastError()) != hipSuccess || (e = build_scan(counts, counts, ncounts, stmp, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_sort_place<0>, tiles, dim3(kSortBlock), 0, s, len, nullptr, n, sigma, per, counts, items, perm);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_sort_count<1>, tiles, dim3(kSortBlock), 0, s, len, items, n, sigma, per, counts);
  if ((e = hipGetLastError()) != hipSuccess || (e = build_scan(counts, counts, ncounts, stmp, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_sort_place<1>, tiles, dim3(kSortBlock), 0, s, len, items, n, sigma, per, counts, nullptr, perm);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_sort_longest, dim3((unsigned)nwin), dim3(kSortBlock), 0, s, len, flags, maxlen, sigma, per, counts,
                     reinterpret_cast<int32_t *>(items), perm);
  return hipGetLastError();
}

hipError_t build_chunkwidth(const int32_t *len, const int32_t *perm, int64_t n, int C, int64_t nchunks, int T, int wpc,
                            int32_t *cl, int64_t *csz, int64_t *padded, int64_t *total_steps, int32_t *max_width,
                            int32_t *few, hipStream_t s) {
  const int64_t per = (int64_t)(kStrideBlock / 64) * (C < 64 ? 64 : C);
  int64_t nb = (nchunks * C + per - 1) / per;
  nb = nb < 1 ? 1 : nb > kStrideGrid ? kStrideGrid : nb;
  hipLaunchKernelGGL(k_chunkwidth, dim3((unsigned)nb), dim3(kStrideBlock), 0, s, len, perm, n, C, nchunks, T, wpc, cl, csz,
                     reinterpret_cast<unsigned long long *>(padded),
                     reinterpret_cast<unsigned long long *>(total_steps), max_width, few);
  return hipGetLastError();
}

int64_t scan_tmp_elems(int64_t n) {
  int64_t total = 0;
  while (n > kScanItems) {
    int64_t nb = (n + kScanItems - 1) / kScanItems;
    total += nb;
    n = nb;
  }
  return total + 1;
}

hipError_t build_scan(const int64_t *in, int64_t *out, int64_t n, int64_t *tmp, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t nb = (n + kScanItems - 1) / kScanItems;
  hipLaunchKernelGGL(k_scan_block, dim3((unsigned)nb), dim3(kScanBlock), 0, s, in, out, n, tmp);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || nb == 1) return e;
  // scan the block totals (in place), then add them
  e = build_scan(tmp, tmp, nb, tmp + nb, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_scan_add, dim3((unsigned)nb), dim3(kScanBlock), 0, s, out, n, tmp);
  return hipGetLastError();
}

hipError_t build_fill(const int64_t *rpt, const int32_t *col, const double *val, int64_t n, int C,
                      const int32_t *perm, const int64_t *cs, int64_t nchunks, int64_t padded, const int32_t *cmap,
                      int32_t *scol, void *sval, int val_dtype, hipStream_t s) {
  if (padded <= 0) return hipSuccess;
  const int lc = __builtin_ctz((unsigned)C);
  // small matrices: fewer columns a wave, slots on their own (50,000 rows of up
  // to 20 entries: 32 us with 64 columns in tiles, 21 with the tiles unused but
  // their LDS taken, 11 so). C < 8: a wave's columns are fewer slots than a tile
  // holds, and its chunks, one after another, leave most of the reads' lanes idle
  // (build of the 27-point stencil 100^3, C = 1, 2, 4: 2,610, 1,398, 817 us with
  // tiles, 606, 400, 298 without)
  int rc = 6;
  const bool tiles = lc >= 3 && padded >> (rc + lc) >= 2048;
  while (!tiles && rc > 1 && padded >> (rc + lc) < 8192) --rc;
  const int64_t waves = (padded + ((int64_t)1 << (rc + lc)) - 1) >> (rc + lc);
  const dim3 nb(blocks_for(waves, kBlock / 64));
#define SELL_L(VD, TT)                                                                                            \
  if (val_dtype == VD && tiles == TT)                                                                            \
    hipLaunchKernelGGL((k_fill<VD, TT>), nb, dim3(kBlock), 0, s, rpt, col, val, n, C, lc, rc, perm, cs, nchunks, \
                       padded, cmap, scol, sval);
  SELL_L(SELL_F64, true) SELL_L(SELL_F32, true) SELL_L(SELL_BF16, true)
  SELL_L(SELL_F64, false) SELL_L(SELL_F32, false) SELL_L(SELL_BF16, false)
#undef SELL_L
  return hipGetLastError();
}

}  // namespace sell
