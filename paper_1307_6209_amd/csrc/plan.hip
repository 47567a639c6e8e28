// Work plans of the products on layouts with wide chunks, made on the device
// from the chunk widths. The host learns the counts with the padded size, in
// the one read-back that a construction needs anyway, and launches the rest
// without waiting. (On the host, the widths copied back, the lists filled and
// copied out: 390 us of the 770 that a power-law matrix of 1M rows took.)
//
// Two plans: the block form's (segments of S columns, one unit per other item)
// and the single-vector product's (segments of S1 <= S columns; runs of 64 / C
// chunks at most 64 / C columns wide are one unit, which one wave covers). A
// "cell" is such a run, aligned: 64 / C chunks for C in 8..32, else one.
#include "sell_internal.h"
#include "xcd_place.h"

namespace sell {
namespace {

constexpr int kPlanBlock = 256;

// Split slices, segments and (single plan) whole units of some cells.
struct Counts {
  int32_t split0, seg0, split1, seg1, whole1, thin1;
  __device__ void add(const Counts &o) {
    split0 += o.split0;
    seg0 += o.seg0;
    split1 += o.split1;
    seg1 += o.seg1;
    whole1 += o.whole1;
    thin1 += o.thin1;
  }
};

struct Cell {
  int64_t c0, c1;  // its chunks
  bool group;      // one unit of the single plan
};

__device__ __forceinline__ Cell cell_of(const PlanArgs &a, int64_t cell) {
  Cell r;
  r.c0 = cell * a.grp;
  r.c1 = r.c0 + a.grp < a.nchunks ? r.c0 + a.grp : a.nchunks;
  r.group = a.grp > 1 && r.c1 - r.c0 == a.grp;
  if (r.group)
    for (int64_t c = r.c0; c < r.c1; ++c) r.group = r.group && a.cl[c] <= a.grp;
  return r;
}

__device__ __forceinline__ Split1 split_item(const PlanArgs &a, int64_t it, int32_t w, int32_t S1) {
  return split1_of(a.few ? a.few + 2 * it : nullptr, w, S1, a.seg_cols > 0);
}

__device__ __forceinline__ Counts count_cell(const PlanArgs &a, const Cell &e, int32_t S, int32_t S1) {
  Counts n{};
  for (int64_t c = e.c0; c < e.c1; ++c) {
    const int32_t w = a.cl[c];
    if (w > S) {
      n.split0 += a.wpc;
      n.seg0 += (w + S - 1) / S * a.wpc;
    }
    if (w > S1) {
      n.split1 += a.wpc;
      for (int h = 0; h < a.wpc; ++h) {
        const Split1 sp = split_item(a, c * a.wpc + h, w, S1);
        n.seg1 += sp.all;
        n.thin1 += sp.all - sp.dense;
      }
    } else if (!e.group) {
      n.whole1 += a.wpc;
    }
  }
  if (e.group) n.whole1 = 1;
  return n;
}

__device__ __forceinline__ int32_t wave_incl(int32_t v) {
  for (int off = 1; off < 64; off <<= 1) {
    const int32_t o = __shfl_up(v, off);
    if ((int)(threadIdx.x & 63) >= off) v += o;
  }
  return v;
}

// Exclusive prefix of v over the block; *total gets the sum.
__device__ Counts block_prefix(const Counts &v, Counts *total) {
  __shared__ Counts ws[kPlanBlock / 64];
  Counts i;
  i.split0 = wave_incl(v.split0);
  i.seg0 = wave_incl(v.seg0);
  i.split1 = wave_incl(v.split1);
  i.seg1 = wave_incl(v.seg1);
  i.whole1 = wave_incl(v.whole1);
  i.thin1 = wave_incl(v.thin1);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 63) ws[w] = i;
  __syncthreads();
  Counts before{}, all{};
  for (int q = 0; q < kPlanBlock / 64; ++q) {
    if (q < w) before.add(ws[q]);
    all.add(ws[q]);
  }
  *total = all;
  before.split0 += i.split0 - v.split0;
  before.seg0 += i.seg0 - v.seg0;
  before.split1 += i.split1 - v.split1;
  before.seg1 += i.seg1 - v.seg1;
  before.whole1 += i.whole1 - v.whole1;
  return before;
}

// The widths of the segments; S = S1 = 2^31 - 1 where nothing is split.
__device__ __forceinline__ void seg_widths(const PlanArgs &a, int32_t *S, int32_t *S1) {
  const PlanSizes z = *a.sizes;
  *S = *S1 = 0x7fffffff;
  if (a.seg_cols < 0) return;
  const int32_t s = a.seg_cols > 0 ? a.seg_cols : auto_seg_cols(z.total_steps, a.T, a.cus);
  if (z.max_width <= s) return;
  *S = s;
  *S1 = a.seg_cols > 0 ? s : single_seg_cols(z.total_steps, a.T, a.cus, s);
}

__global__ void __launch_bounds__(kPlanBlock) k_plan_count(PlanArgs a) {
  int32_t S, S1;
  seg_widths(a, &S, &S1);
  const int64_t cell = (int64_t)blockIdx.x * kPlanBlock + threadIdx.x;
  Counts n{}, total;
  if (cell < a.ncells) n = count_cell(a, cell_of(a, cell), S, S1);
  block_prefix(n, &total);
  if (threadIdx.x == 0) {
    // a single block: its prefixes are zero, its counts the totals
    int64_t *b = gridDim.x > 1 ? a.blocks + kPlanCounts * (int64_t)blockIdx.x : &a.sizes->nsplit;
    b[0] = total.split0;
    b[1] = total.seg0;
    b[2] = total.split1;
    b[3] = total.seg1;
    b[4] = total.whole1;
    b[5] = total.thin1;
    if (gridDim.x == 1)
      for (int q = 0; q < kPlanCounts; ++q) a.blocks[q] = 0;
  }
}

// One workgroup: the blocks' counts to their exclusive prefixes (lane l of a
// wave takes block l of 64, wave q quantity q), the totals to *sizes.
__global__ void __launch_bounds__(kPlanCounts * 64) k_plan_scan(PlanArgs a, int64_t nblocks) {
  const int q = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int64_t sum = 0;
  for (int64_t b = 0; b < nblocks; b += 64) {
    int64_t v = b + lane < nblocks ? a.blocks[kPlanCounts * (b + lane) + q] : 0;
    int64_t i = v;
    for (int off = 1; off < 64; off <<= 1) {
      const int64_t o = __shfl_up(i, off);
      if (lane >= off) i += o;
    }
    if (b + lane < nblocks) a.blocks[kPlanCounts * (b + lane) + q] = sum + i - v;
    sum += __shfl(i, 63);
  }
  if (lane == 0) (&a.sizes->nsplit)[q] = sum;
}

// Split slices and whole units of both plans.
__global__ void __launch_bounds__(kPlanBlock) k_plan_emit(PlanArgs a, int32_t S, int32_t S1, int64_t nsegs,
                                                          int64_t nsegs1, PlanOut o) {
  const int64_t cell = (int64_t)blockIdx.x * kPlanBlock + threadIdx.x;
  Counts n{}, total;
  Cell e{0, 0, false};
  if (cell < a.ncells) {
    e = cell_of(a, cell);
    n = count_cell(a, e, S, S1);
  }
  const Counts at = block_prefix(n, &total);
  if (cell >= a.ncells) return;
  const int64_t *b = a.blocks + kPlanCounts * (int64_t)blockIdx.x;
  int64_t split0 = b[0] + at.split0, seg0 = b[1] + at.seg0, split1 = b[2] + at.split1, seg1 = b[3] + at.seg1;
  int64_t whole1 = b[4] + at.whole1;
  if (e.group) o.units1[nsegs1 + whole1++] = {(int32_t)(e.c0 * a.wpc), 0, 0, 0, -1, 0, 0};
  for (int64_t c = e.c0; c < e.c1; ++c) {
    const int32_t w = a.cl[c];
    for (int h = 0; h < a.wpc; ++h) {
      const int32_t item = (int32_t)(c * a.wpc + h);
      if (w > S) {
        const int32_t ns = (w + S - 1) / S;
        o.splits[split0++] = {item, ns, seg0 * a.rpw};
        seg0 += ns;
      } else {
        o.units[nsegs + item - split0] = {item, 0, 1, 0};
      }
      if (w > S1) {
        const int32_t ns = split_item(a, item, w, S1).all;
        o.splits1[split1++] = {item, ns, seg1 * a.rpw};
        seg1 += ns;
      } else if (!e.group) {
        o.units1[nsegs1 + whole1++] = {item, 1, 0, w, -1, 0, 0};
      }
    }
  }
}

// Segment i of the list belongs to the last slice whose sums start at or
// before i * rpw.
__global__ void __launch_bounds__(kPlanBlock) k_plan_segs(const SplitDesc *__restrict__ splits, int64_t nsplit,
                                                          int64_t nsegs, int rpw, Unit *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * kPlanBlock + threadIdx.x;
  if (i >= nsegs) return;
  int64_t lo = 0, hi = nsplit;
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (splits[mid].poff <= i * rpw) lo = mid;
    else hi = mid;
  }
  const SplitDesc d = splits[lo];
  out[i] = {d.item, (int32_t)(i - d.poff / rpw), d.nseg, (int32_t)lo};
}

// The same for the single plan, one wave per segment, with the rows of the thin
// ones.
__global__ void __launch_bounds__(kPlanBlock) k_plan_segs1(PlanArgs a, const SplitDesc *__restrict__ splits,
                                                           int64_t nsplit, int64_t nsegs, int32_t S1,
                                                           Unit1 *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * (kPlanBlock / 64) +
                    __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (i >= nsegs) return;
  int64_t lo = 0, hi = nsplit;
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (splits[mid].poff <= i * a.rpw) lo = mid;
    else hi = mid;
  }
  const SplitDesc d = splits[lo];
  const int32_t q = (int32_t)(i - d.poff / a.rpw), w = a.cl[d.item / a.wpc];
  const Split1 sp = split_item(a, d.item, w, S1);
  Unit1 u{d.item, d.nseg, 0, 0, (int32_t)(i * a.rpw), 0, 0};
  if (q < sp.dense) {
    u.jb = q * S1;
    u.je = u.jb + S1 < sp.thin ? u.jb + S1 : sp.thin;
  } else {
    if (q < sp.segs) {
      u.jb = sp.thin + (q - sp.dense) * sp.tc;
      u.je = u.jb + sp.tc < sp.thinnest ? u.jb + sp.tc : sp.thinnest;
    } else {
      u.jb = sp.thinnest + (q - sp.segs) * sp.uc;
      u.je = u.jb + sp.uc < w ? u.jb + sp.uc : w;
    }
    const int r = threadIdx.x & 63;
    const int64_t p = (int64_t)d.item * a.rpw + r;
    u.rows = __ballot(r < a.rpw && p < a.nrows && a.len[a.perm ? (int64_t)a.perm[p] : p] > u.jb);
  }
  if ((threadIdx.x & 63) == 0) {
    if (u.rows != 0) u.thin = (int32_t)atomicAdd(a.next_thin, 1u);
    out[i] = u;
  }
}

// One wave per split segment: the mean column of its rows at the middle of
// the segment (rows that have ended hold column 0 there and don't count), and
// how many those are.
__global__ void __launch_bounds__(kPlanBlock) k_unit_cols(const Unit1 *__restrict__ units, int64_t n, int rpw, int wpc,
                                                          int C, const int64_t *__restrict__ cs,
                                                          const int32_t *__restrict__ col, UnitCol *__restrict__ out) {
  const int64_t w = (int64_t)blockIdx.x * (kPlanBlock / 64) + (threadIdx.x >> 6);
  if (w >= n) return;
  const Unit1 u = units[w];
  const int64_t chunk = u.item / wpc;
  const int r = threadIdx.x & 63;
  unsigned long long sum = 0;
  if (r < rpw)
    sum = (unsigned long long)col[cs[chunk] + ((int64_t)u.jb + u.je) / 2 * C + (u.item - chunk * wpc) * rpw + r];
  const int cnt = __popcll(__ballot(sum > 0));
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
  if (r == 0) out[w] = {cnt ? (int32_t)(sum / (unsigned)cnt) : 0, cnt};
}

// One workgroup: the n segments of `segs` to their launch places in `out`.
// Where most rows of the segments hold entries, in the order of their columns
// (to kOrderBins bins; inside a bin in any order: a segment's sums have a place
// of their own, so the results do not depend on it), each XCD an eighth of them
// (xcd_place).
constexpr int kOrderBlock = 1024;
constexpr int kOrderBins = 4096;

__global__ void __launch_bounds__(kOrderBlock) k_order_segs(const Unit1 *__restrict__ segs,
                                                            const UnitCol *__restrict__ at, int64_t n, int rpw,
                                                            int64_t ncols, Unit1 *__restrict__ out) {
  __shared__ int32_t bin[kOrderBins];
  __shared__ int32_t ws[kOrderBlock / 64];
  __shared__ unsigned long long live, cols;  // entries (by the middle columns) and columns of all segments
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  for (int b = tid; b < kOrderBins; b += kOrderBlock) bin[b] = 0;
  if (tid == 0) live = cols = 0;
  __syncthreads();
  unsigned long long mine = 0, width = 0;
  for (int64_t i = tid; i < n; i += kOrderBlock) {
    const UnitCol u = at[i];
    const unsigned w = (unsigned)(segs[i].je - segs[i].jb);
    mine += (unsigned long long)u.live * w;
    width += w;
    atomicAdd(&bin[(int64_t)u.col * kOrderBins / ncols], 1);
  }
  if (mine) atomicAdd(&live, mine);
  if (width) atomicAdd(&cols, width);
  __syncthreads();
  if ((double)live < kXcdMinLive * (double)rpw * (double)cols) {  // uniform
    for (int64_t i = tid; i < n; i += kOrderBlock) out[i] = segs[i];
    return;
  }
  // exclusive prefix of the bins
  constexpr int P = kOrderBins / kOrderBlock;
  int32_t v[P], sum = 0;
  for (int k = 0; k < P; ++k) {
    v[k] = bin[tid * P + k];
    sum += v[k];
  }
  const int32_t incl = wave_incl(sum);
  if (lane == 63) ws[wid] = incl;
  __syncthreads();
  int32_t before = incl - sum;
  for (int w = 0; w < wid; ++w) before += ws[w];
  for (int k = 0; k < P; ++k) {
    bin[tid * P + k] = before;
    before += v[k];
  }
  __syncthreads();
  for (int64_t i = tid; i < n; i += kOrderBlock) {
    const int64_t k = atomicAdd(&bin[(int64_t)at[i].col * kOrderBins / ncols], 1);
    out[xcd_place(k, n, kWavesPerBlock, kXcds)] = segs[i];
  }
}

inline dim3 grid(int64_t n) { return dim3((unsigned)((n + kPlanBlock - 1) / kPlanBlock)); }

}  // namespace

int64_t plan_blocks(int64_t ncells) { return (ncells + kPlanBlock - 1) / kPlanBlock; }

hipError_t plan_count(const PlanArgs &a, hipStream_t s) {
  if (a.ncells <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_plan_count, grid(a.ncells), dim3(kPlanBlock), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || plan_blocks(a.ncells) == 1) return e;
  hipLaunchKernelGGL(k_plan_scan, dim3(1), dim3(kPlanCounts * 64), 0, s, a, plan_blocks(a.ncells));
  return hipGetLastError();
}

hipError_t plan_emit(const PlanArgs &a, int32_t S, int32_t S1, const PlanSizes &z, const PlanOut &o, hipStream_t s) {
  hipLaunchKernelGGL(k_plan_emit, grid(a.ncells), dim3(kPlanBlock), 0, s, a, S, S1, z.nsegs, z.nsegs1, o);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_plan_segs, grid(z.nsegs), dim3(kPlanBlock), 0, s, o.splits, z.nsplit, z.nsegs, a.rpw, o.units);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // o.segs: the single plan's segments are placed by column from there
  hipLaunchKernelGGL(k_plan_segs1, dim3((unsigned)((z.nsegs1 + kPlanBlock / 64 - 1) / (kPlanBlock / 64))),
                     dim3(kPlanBlock), 0, s, a, o.splits1, z.nsplit1, z.nsegs1, S1, o.segs ? o.segs : o.units1);
  return hipGetLastError();
}

hipError_t plan_place(const PlanArgs &a, int C, const PlanSizes &z, const PlanOut &o, const int64_t *cs,
                      const int32_t *col, int64_t ncols, UnitCol *at, hipStream_t s) {
  hipLaunchKernelGGL(k_unit_cols, dim3((unsigned)((z.nsegs1 + kPlanBlock / 64 - 1) / (kPlanBlock / 64))),
                     dim3(kPlanBlock), 0, s, o.segs, z.nsegs1, a.rpw, a.wpc, C, cs, col, at);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_order_segs, dim3(1), dim3(kOrderBlock), 0, s, o.segs, at, z.nsegs1, a.rpw, ncols, o.units1);
  return hipGetLastError();
}

}  // namespace sell
