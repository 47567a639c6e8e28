// Internal declarations shared by the host orchestration and the kernels of
// the SELL-C-sigma library (gfx950). Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <string>
#include <vector>

#include "block_rule.h"
#include "sellcs.h"
#include "store_rule.h"

namespace sell {

// One work unit of an spMVM launch: a row slice ("item") of a chunk and the
// range of chunk columns it covers. Items are (chunk, half) pairs: a chunk of
// C <= 64 rows is one item; C = 128 is two items of 64 rows. A unit with
// nseg == 1 covers the whole item and writes y directly; otherwise it is
// segment seg of nseg of split slice sid, and it stores its row sums for the
// combining kernel.
struct Unit {
  int32_t item;
  int32_t seg;
  int32_t nseg;
  int32_t sid;
};

// A row slice whose chunk is split: its nseg segments stored their row sums
// at partial[poff + seg*rpw + r] (block form: see k_spmmv); a second kernel
// adds them in segment order.
struct SplitDesc {
  int32_t item;
  int32_t nseg;
  int64_t poff;
};

// One work unit of the single-vector product on a layout with split chunks:
// columns [jb, je) of an item. nseg 0: a group of short chunks from item on;
// part < 0: the whole item, y is written; else a segment, whose row sums go to
// partial[part ...]. rows: the rows that a thin segment holds, at most eight
// (bit r: row r of the item); 0: all. thin: its number among the thin segments
// (its copy of its slots).
struct Unit1 {
  int32_t item;
  int32_t nseg;
  int32_t jb, je;
  int32_t part;
  int32_t thin;
  uint64_t rows;
};

// Of a split segment, at its middle column: the mean column of the rows that
// hold an entry there, and their number.
struct UnitCol {
  int32_t col;
  int32_t live;
};

// Work unit of the batched kernel (mat < 0: an empty unit that only fills the
// grid): columns [jb, je) of a row slice whose chunk starts at slot off, its sums
// to y (part < 0) or to partial[part ...]; jb < 0: a group of short chunks from
// item on, the width of its q-th chunk in bits 4q of je. With all of it here a
// wave goes from its unit to the slots, not over the chunk's width and start (64
// power-law matrices, sigma = 200, before thin segments: 327 us so, 319 from the
// unit; sigma = n: the same).
struct BUnit {
  int32_t mat;
  int32_t item;
  int32_t jb, je;
  int64_t off;
  int64_t part;
  uint64_t rows;  // thin segment: its rows, and its number among the matrix's
  int32_t thin;
  int32_t pad;
};

// Geometry of a chunk height on a 64-lane wavefront whose lanes each hold
// V consecutive slots of a wave step (V > 1 only for C <= 64).
struct Geom {
  int C;    // chunk height
  int V;    // slots (rows) per lane
  int rpw;  // rows of one item (min(C, 64))
  int T;    // chunk columns per wave step (64 * V / rpw)
  int wpc;  // items (waves) per chunk (C / 64 for C = 128, else 1)
};

inline Geom geom_of(int C, int V = 1) {
  Geom g;
  g.C = C;
  g.V = V;
  g.rpw = C < 64 ? C : 64;
  g.T = 64 * V / g.rpw;
  g.wpc = C > 64 ? C / 64 : 1;
  return g;
}

// Waves per workgroup of the kernels that give each wave one work unit.
constexpr int kWavesPerBlock = 4;
// Waves per workgroup of the persistent batched kernel: one (its waves run
// slices of different lengths; a workgroup holds its CU slots until its
// last wave ends).
constexpr int kBatchPersistentWaves = 1;
// Accelerator dies (XCDs) of the device, each with its own L2; the hardware
// dispatcher sends workgroup b of a launch to XCD b mod kXcds.
constexpr int kXcds = 8;

// Segments of split chunks are whole multiples of this many chunk columns,
// so that every kernel's step width (at most 64 columns) divides them.
constexpr int kSegAlign = 64;

// Split segments are placed on the XCDs by their columns from this size of x on
// (one XCD's L2) and from this share of slots that hold an entry on (thin segments
// count with all rows of the slice). A row's entries are usually sorted, so a
// segment reads a range of x, and an eighth of x stays in an L2. Measured in chunk
// order / by column, us (share): 4,284 x 1,092,610, 2,633 entries per row, sigma = n,
// C = 16, 32, 64 113 / 73 (0.86), 119 / 79 (0.74), 134 / 102 (0.58; L2 misses at C = 16
// before thin segments 6.1 M -> 1.6 M lines, of which 1.1 M are the matrix), sigma = 512,
// C = 32 133 / 103 (0.48), 2,000 x 700,000, 600 per row, C = 64 22.0 / 18.2 (0.39);
// power-law 2M, C = 32, sigma = n, 2^17, 2^16 120 / 111 (0.96), 118 / 113 (0.56),
// 120 / 118 (0.41). Where most of a segment is padding the order of the chunks, whose
// rows lie near each other, wins: power-law 2M, C = 64, sigma = 2^17, 2^16 127 / 135
// (0.37), 129 / 149 (0.24), C = 32, sigma = 2^14, 1024 121 / 133 (0.20), 131 / 140 (0.08).
constexpr size_t kXcdMinX = 4 << 20;
constexpr double kXcdMinLive = 0.4;
// Most segments that one workgroup orders (automatic widths: some 30,000).
constexpr int64_t kXcdMaxSegs = 1 << 17;

// Segment width of the block form (automatic): long enough that a unit
// amortises its fixed cost (at least 64 wave steps), short enough that no unit
// is much longer than an average wave's share of the whole product (resident
// waves: CUs x 32). Converted from wave steps to chunk columns.
__host__ __device__ inline int32_t round_seg(int64_t cols) {
  int64_t s = (cols + kSegAlign - 1) / kSegAlign * kSegAlign;
  if (s < kSegAlign) s = kSegAlign;
  if (s > (1 << 30)) s = 1 << 30;
  return (int32_t)s;
}
__host__ __device__ inline int32_t auto_seg_cols(int64_t total_steps, int T, int cus) {
  const int64_t steps = total_steps / (2 * (int64_t)cus * 32);
  return round_seg((steps < 64 ? 64 : steps) * T);
}

// Segment width of the single-vector product, at most S: at least eight wave
// steps (one round of loads in flight) and 32 columns, more only where there
// would be more than two segments per resident wave. The block form keeps
// longer ones (S): its lanes walk the columns of a row alone and its segment
// sums are k times as many. us at 32 / 64 / 128 / 256 columns, C = 32: power-law
// 2M, sigma = n 109.7 / 111.0 / 115.4 / 116.0; 200k 13.3 / 15.8 / 24.4 / 24.3;
// 1M, sigma = 1024, FP32 70.3 / 70.1 / 77.6 / 77.7; 4,284 rows of 2,633 entries
// 72 / 70 / 82 / 87; at 16 columns 106, 14.5, 74 and 79.
__host__ __device__ inline int32_t single_seg_cols(int64_t total_steps, int T, int cus, int32_t S) {
  int64_t cols = total_steps / (2 * (int64_t)cus * 32);
  cols = (cols < 8 ? 8 : cols) * T;
  if (cols < 32) cols = 32;
  const int64_t a = T > 16 ? T : 16;
  cols = (cols + a - 1) / a * a;
  return cols < S ? (int32_t)cols : S;
}

// Thin segments: where at most thin_rows rows of a slice still hold entries the
// single-vector product takes those rows alone, 64 / rows columns a step and no
// fewer than the T of the others, whose lanes would step over padding for 24 of 32
// rows and more. kThinCols columns a unit with up to eight rows, kThinnestCols with
// up to two: at most eight steps, one round of loads. us without thin segments /
// with them, slots in their places / slots copied, at C = 16; 32; 64:
//   power-law 1M, sigma 1024  71 / 70 / 53;    98 / 80 / 55;    155 / 89 / 63
//   the same in FP32          53 / 51 / 41;    69 / 65 / 41;    105 / 73 / 49
//   2M, sigma 2^14            125 / 124 / 117; 138 / 130 / 120; 171 / 140 / 129
//   50k, sigma 1024           10.6 / 10.7 / 10.9; 12.6 / 10.9 / 11.0; 19.4 / 12.2 / 12.0
//   200k, sigma n             11.9 / 12.5 / 12.3; 13.5 / 12.7 / 13.2; 18.5 / 16.1 / 16.6
// In place, 256 columns with up to two rows: 200k 13.9, 14.2, 16.4; 256 with up to
// eight: 18, 18, 19. Copied, with up to sixteen rows (half or a quarter of the
// slice): within 2 %, at up to 20 % more memory.
constexpr int32_t kThinCols = 64;
constexpr int32_t kThinnestCols = 128;
constexpr int kThinnestRows = 2;
__host__ __device__ inline int thin_rows(int rpw, int T) {
  const int few = rpw < 16 ? 0 : rpw < 32 ? 4 : 8;  // a quarter of the rows at most
  return 64 / T < few ? 64 / T : few;
}

// Slots of a thin segment's copy, in the order that the lanes take them (64 a
// step): whole steps of eight rows, or of two. Split slices are wider than a
// segment and their segments full but for the last, so with C >= 16 rows the copies
// hold about as many slots as val at most.
__host__ __device__ inline int64_t thin_slots(int32_t S1, bool fixed) {
  const int64_t tc = fixed || S1 > kThinCols ? S1 : kThinCols, uc = fixed || S1 > kThinnestCols ? S1 : kThinnestCols;
  return ((8 * tc > 2 * uc ? 8 * tc : 2 * uc) + 63) / 64 * 64;
}

// Segments of a slice w columns wide in the single plan: dense ones of S1
// columns up to column thin, thin ones of tc columns up to column thinnest, then
// thin ones of uc columns. few: the columns in which more than thin_rows, and
// more than kThinnestRows, rows hold entries (nullptr: no thin segments).
struct Split1 {
  int32_t thin, thinnest, tc, uc;
  int32_t dense, segs;  // dense segments, dense and thin ones of tc columns
  int32_t all;
};
__host__ __device__ inline Split1 split1_of(const int32_t *few, int32_t w, int32_t S1, bool fixed) {
  Split1 r;
  const int64_t t = few ? ((int64_t)few[0] + S1 - 1) / S1 * S1 : w;
  r.thin = t < w ? (int32_t)t : w;
  r.tc = fixed || S1 > kThinCols ? S1 : kThinCols;
  r.uc = fixed || S1 > kThinnestCols ? S1 : kThinnestCols;
  const int64_t f2 = few && few[1] > r.thin ? few[1] - r.thin : 0;
  const int64_t t2 = r.thin + (f2 + r.tc - 1) / r.tc * r.tc;
  r.thinnest = t2 < w ? (int32_t)t2 : w;
  r.dense = (int32_t)(((int64_t)r.thin + S1 - 1) / S1);
  r.segs = r.dense + (int32_t)(((int64_t)r.thinnest - r.thin + r.tc - 1) / r.tc);
  r.all = r.segs + (int32_t)(((int64_t)w - r.thinnest + r.uc - 1) / r.uc);
  return r;
}

#if defined(__HIPCC__)
// A lane's share of a thin segment: row of the item (-1: none), column offset,
// columns per step, log2 of the lanes side by side.
struct ThinLane {
  int row, col, step, lg;
};
__device__ __forceinline__ ThinLane thin_lane(uint64_t rows, int lane) {
  const int n = __popcll(rows);
  ThinLane t;
  t.lg = n > 4 ? 3 : n > 2 ? 2 : n > 1 ? 1 : 0;
  t.step = 64 >> t.lg;
  t.col = lane >> t.lg;
  const int q = lane & ((1 << t.lg) - 1);
  for (int e = 0; e < q; ++e) rows &= rows - 1;
  t.row = q < n ? __ffsll((unsigned long long)rows) - 1 : -1;
  return t;
}
#endif

// Arguments of the spMVM kernels (by value).
struct SpmvArgs {
  const void *val;
  const int32_t *col;
  const int64_t *cs;
  const int32_t *cl;
  const int32_t *perm;  // nullptr: identity
  const void *x;
  void *y;
  int64_t nrows;
  int64_t nwork;        // items (no unit list) or units
  const Unit *units;    // block form: its units, or nullptr (wave w handles item w whole)
  const SplitDesc *splits;
  int64_t nsplit;
  void *partial;
  int32_t seg_cols;     // block form: chunk columns per segment (multiple of kSegAlign)
  const Unit1 *units1;  // single-vector product: its units, or nullptr (wave w handles item w)
  const int32_t *tcol;  // thin segments' copies of their slots (tslots each), or nullptr
  const void *tval;
  int64_t tslots;
  bool keep_y;          // single-vector product: permuted rows of y through the L2 (keeps_y)
  const int32_t *rl;    // single-vector product: length of every row in sorted
                        // order (N_c * C entries), or nullptr
  // block form only
  int32_t k;            // right-hand sides
  int32_t kt;           // right-hand sides per pass (ktile)
};

// Per-matrix descriptor of the batched kernel (device resident).
struct BatchMat {
  const void *val;
  const int32_t *col;
  const int32_t *perm;
  const void *x;
  void *y;
  int64_t nrows;
  const int32_t *tcol;  // thin segments' copies
  const void *tval;
  int64_t tslots;
  int32_t keep_y;       // permuted rows of y through the L2 (keeps_y)
};

// Split row slice of the batched kernel.
struct BSplitDesc {
  int32_t mat;
  int32_t item;
  int32_t nseg;
  int32_t pad;
  int64_t poff;
};

struct BatchArgs {
  const BatchMat *mats;
  const BUnit *units;
  int64_t nunits;
  const int32_t *slice;  // persistent form: nwaves + 1 unit offsets; nullptr: one unit per wave
  int32_t nwaves;
  const BSplitDesc *splits;
  int64_t nsplit;
  void *partial;
};

// x window of a product workgroup (LDS staging): groups of G consecutive
// chunks (G = kXwChunksWide when the windows of that many fit, else
// kXwChunks), at most kXwMaxSlots slots each.
constexpr int kXwChunks = 4;
constexpr int kXwChunksWide = 8;
constexpr int kXwMaxSlots = 8192;
struct XwArgs {
  const uint16_t *lcol;   // window position of every slot
  const int64_t *segoff;  // ngroups + 1 segment offsets
  const int32_t *seg;     // per segment: start column, window position, length
  int32_t wcap;           // LDS elements reserved for the window (the largest one)
  int32_t gc;             // chunks per group (one wave each): kXwChunks or kXwChunksWide
};
// Most segments a group's window may have (its table is staged in LDS too).
constexpr int kXwMaxSeg = 1024;

enum DtypeCombo {
  COMBO_F64_F64 = 0,   // val f64, x f64, acc f64
  COMBO_F32_F32 = 1,   // val f32, x f32, acc f32
  COMBO_F32_F64 = 2,   // val f32, x f32, acc f64
  COMBO_BF16_F32 = 3,  // val bf16, x f32, acc f32
  COMBO_BF16_F64 = 4,  // val bf16, x f32, acc f64
};

// Kernel launchers (return hipError of the launch).
// Each launcher enqueues the product kernel and, when rows are split, the
// kernel that adds their segment sums.
// skip_zero: slots holding value 0 skip their gather (for padding-heavy layouts).
hipError_t launch_spmv(int combo, int C, int U, int V, bool skip_zero, const SpmvArgs &a, hipStream_t s);
hipError_t launch_spmmv(int C, int KV, const SpmvArgs &a, hipStream_t s);
// Block form with LPR lanes per row (LPR 4: k = 16; LPR 8: k = 32 or 64;
// C >= 16): one pass, a.kt == a.k.
hipError_t launch_spmmv_rows(int C, int LPR, const SpmvArgs &a, hipStream_t s);
// Block form of any 2 <= k <= 64 in one pass (C in 8..128), a.kt == a.k. local: see
// spmmv_any_lanes.
hipError_t launch_spmmv_any(int C, bool local, const SpmvArgs &a, hipStream_t s);
// Block form with the x windows in LDS (C 16, 32 or 64, any k; no split chunks):
// kb right-hand sides at a time, `turns` times in a launch column, as block_turns
// says; lds_bytes: block_window_lds.
hipError_t launch_spmmv_xw(int C, int kb, int turns, const SpmvArgs &a, const XwArgs &w, size_t lds_bytes,
                           hipStream_t s);
// Product with the x window staged in LDS (C in 8..64, V 1 or 2, no split
// chunks); lds_bytes: the largest window times the x element size, rounded
// up to 8 bytes, plus 8 bytes per segment of the largest segment table.
hipError_t launch_spmv_xw(int combo, int C, int V, int U, const SpmvArgs &a, const XwArgs &w, size_t lds_bytes,
                          hipStream_t s);
hipError_t launch_batch(int combo, int C, int U, const BatchArgs &a, hipStream_t s);
// Resident waves per CU of the persistent batched kernel (its grid size).
int batch_waves_per_cu(int combo, int C, int U);

// Build kernels.
hipError_t build_rowlen(const int64_t *rpt, int64_t n, int64_t nnz, int32_t *len, uint32_t *flags,
                        unsigned long long *sumsq, int32_t *maxlen, hipStream_t s);
hipError_t build_colcheck(const int32_t *col, int64_t nnz, int64_t ncols, uint32_t *flags, hipStream_t s);
// Sorted row order for sigma > 1; tmp needs sort_tmp_elems(n, sigma) int64; flags and
// maxlen are build_rowlen's.
int64_t sort_tmp_elems(int64_t n, int64_t sigma);
hipError_t build_sort(const int32_t *len, const uint32_t *flags, const int32_t *maxlen, int64_t n, int64_t sigma,
                      int64_t *tmp, int32_t *perm, hipStream_t s);
// padded, total_steps: += the slots, the wave steps of T columns over all items
// (wpc per chunk); max_width: the widest chunk (all zeroed by the caller). few
// (or nullptr): per item, the lengths of its (thin_rows + 1)-th and its
// (kThinnestRows + 1)-th longest row.
hipError_t build_chunkwidth(const int32_t *len, const int32_t *perm, int64_t n, int C, int64_t nchunks, int T, int wpc,
                            int32_t *cl, int64_t *csz, int64_t *padded, int64_t *total_steps, int32_t *max_width,
                            int32_t *few, hipStream_t s);
// Exclusive scan of n int64 values (in-place allowed); tmp needs scan_tmp_elems(n) int64.
int64_t scan_tmp_elems(int64_t n);
hipError_t build_scan(const int64_t *in, int64_t *out, int64_t n, int64_t *tmp, hipStream_t s);
// cmap: column map applied to every stored column index (nullptr: none).
hipError_t build_fill(const int64_t *rpt, const int32_t *col, const double *val, int64_t n, int C,
                      const int32_t *perm, const int64_t *cs, int64_t nchunks, int64_t padded, const int32_t *cmap,
                      int32_t *scol, void *sval, int val_dtype, hipStream_t s);
hipError_t build_invert(const int32_t *perm, int64_t n, int32_t *iperm, hipStream_t s);
// Sizes of a layout and of its work plans, counted on the device.
struct PlanSizes {
  int64_t total_steps;  // wave steps of all items (from build_chunkwidth)
  int64_t nsplit, nsegs;            // block form: split slices, their segments
  int64_t nsplit1, nsegs1, nwhole1, nthin1;  // single-vector product: nthin1 of the segments are thin
  int32_t max_width;    // widest chunk (from build_chunkwidth)
  int32_t pad;
};
constexpr int kPlanCounts = 6;
struct PlanArgs {
  const int32_t *cl;
  int64_t nchunks, ncells;  // cells of grp chunks
  int grp;                  // 64 / C for C in 8..32, else 1
  int wpc, rpw, T, cus;
  int32_t seg_cols;         // > 0: given (rounded), 0: automatic, < 0: never split
  const int32_t *few;       // two per item (split1_of), or nullptr
  const int32_t *len, *perm;  // row lengths and order (perm nullptr: identity)
  int64_t nrows;
  int64_t *blocks;          // kPlanCounts * plan_blocks(ncells)
  uint32_t *next_thin;      // zeroed: numbers the thin segments
  PlanSizes *sizes;         // total_steps and max_width set, the rest written
};
struct PlanOut {
  Unit *units;        // block form: nsegs segments, then the whole items
  SplitDesc *splits;
  Unit1 *units1;      // single-vector product
  SplitDesc *splits1;
  Unit1 *segs;        // nullptr, or nsegs1 segments for plan_place to put into units1
};
int64_t plan_blocks(int64_t ncells);
hipError_t plan_count(const PlanArgs &a, hipStream_t s);
hipError_t plan_emit(const PlanArgs &a, int32_t S, int32_t S1, const PlanSizes &z, const PlanOut &o, hipStream_t s);
hipError_t plan_place(const PlanArgs &a, int C, const PlanSizes &z, const PlanOut &o, const int64_t *cs,
                      const int32_t *col, int64_t ncols, UnitCol *at, hipStream_t s);
// The thin segments' slots (units: nunits of a single plan; of those with rows,
// slots per segment) copied to tcol and tval, elements of esize bytes.
hipError_t build_thin(const Unit1 *units, int64_t nunits, int C, const int64_t *cs, const int32_t *col, const void *val,
                      int esize, int64_t slots, int32_t *tcol, void *tval, hipStream_t s);
// rl[p] = length of the row in sorted position p (0 for p >= n), p < np
hipError_t build_sorted_len(const int32_t *len, const int32_t *perm, int64_t n, int64_t np, int32_t *rl,
                            hipStream_t s);
// x windows of groups of gc consecutive chunks: segment count per group
// (nseg: ngroups + 1 int64, the last set to 0), the largest window (*maxwin,
// zeroed by the caller), flag bit 1 when a group holds more than kXwMaxSlots
// slots; then the segments and the window position of every slot.
hipError_t build_xw_count(const int32_t *col, const int64_t *cs, int64_t nchunks, int gc, int64_t *nseg,
                          uint32_t *flags, int32_t *maxwin, int32_t *maxseg, hipStream_t s);
hipError_t build_xw_fill(const int32_t *col, const int64_t *cs, int64_t nchunks, int gc, const int64_t *segoff,
                         int32_t *seg, uint16_t *lcol, hipStream_t s);
// The same in one pass where no group spans more than 131,072 columns (flag 2
// otherwise: nothing is defined; flag 1 or 4: so too, and some window has too
// many slots, or runs, or over maxwin_ok columns): counts, maxima and the
// positions; the runs go to segtab (xw_fast_table_elems int32) until
// build_xw_segs packs them. Flag 8: some group has over 64 runs, and only the
// counts and maxima are defined.
int64_t xw_fast_table_elems(int64_t nchunks, int gc);
hipError_t build_xw_fast(const int32_t *col, const int64_t *cs, int64_t nchunks, int gc, int maxwin_ok, int64_t *nseg,
                         uint32_t *flags, int32_t *maxwin, int32_t *maxseg, int32_t *segtab, uint16_t *lcol,
                         hipStream_t s);
hipError_t build_xw_segs(const int32_t *segtab, const int64_t *segoff, int64_t ngroups, int32_t *seg, hipStream_t s);
// out[p] = in[perm[p]] (scatter = false) or out[perm[p]] = in[p] (scatter = true).
hipError_t permute_vector(const void *in, void *out, const int32_t *perm, int64_t n, int elem_bytes, bool scatter,
                          hipStream_t s);
hipError_t launch_crs(const int64_t *rpt, const int32_t *col, const double *val, const double *x, double *y,
                      int64_t n, int L, hipStream_t s);

// Bandwidth probes.
hipError_t probe_read(const void *a, size_t bytes, double *sink, hipStream_t s);
hipError_t probe_copy(const void *a, void *b, size_t bytes, hipStream_t s);
hipError_t probe_write(void *a, size_t bytes, hipStream_t s);
// Four random rows of row_bytes read per row written in order, over an input
// of the largest power-of-two row count that fits in bytes and an output of
// as many rows; returns the rows moved (read and written).
int64_t probe_rows_write(const void *a, void *out, size_t bytes, int row_bytes, hipStream_t s, hipError_t *err);
// Launches 2^27 random 8-byte gathers over the largest power-of-two prefix
// of a (bytes); returns the gather count.
int64_t probe_gather(const void *a, size_t bytes, double *sink, hipStream_t s, hipError_t *err);
// Launches random whole-row reads (rows of row_bytes = 128, 256 or 512 bytes)
// over the largest power-of-two number of rows that fits in bytes; returns
// the row count.
int64_t probe_rows(const void *a, size_t bytes, int row_bytes, double *sink, hipStream_t s, hipError_t *err);

}  // namespace sell

// The handle.
struct sell_matrix {
  int64_t nrows = 0, ncols = 0, nnz = 0;
  int32_t C = 0;
  int64_t sigma = 1;
  sell::Geom g{};
  int64_t nchunks = 0, padded = 0;
  int64_t max_len = 0;
  double beta = 1.0, zeta = 0.0;
  sell_dtype vdt = SELL_F64, xdt = SELL_F64, adt = SELL_F64;
  int combo = 0;
  int32_t unroll = 8;
  int32_t seg_cols = 0;
  int32_t ktile = 0;
  int32_t kmax = 32;
  bool sym = false;  // column indices permuted too: x and y live in sorted order
  int device = 0;

  int32_t *perm = nullptr;
  int32_t *rl = nullptr;   // row_lengths: length of every row in sorted order (N_c * C)
  int32_t *cl = nullptr;
  int64_t *cs = nullptr;
  int32_t *col = nullptr;
  void *val = nullptr;

  int64_t nitems = 0;
  int64_t nunits = 0;
  sell::Unit *units = nullptr;  // nullptr when no chunk is split
  // the single-vector product's plan on split layouts (plan_single)
  sell::Unit1 *units1 = nullptr;
  int64_t nunits1 = 0;
  sell::SplitDesc *splits1 = nullptr;
  int32_t *tcol = nullptr;  // thin segments' copies of their slots
  void *tval = nullptr;
  int64_t tslots = 0;
  bool auto_seg = false;    // segment widths chosen here, not by the caller
  int64_t nsplit1 = 0, nsegs1 = 0;
  int64_t nsplit = 0;
  int64_t nsegs = 0;                  // total segments of split items
  sell::SplitDesc *splits = nullptr;  // per split id
  void *partial = nullptr;            // nsegs * rpw * next_pow2(kmax) doubles, or nsegs1 * rpw where that is more

  uint16_t *lcol = nullptr;     // x window mode: window position of every slot
  int64_t *xsegoff = nullptr;   // ngroups + 1 segment offsets
  int32_t *xseg = nullptr;      // per segment: start column, window position, length
  int64_t nxseg = 0;
  int32_t xwin_max = 0;         // largest window, in x elements
  int32_t xseg_max = 0;         // most segments of one window
  int32_t xw_gc = 0;            // chunks per window group
  sell::BlockWindows xw_block;  // the windows, where the block form may use them

  sell_allocator alloc{};
  bool custom_alloc = false;
  std::vector<std::pair<void *, size_t>> owned;
  int64_t device_bytes = 0;
};
