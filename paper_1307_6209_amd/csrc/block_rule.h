// Which kernel a block product runs. No HIP, so that it can be checked on its own.
//
// The x windows in LDS (k_spmmv_xw): the kernel stages kb right-hand sides of a group's
// window at a time, `turns` times for one launch column. It wins where a staged element
// serves many slots and the matrix passes by once; it loses to the kernels that read X
// through L1 and L2 where rows are so short that staging is most of the work, where the
// columns past kBlockRegCols, read again in each turn, and a large window meet, or where
// few workgroups run. All figures: us, other kernels / this one, FP64; w: mean chunk
// width, r: slots per window element.
#pragma once

#include <cstddef>
#include <cstdint>

namespace sell {

// Chunk columns that stay in registers over the turns.
constexpr int kBlockRegCols = 28;

// The x windows of an FP64 layout, C 16, 32 or 64; C 0: none that the block form uses.
struct BlockWindows {
  int C = 0, group = 0;  // chunk height, chunks per workgroup
  int64_t groups = 0;
  int maxwin = 0, maxseg = 0;  // elements and runs of the largest window
  double width = 0, reuse = 0;  // w and r
  size_t lds = 0;  // bytes of LDS on a CU
  int cus = 0;
};

inline size_t block_window_lds(int kb, int maxwin, int maxseg) {
  return (size_t)maxwin * (size_t)kb * sizeof(double) + 8 * (size_t)maxseg;
}

// The windows that a layout offers to the block form. They have to be worth staging:
// each element read by 2.5 slots or more, in runs of 8 or more on average. 5-point
// Laplacian 1000^2 (r 1.7), k = 4, C = 16, 32, 64: 44, 29, 26 / 50, 45, 40; 60,000
// rows of up to 40 random columns of 2,000 (r 2.6, runs of one or two), k = 8, C = 16:
// 19 / 28.
inline BlockWindows block_windows(int C, int group, int64_t nchunks, int64_t padded, int maxwin, int maxseg,
                                  int64_t runs, size_t lds, int cus) {
  BlockWindows b;
  b.group = group;
  b.groups = (nchunks + group - 1) / group;
  b.maxwin = maxwin;
  b.maxseg = maxseg;
  b.lds = lds;
  b.cus = cus;
  const double elems = (double)maxwin * (double)b.groups;
  if (elems <= 0 || (C != 16 && C != 32 && C != 64)) return b;
  b.width = (double)padded / (double)nchunks / C;
  b.reuse = (double)padded / elems;
  // two workgroups on a CU: 96^3 stencil, k = 8 all at once, one (86 KB) 122 / 130
  if (b.reuse >= 2.5 && elems >= 8.0 * (double)runs && 2 * block_window_lds(4, maxwin, maxseg) <= lds) b.C = C;
  return b;
}

struct BlockTurns {
  int kb, turns;  // kb 0: the other kernels
};

// Resident waves of a CU as far as LDS limits them.
inline int block_waves(const BlockWindows &b, int kb) {
  return (int)(b.lds / block_window_lds(kb, b.maxwin, b.maxseg)) * b.group;
}

// How k right-hand sides run on windows b, with the automatic pass width.
inline BlockTurns block_turns(const BlockWindows &b, int k) {
  const BlockTurns other{0, 0};
  if (b.C == 0 || k < 2 || k > 32) return other;
  const bool dense = b.reuse >= 15;  // bands: the window is little more than the group's rows
  if (b.C == 64) {
    // One lane a row: k = 2 leaves half of it idle, 5 to 7 part of it. Stencil 60^3
    // (w 26.6, r 6), k = 2 .. 8: 17, 26, 26, 31, 31, 33, 47 / 16, 17, 17, 32, 34, 40,
    // 42; 25-point 500^2 (w 25, r 4.9) 18, 27, 24, 32, 33, 34, 45 / 20, 21, 22, 34, 36,
    // 43, 45; band of 16 (r 15) 21, 32, 28, 40, 40, 42, 59 / 19, 21, 22, 34, 37, 51, 56;
    // of 28 28, 43, 37, 54, 55, 56, 70 / 21, 23, 24, 36, 40, 51, 56; of 12 19, 32, 27,
    // 38, 39, 41, 57 / 21, 23, 23, 38, 43, 58, 65.
    if (k > 8) return other;
    const bool ok = k == 2 || k == 5 || k == 6 ? b.width >= 26 || (b.width >= 16 && dense)
                    : k <= 4                   ? b.width >= 12
                    : k == 7                   ? b.width >= 28 && dense
                                               : b.width >= 20;
    if (!ok) return other;
  } else if (b.C == 32) {
    // 9-point 700^2 (w 9, r 3), k = 2, 4, 8, 12: 19, 22, 36, 51 / 24, 25, 37, 65; band of
    // 12 27, 29, 46, 67 / 28, 30, 41, 70; of 16 31, 33, 47, 72 / 26, 26, 36, 61; 19-point
    // 90^3 (w 18.8, r 3.7) 50, 53, 81, 123 / 43, 44, 70, 124.
    if (b.width < 16) return other;
  } else if (b.width < 12 && (b.width < 8 || (k > 4 && b.reuse < 7.5))) {
    // 9-point 700^2 (r 2.9), k = 2, 4, 8, 12: 31, 32, 36, 60 / 27, 28, 38, 55, 400^2
    // 11, 12, 14, 23 / 12, 12, 17, 23; band of 9 (r 8) 36, 37, 43, 71 / 29, 30, 40, 55;
    // of 6 41, 43, 51, 70 / 39, 41, 54, 74.
    return other;
  }
  if (k <= 4) return {4, 1};
  if (k <= 12) {
    // Two turns and four. Past kBlockRegCols columns the others are read again in each,
    // from 20 waves on a CU on, 24 at C = 16: 125-point 60^3 (w 120, r 5, 12 waves),
    // k = 8, 12: 157, 228 / 238, 357, 40^3 (16 waves) 52, 94 / 55, 82; 300,000 rows of
    // up to 90 of 1,000 columns (20 waves) 150, 218 / 190, 278; three unknowns a node
    // of 44^3 (w 79, r 7.8, 28 waves) 122, 178 / 111, 170; 49-point 400^2 at C = 32
    // (w 49, 20 waves) 47, 71 / 35, 53; band of 128 84, 125 / 62, 89.
    if (b.width > kBlockRegCols && block_waves(b, 4) < (b.C == 16 ? 24 : 20)) return other;
    // Small groups need three workgroups a CU: stencil, C = 16, k = 8, 12: 34^3 (615
    // groups) 11, 14 / 12, 15; 38^3 (858) 15, 23 / 13, 16.
    if (b.C == 16 && b.groups < 3 * (int64_t)b.cus) return other;
    return {4, k <= 8 ? 2 : 4};
  }
  // Two turns of eight, whole ones (rows of Y end inside a line otherwise, written
  // by halves): stencil 80^3, C = 32, k = 16, 20, 24, 28, 31, 32: 143, 206, 210, 218,
  // 233, 257 / 104, 207, 162, 258, 320, 203; or where the window is little more than
  // the group's rows: band of 40 (r 31) 117, 180, 181, 183, 188, 216 / 58, 114, 91, 139, 172, 114;
  // of 28 (r 25) k = 28, 31: 173, 177 / 172, 215. C = 16, k = 20, 28, 31: band of 16
  // (r 13) 126, 132, 140 / 85, 99, 128; of 12 (r 10) 118, 125, 146 / 96, 114, 150.
  if (k % 8 != 0 && b.reuse < (b.C == 16 ? 12.5 : 30)) return other;
  // Three unknowns a node of 44^3 (w 79, 12 waves), k = 16, 32: 190, 335 / 192, 365;
  // 125-point 40^3 (8 waves) 79, 138 / 104, 203; stencil 44^3, C = 32 (w 26, 12 waves)
  // 32, 62 / 22, 42; 60^3 (16 waves) 64, 120 / 49, 92.
  const int waves = block_waves(b, 8);
  if (2 * block_window_lds(8, b.maxwin, b.maxseg) > b.lds) return other;
  if (waves < (b.width > kBlockRegCols ? 16 : 12)) return other;
  return {8, 2};
}

// Right-hand sides per lane of the pass kernel: a power of two <= 8 that divides k
// (aligned vector gathers), with the pass width, 64 / rpw times as many, not above
// ktile or (0) the next power of two of k, 16 at most.
inline int pass_width(int rpw, int k, int ktile) {
  int next = 1;
  while (next < k && next < 16) next <<= 1;
  const int most = (ktile > 0 ? ktile : next) / (64 / rpw), want = most > 1 ? most : 1;
  int kv = 1;
  while (kv * 2 <= want && kv * 2 <= 8 && k % (kv * 2) == 0) kv *= 2;
  return kv;
}

// Lanes per row of the one-pass kernel of any width (k_spmmv_any): no fewer than
// spread a chunk over a wave. local: neighbouring rows share their columns (the layout
// has x windows), the X rows come from L1 and L2 and the fewest accesses of a wave per
// nonzero win (7-point stencil 96^3, k = 5, C = 32: 2 lanes 40 us, 4 lanes 55); else
// each access of a row is a request of its own beyond L1 and one access per row wins
// (random rows, k = 5: 2 lanes 123 us, 4 lanes 106), up to k = 16, where 4 lanes with
// two accesses and 8 with one are even (k = 9: random 148 / 143, power-law 144 / 169).
inline int spmmv_any_lanes(int C, int k, bool local) {
  const int least = C < 64 ? 64 / C : 2;
  const int want = local ? (k <= 8 ? 2 : k <= 16 ? 4 : 8) : (k <= 4 ? 2 : k <= 16 ? 4 : 8);
  return want > least ? want : least;
}

// Chunk columns in flight of k_spmmv_any (np pairs of right-hand sides a lane) and of
// the pass kernel (kv right-hand sides a lane).
constexpr int any_columns(int lpr, int np) { return np >= 3 ? 3 : np == 2 ? (lpr == 2 ? 8 : 4) : 8; }
constexpr int pass_columns(int kv) { return kv >= 8 ? 4 : kv >= 4 ? 8 : 12; }

// Whether one pass of any width beats the `passes` (two or more) of the pass kernel,
// kv right-hand sides a lane. It reads the matrix and the lines of X once, but walks
// a unit's columns in shorter rounds, while the passes walk them side by side: where
// the product lasts as long as its longest units, of `longest` columns, it loses.
// `full` counts how many such units the slots would fill; the shorter its rounds and
// the fewer the passes, the more of them it takes. us, passes / one pass:
//   power-law 1M, sigma n, C = 16, 32, 64, k = 5        204, 273, 429 / 115, 118, 124
//   200,003 rows of up to 48, sigma 1024, k = 5, 24     156, 152, 259 / 106; 224, 227, 263 / 192
//   27-point stencil 96^3, k = 5, 24 (no windows)       280, 249, 383 / 146, 107, 107; 473, 576, 733 / 369
//   power-law 50,000, sigma n, C = 8, k = 20 (full 50)  94 / 163
//   150,000, C = 16, k = 10 (full 170)                  69 / 92
//   500,000, C = 8, k = 20 (full 520)                   192 / 196
//   300 x 50,000, 300 per row, C = 16, k = 10 (19)      77 / 146
inline bool one_pass_wins(int64_t padded, int64_t longest, int rpw, int lpr, int np, int kv, int passes) {
  const double full = (double)padded / ((double)(longest > 1 ? longest : 1) * rpw);
  const double ratio = (double)pass_columns(kv) / any_columns(lpr, np), need = (ratio - 1) / (passes - 1);
  if (need >= 0.55) return full >= 450 * need;
  return ratio < 2.5 || full >= 32;
}

}  // namespace sell
