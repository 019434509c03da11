// Copies of ragged dense operands (spmm.hip): which handles keep room for one, which calls take one, and how much
// workspace that costs.  Host arithmetic only, so that it can be checked without a device.
//
// Rows of a dense operand that do not start on 128-byte lines make every gathered slice touch one line more than it holds.
// The copy (k_stage_cols: the columns of one launch, row by row, to whole lines) costs one pass over X and a launch per 128
// columns.  us per SpMM without / with it, mean over several X in turn:
//   233 k columns, 115 M entries: 602 columns 13853 / 11816, 301 7200 / 6140, 50 1404 / 1241;
//   2.4 M, 124 M: 301 15246 / 12698, 50 2745 / 2507;
//   1 M, 40 M: 602 9066 / 8221, 140 2337 / 2078, 50 852 / 793, 28 557 / 409, 12 366 / 361;
//   200 k, 20 M: 140 795 / 719, 20 178 / 153, 12 145 / 141;  200 k, 6.4 M: 602 1425 / 1206;
//   257 columns, whose last launch starts 3 columns earlier: 233 k, 115 M 6616 / 5744; 2.4 M, 60 M 8092 / 7392; 200 k, 20 M 1510 / 1355;
//   200 k, 6.4 M 694 / 596.
// Outside the rule:
//   1 M, 40 M: 6 302 / 328, 9 352 / 357, 42 752 / 770, 76 1197 / 1264;  1 M, 16 M: 602 4720 / 4870;
//   50 k, 1.5 M: 602 290 / 330;  10 k, 1 M: 602 154 / 196;  50 k, 6 M: 20 58 / 61;
//   100 columns, whose 400 bytes touch four lines anyway: 2349 / 2426 (233 k), 4832 / 5364 (2.4 M);
//   cut, without slices: 500 k, 16.5 M: 500 2750 / 2869, 602 3387 / 3418, 19 M: 500 3057 / 3142 (inside: 22 M: 301 2226 / 2120, 602
//   4267 / 4049);
//   cut, two slices: 524 k, 17 M: 200 1238 / 1325, 500 2956 / 3123; 560 k, 20 M: 200 1493 / 1531 (inside: 257 2046 / 2022); 640 k, 21 M:
//   200 1632 / 1671 (inside: 301 2532 / 2445; 800 k, 26 M: 200 2089 / 2102, 500 4939 / 4927; 1.4 M, 46 M: 200 3990 / 3858, 500 9639 / 8954);
//   rows that begin at half lines, 1.1 M, 37 M: 303 of 304 columns 5 % slower; 882 k, 30 M: 592 5894 / 6208; 1.06 M, 36 M: 196 of 208 2660 / 2798;
//   uniform, all rows cut: 350 k, 105 M: 17 1273 / 1445, 20 1407 / 1444; 150 k, 45 M: 50 985 / 1042 (inside: 350 k: 13 1082 / 964, 22 1626 /
//   1445, 28 2088 / 1452; 150 k: 28 528 / 396);
//   uniform, not cut, per cent slower with: 91 k, 8.9 M: 18 16; 76 k, 12 M: 18 16; 115 k, 9.3 M: 17 9; 167 k, 14 M: 12 9 (inside, faster: 85 k, 12 M:
//   13 6, 24 9; 183 k, 11 M: 18 14; 222 k, 25 M: 12 2);
//   not cut, hub rows, per cent slower with, mean over graphs of 30 k to 240 k columns: 272, 304, 528, 560, 592 columns 1.6 to 2.0, at worst 7.8 (98 k,
//   6.3 M: 528) (inside, faster: those around 390 2.4, 460 1.8, 490 5.5; widths that save 6 to 7 % of the lines 3.4).
#pragma once
#include "partition_sizes.h"

namespace isp_stage {

constexpr int COLS = 128;  // columns of a launch that gathers from a copy
constexpr int ALIGN = 32;  // floats of a line

// 32 times the 128-byte lines that w floats of a row touch, on average over the rows: `ld` floats apart, the first begins at
// address `at`.
inline int64_t line_sum(uintptr_t at, int64_t ld, int w) {
  const int base = (int)(at & (4 * ALIGN - 1)) / 4;  // (in floats)
  int step = ALIGN;
  while (ld % step != 0) step /= 2;  // rows begin at base + multiples of step
  int64_t sum = 0;
  for (int o = 0; o < ALIGN; o += step) sum += step * (((base + o) % ALIGN + w + ALIGN - 1) / ALIGN);
  return sum;
}

// The launches that cover d columns: first column (a last tile of fewer than 4 columns starts earlier and computes some
// columns again: float4 lanes) and width of the one that continues at k0.
inline int tile_start(int k0, int d) { return d >= 4 && d - k0 < 4 ? d - 4 : k0; }
inline int tile_width(int k_base, int d, int tile, int64_t n_cols) {
  const int w = d - k_base < tile ? d - k_base : tile;
  return w > 128 && w <= 224 && n_cols >= 512 << 10 ? 128 : w;
}

// line_sum of all of them.
inline int64_t tile_lines(uintptr_t at, int64_t ldx, int d, int tile, int64_t n_cols) {
  int64_t sum = 0;
  for (int k0 = 0, w; k0 < d; k0 += w) {
    const int k_base = tile_start(k0, d);
    w = tile_width(k_base, d, tile, n_cols);
    sum += line_sum(at + 4 * (uintptr_t)k_base, ldx, w);
  }
  return sum;
}

// The lines that a call on X touches, and with copies, for its rule.  The same values give the same bits wherever X lies,
// so its address counts only where a copy leaves the launches as they are: rows of whole lines (128 columns at a time anyway)
// and less than 128 columns (one launch).  Other rows count as if the first began a line: a view that begins elsewhere can miss
// a copy for it (132 of 136 columns from the sixth on, 233 k columns, 115 M entries: 3830 us, 3240 with copies).
inline int64_t operand_lines(uintptr_t at, int64_t ldx, int d, int tile, int64_t n_cols) {
  return tile_lines(ldx % ALIGN == 0 || d < COLS ? at : 0, ldx, d, tile, n_cols);
}
// (every copied tile begins its rows at lines, or within the part of one that they fit: also the last tile that starts earlier)
inline int64_t copied_lines(int d) {
  int64_t sum = 0;
  for (int k0 = 0, w; k0 < d; k0 += w) {
    const int k_base = tile_start(k0, d);
    w = d - k_base < COLS ? d - k_base : COLS;
    sum += line_sum(0, ALIGN, w);
  }
  return sum;
}

// A handle keeps room for 128 columns where a column has so many entries that its row is gathered far more often than
// copied, and the matrix is of a size at which any call takes a copy.
constexpr int64_t MIN_PER_COL = 32, MIN_NNZ = 3000000;
// A call takes the copy from 12 columns up, where the work outweighs the launches, and where the lines that a row touches
// fall by a fifth, or by 5 % beyond 128 columns, which the copies also let run 128 at a time; by 6 % where hub rows on the
// ordinary partition hide some of it, unless a launch of 129 to 255 columns, which take longest for their width, is replaced.
constexpr int MIN_D = 12;
constexpr int64_t MANY_NNZ = (int64_t)8 << 20, MANY_MULS = 2000000000;
constexpr int LINES_NARROW = 120, LINES_WIDE = 105, LINES_WIDE_UNEVEN = 106;  // per cent
// On the packed layout, where most gathers hit the L2s, the lines saved have to outweigh the lines copied: a copied line costs
// as much as gathering five; four where the copies also give two slices, two and a half there from SLICES_FAR columns on.  (In
// tenths.)
constexpr int COPIED_LINE = 50, COPIED_LINE_SLICES = 40, COPIED_LINE_FAR = 25;
constexpr int64_t SLICES_FAR = 640 << 10;
constexpr int64_t KEPT_BYTES = 8 << 20;  // (an L2: 4 MB)

// What a call brings along: lines and lines_copied in the units of line_sum; cut: it runs on the packed layout, two_slices:
// its 128-column launches run as two slices if they gather from copies, even: its rows are about equally long, more than half
// of them cut or, on the ordinary partition, none a hub row.
struct call {
  int64_t nnz, n_cols, ldx;
  int d;
  int64_t lines, lines_copied;
  bool cut, two_slices, even;
};

// Floats per row of the copy of w columns: whole lines, or the part of one (16 floats, 8) that the row fits, so that rows
// share lines but none is cut.
inline int pitch(int w) { return w <= 8 ? 8 : w <= 16 ? 16 : (w + ALIGN - 1) / ALIGN * ALIGN; }

inline bool call_pays(const call& c) {
  if (c.d < MIN_D || (c.nnz < MANY_NNZ && c.nnz * c.d < MANY_MULS)) return false;
  const bool wide_tail = c.d % ISP_PARTIAL_TILE > COLS;  // (the copies replace a launch of 129 to 255 columns)
  const int lines = c.d <= COLS ? LINES_NARROW : c.cut || c.even || wide_tail ? LINES_WIDE : LINES_WIDE_UNEVEN;
  if (100 * c.lines < lines * c.lines_copied) return false;
  const int copied_line = !c.two_slices ? COPIED_LINE : c.n_cols < SLICES_FAR ? COPIED_LINE_SLICES : COPIED_LINE_FAR;
  if (c.cut && 10 * (c.nnz / c.n_cols) * (c.lines - c.lines_copied) < copied_line * c.lines_copied) return false;
  // Where rows are equally long no columns are popular: the L2s keep a part of X, the band in work on the packed layout, and a copy
  // that takes more room than X by a larger factor than it saves lines makes more of them miss; without bands where X is little
  // larger than an L2.
  const bool kept = c.cut || c.n_cols * c.ldx * 4 < KEPT_BYTES;
  return !(kept && c.even && c.d <= COLS && c.lines * c.ldx < c.lines_copied * pitch(c.d));
}

// The widest pitch that calls of up to max_d columns ask for; `always`: ISP_STAGE_MIN is set.
inline int pitch_up_to(int max_d, bool always) {
  return max_d < (always ? 4 : MIN_D) ? 0 : pitch(max_d < COLS ? max_d : COLS);
}

inline size_t bytes(int64_t n_cols, int n_floats) { return isp_align((size_t)n_cols * n_floats * sizeof(float)); }

// ISP_STAGE_MIN (entries per column; 0 = no copies) overrides the rule and its limit on the size: isp_tuning::stage_min, 0 where
// it is not set and -1 for no copies.
inline int read_min() {
  const int m = isp_part::env_int("ISP_STAGE_MIN", -1, -1, 1 << 20);
  return m < 0 ? 0 : m == 0 ? -1 : m;
}

// Bytes that a matrix of this shape needs for its copies; 0 where none is taken.
inline size_t wanted(int64_t n_cols, int64_t nnz, int forced = 0) {
  if (n_cols <= 0 || forced < 0) return 0;
  if (forced > 0 ? nnz / n_cols < forced : nnz / n_cols < MIN_PER_COL || nnz < MIN_NNZ) return 0;
  return bytes(n_cols, COLS);
}

// Workspace laid out for the copies besides the partial rows.  These are sized for the worst case, some 12 bytes per entry
// where the copies ask for at most 16, and a SpMM leaves most of them idle; with the packed layout it leaves all rows of the
// ordinary partition, so that only what those lack is added and the copies always have a place.  Without it (less than 8 Mi
// entries, less than 64 Ki columns, or more than 256 Mi entries) the copies have workspace of their own up to OWN_MAX
// and beyond that whatever is idle, or there are none.
constexpr size_t OWN_MAX = (size_t)128 << 20;
inline size_t own_bytes(int64_t n_cols, int64_t nnz, size_t partial_bytes, bool packed, int forced = 0) {
  const size_t b = wanted(n_cols, nnz, forced);
  if (packed) return b > partial_bytes ? isp_align(b - partial_bytes) : 0;
  return b <= OWN_MAX ? b : 0;
}

// A stretch of workspace, 256-byte aligned.
struct room { char *begin, *end; };
inline float* take(room& r, size_t n) {
  if (r.end < r.begin || (size_t)(r.end - r.begin) < n) return nullptr;
  r.end -= n;
  return reinterpret_cast<float*>(r.end);
}

// The first of n rooms that holds the copies of A's ragged operands becomes their place; without one A takes none.  No other
// call writes in the rooms but in the last, which takes in the one before it to its end: the calls on a handle follow each
// other, the last room serves all the same.  isp_spmm_static_scratch, where it serves the handle, gets a place in what is
// left of the others (nothing that would hold it, if the first copy had to take the last).
inline void place(isp_csr* A, room* rooms, int n) {
  const size_t b = wanted(A->v.n_cols, A->v.nnz, A->tune.stage_min);
  A->stage = A->static_stage = nullptr;
  for (int k = 0; k < n && b > 0 && !A->stage; ++k) A->stage = take(rooms[k], b);
  A->stages = A->stage != nullptr;
  A->stage_cols = A->stages ? COLS : 0;
  if (!A->stages || A->spmm_rows > ISP_STATIC_SCRATCH_ROWS) return;
  for (int k = 0; k < n - 1 && !A->static_stage; ++k) A->static_stage = take(rooms[k], b);
}

}  // namespace isp_stage
