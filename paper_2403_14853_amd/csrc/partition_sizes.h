// Sizes of the work partitions (csr_build.hip) as functions of the matrix's shape: host arithmetic only, so that the
// bounds the workspaces are laid out by can be checked without a device.
#pragma once
#include <math.h>
#include <stdlib.h>
#include "isp_internal.h"

namespace isp_part {

struct partition_params {
  int block_cost, hub_t, seg_len;
  int row_cost;   // cost units of a row besides its entries (1; 2 in the derived matrix, which allows larger blocks)
  int bands;      // column bands of the finest cut (a power of two); 1 = no band cuts
  int min_piece;  // a hub row is cut into at most degree / min_piece bands
};

constexpr int MAX_BANDS = 64;  // one piece per lane
// Column bands a hub row of deg entries is cut into: the largest power of two <= min(bands, deg / min_piece).
__host__ __device__ inline int hub_bands(int64_t deg, const partition_params& pp) {
  int br = 1;
  while (br * 2 <= pp.bands && (int64_t)(br * 2) * pp.min_piece <= deg) br *= 2;
  return br;
}

// About how many segments a hub row of deg entries has: its columns spread over the bands, chance included (bands of 79 entries on average and
// segments of 80: not a segment to a band but 1.4).
inline int64_t row_segments(int64_t deg, const partition_params& pp) {
  const int64_t br = hub_bands(deg, pp);
  int64_t len = (deg + br - 1) / br;
  if (br > 1) len += (int64_t)sqrt((double)len);
  return br * ((len + pp.seg_len - 1) / pp.seg_len);
}

inline int64_t max_hub_rows(int64_t n_rows, int64_t nnz, const partition_params& pp) {
  const int64_t h = nnz / ((int64_t)pp.hub_t + 1);
  return h < n_rows ? h : n_rows;
}

// Most segments: a row of degree deg has at most deg / min_piece pieces, and a piece of len entries at most
// len / seg_len + 1 segments.
inline int64_t max_segments(int64_t n_rows, int64_t nnz, const partition_params& pp) {
  return nnz / pp.seg_len + (pp.bands > 1 ? nnz / pp.min_piece : 0) + max_hub_rows(n_rows, nnz, pp) + 1;
}

inline int env_int(const char* name, int dflt, int lo, int hi) {
  const char* s = getenv(name);
  if (!s || !*s) return dflt;
  long v = strtol(s, nullptr, 10);
  if (v < lo) v = lo;
  if (v > hi) v = hi;
  return (int)v;
}

// slots: wavefront slots of the device (4,096 on an MI355X: 256 compute units); n_cols: where a cut by columns can pay (below)
inline partition_params get_params(int64_t n_rows, int64_t nnz, int64_t slots, int64_t n_cols) {
  partition_params p;
  p.row_cost = 1;
  // Upper limits = what the grouped kernels' per-wave LDS tables hold (block_cost + hub_t <= 768
  // entries, block_cost <= 256 rows, seg_len <= 768 entries).  The environment overrides exist for
  // tuning and for tests that want many small work items.
  // Small matrices get smaller row blocks, about as many as the chip has wavefront slots (compute units x 16):
  // a wavefront's work is a chain of dependent memory round trips, and a short chain on every slot
  // finishes sooner than a long one on a few (4,096 rows x 9 entries: 16 -> 7 us per SpMM).
  const int64_t share = (nnz + n_rows + slots - 1) / slots;  // cost units per slot
  const int64_t auto_cost = share < 16 ? 16 : (share > 256 ? 256 : share);
  p.block_cost = env_int("ISP_BLOCK_COST", (int)auto_cost, 16, 256);
  // ... and shorter hub segments, for the same reason and because the segments are the heavy items that the
  // launch hands out last: a quarter of the per-slot share, between 80 and 512 entries, rows of more than two
  // segments' worth being hubs (2.4 M entries: segments of 157 instead of 512, 0.512 -> 0.468 ms for four
  // SpMMs; 0.6 M entries: 0.167 -> 0.155 ms; from 8 M entries up the sizes are 512 / 512 as before).
  // With many columns a column band of the dense operand is far larger than an L2, and finer pieces of the
  // hub rows (segments of at most 384, pieces from 192 entries) keep more of each segment's gathers inside its
  // band (2.4 M columns: 5.30 -> 5.19 ms per SpMM, the other kernels 1-3 %); with few columns a band's popular
  // rows fit an L2 anyway and the longer segments win (233 k columns: SDDMM 3.21 vs 3.32 ms).
  // Measured again with the present kernels (segments 256 .. 512, smallest pieces 64 .. 256, on the three large
  // benchmark graphs): segments of at most 320 and pieces from 128 entries are best or within 1 % of it for every
  // kernel on every one of them (233 k columns: SpMM 2.68 -> 2.59 ms, SDDMM 2.71 -> 2.60 ms; 2.4 M columns:
  // FusedMM 5.59 -> 5.41 ms; 1 M columns: FusedMM backward 1.36 -> 1.32 ms).
  // Where the slots outnumber the items, the longest row of a block and the longest segment are the launch: 48 entries and
  // 64 to a row up to 28 units per slot (115 k units), 64 and 96 up to 128 (520 k), 80 and 160 above.  With 80 and 160 / 48 and 64 / 64 and
  // 96 (us; R-MAT): 2,859 rows, 34 k entries, 80 columns: SpMM 7.4 / 6.6 / 7.0, SDDMM 9.7 / 6.4 / 7.6, FusedMM 15.0 / 9.5 / 11.9, its backward
  // 22.1 / 12.8 / 17.0; 4,092, 90 k, 200 columns: 11.9 / 10.5 / 10.1, 13.1 / 10.3 / 11.1, 32.2 / 17.4 / 26.1, 51.8 / 28.5 / 42.0; 7,881, 157 k, 133:
  // 15.6 / 13.4 / 12.6, 19.5 / 14.6 / 15.2, 40.8 / 22.8 / 24.1; 30 k, 376 k, 24: 9.5 / 11.2 / 9.0, 8.1 / 8.0 / 7.8, 12.1 / 12.2 / 11.4; 19 k, 436 k, 24:
  // 9.9 / 11.4 / 10.1.  SDDMM and FusedMM gain by short rows in a block; SpMM, which writes and adds a partial row per segment, loses by many segments from some 300 k units up.
  // With 80 and 160 / 64 and 96: 7 k, 406 k: SpMM, 16, 128 and 200 columns 7.9 / 9.6, 16.0 / 15.5, 24.2 / 27.5, SDDMM, 128 and 256: 19.3 / 14.5, 30.7 / 24.3, FusedMM's backward, 200:
  // 106.6 / 89.6; 12 k, 482 k: SpMM, 16, 128 and 200: 8.5 / 10.9, 17.6 / 20.3, 29.9 / 30.0, SDDMM, 128: 20.6 / 17.3, FusedMM's backward, 200: 126.5 / 105.8; over eight kinds of graphs (12 to 200
  // entries to a row, square, symmetric, wide, tall), 16 to 256 columns: 250 to 307 k units: SpMM the same, SDDMM 15 % less, FusedMM 2 and 6 % less, max 1 % more; 307 to 369 k: SpMM 1 % more, 12 %,
  // 1 and 7 %, max 1 % less; 369 to 451 k: 5 % more, 11 %, 1 and 6 %, 1 %; to 524 k: 4 % more, 8 %, 1 and 3 %, max 3 % more.  Segments of 80 with rows of 112 or 128, or
  // of 96 with 112, take from SDDMM and FusedMM what they give SpMM.  A graph seen once is built as fast; above, more segments cost the build more than they save (0.4 to 6 M entries: builds 20 % longer).
  const int seg_cap = 320;
  const int seg_min = share <= 28 ? 48 : share <= 128 ? 64 : 80;
  const int64_t auto_seg = share / 4 < seg_min ? seg_min : (share / 4 > seg_cap ? seg_cap : share / 4);
  const int auto_hub = seg_min < 80 ? 2 * seg_min - 32 : 2 * auto_seg > 512 ? 512 : (int)(2 * auto_seg);
  p.hub_t = env_int("ISP_HUB_THRESHOLD", auto_hub, 8, 512);
  p.seg_len = env_int("ISP_SEGMENT_LEN", (int)auto_seg, 8, 768);
  // Rows are cut into equal segments instead of at column bands on matrices of up to 1.3 M units, and with fewer than 64 Ki columns
  // up to 4 M: the segments' own order by first column is all the locality that they need, and bands leave about half as many again of
  // them (a band of 45 entries, chance included, is a whole segment of 80 and the start of another).  us at 32, 64, 128 and 256 columns with 32 bands / without: 12 k columns,
  // 1.5 M entries: SpMM 20.7 / 18.7, 27.5 / 26.3, 42.8 / 41.2, 79.8 / 79.4, FusedMM 25.8 / 22.8, 36.6 / 33.6, 59 / 55, 108 / 102, the build 82 / 57; 32 k, 4 M:
  // SpMM 38.4 / 37.2, 58.5 / 57.4, 99.6 / 99.2, 199 / 197, the build 58 / 49; 100 k, 1 M: SpMM 17.3 / 15.9, 25.7 / 25.3, 45.1 / 42.9, 80.7 / 78.8, SDDMM
  // 15.3 / 14.1, 22.6 / 22.4, 42.1 / 42.7, 87.4 / 88.2.  Of 36 graphs up to 1.3 M units (5 to 200 entries to a row, square, wide and tall) none takes longer
  // over all operations and widths (up to 12 % less, builds 2 to 41 %), but SDDMM takes 1 to 4 % longer from 256 columns up where there are many (54 k square, 646 k
  // entries 56.8 / 58.8, 98 k, 1.2 M 98.5 / 100.6, 165 k x 41 k, 1.1 M 114.5 / 117.6, 6.9 k x 27.7 k, 693 k 50.0 / 52.0; no more on the larger of them), the max backward from 200 up
  // 4 to 8 % (30 k, 1 M, 256 columns 107 / 115), and a wide or tall matrix gains nothing but
  // its build (41 k x 165 k, 1.2 M, 128 columns: SpMM 48.7 / 46.9, its transpose 59.2 / 60.0, SDDMM 55.0 / 55.9; 200: 102.7 / 104.9, 104.9 / 108.8, 108.9 / 112.0).
  // Beyond, up to 4 M units, narrow rows and the build gain and wide ones lose: 37 k, 3 M, SpMM, 128 columns 77.6 / 76.6, SDDMM 80.9 / 80.5, the max backward at 200 181.6 / 194.4, all of it 1 %
  // less, the build 232 / 194; 60 k, 2.8 M: 8 columns, SpMM 27.1 / 25.6, SDDMM 23.8 / 22.4, 200: SpMM 138 / 144, SDDMM 256 159 / 169, the max backward 244 / 266, all of it 1 % less, the build 225 / 191;
  // 95 k x 24 k, 2.3 M 1 % less, 140 k x 36 k, 3.5 M the same, 49 k, 4 M 1 % more (the build 261 / 225), and beyond: 50 k, 6 M: SpMM 56.0 / 53.5, 84.8 / 83.7, 147.5 / 150.3, 295 / 300,
  // SDDMM at 256 302 / 317; with more columns 99 k, 3 M, 196 columns 206 / 215; 121 k, 4.5 M, 176 columns 239 / 251.
  const int auto_bands = share <= 320 || (n_cols < (64 << 10) && share <= 1024) ? 1 : 32;
  int b = env_int("ISP_BANDS", auto_bands, 1, MAX_BANDS);
  while (b & (b - 1)) b &= b - 1;  // round down to a power of two
  p.bands = b;
  // (the lower limit bounds the number of segments, hence the partial-sum rows the workspace must hold)
  const int mp_lo = p.seg_len / 8 > 4 ? p.seg_len / 8 : 4;
  int mp = p.seg_len / 2 < 128 ? p.seg_len / 2 : 128;
  if (mp < mp_lo) mp = mp_lo;
  p.min_piece = env_int("ISP_MIN_PIECE", mp, mp_lo, 1 << 20);
  return p;
}

// Block cost of the derived matrix.  Its rows cost two units besides their entries, so a block of B units holds
// at most B / 2 rows and B may reach twice the ordinary 256 within the kernels' 256-row tables; its entries
// (fewer than B plus the longest row) must fit their 768-entry tables.
// One and a half times the ordinary block where the longest row leaves room for it (config 3: 384 units next to
// rows of up to 384 entries; measured 4.75 ms per SpMM against 4.81 at 256 and 4.76 at 512, where the segments
// have to shrink to 256 entries): every work item starts with a chain of dependent loads before its first
// gather, and fewer, larger items pay it less often.
inline int derived_block_cost(const partition_params& p1, int mid_t) {
  const int longest = mid_t > p1.seg_len ? mid_t : p1.seg_len;
  int dflt = p1.block_cost * 3 / 2;
  if (dflt > 768 - longest) dflt = 768 - longest;
  if (dflt < 16) dflt = 16;
  return env_int("ISP_PACKED_BLOCK", dflt, 16, 512);
}

inline partition_params cut_params(const partition_params& p1, int mid_t) {
  partition_params c = p1;
  c.hub_t = mid_t;
  const int room = 768 - derived_block_cost(p1, mid_t);  // longest row the derived matrix may have
  // (the ordinary partition's segment length also bounds the pieces here: 320 against 384 measured 4.65 / 4.64 ms
  // per SpMM on 2.4 M columns, 0.345 / 0.357 ms on 1 M columns at d = 64)
  if (c.seg_len > room) c.seg_len = room;
  // pieces of 64 entries or more, on up to 32 bands (measured on 2.4 M columns: smaller pieces fetch less but
  // pay it back in partial rows)
  c.min_piece = env_int("ISP_MIN_PIECE", 64, c.seg_len / 8 > 4 ? c.seg_len / 8 : 4, 1 << 20);
  return c;
}

inline partition_params derived_params(const partition_params& p1, const partition_params& cut) {
  partition_params d = p1;
  d.hub_t = cut.hub_t > cut.seg_len ? cut.hub_t : cut.seg_len;  // no row of the derived matrix is longer
  d.seg_len = d.hub_t;
  d.bands = 1;
  d.row_cost = 2;
  d.block_cost = derived_block_cost(p1, cut.hub_t);
  return d;
}

}  // namespace isp_part
