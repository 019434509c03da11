// How many lanes hold a row, and with how many vectors each, in the kernels whose choice follows from sizes alone: host arithmetic, so that the
// rules can be checked without a device.
#pragma once
#include <stdint.h>

namespace isp_dev {

// The passes of FusedMM: forward; the row and column passes that a directed graph's backward takes; the one of a symmetric pattern's.
enum class fused_pass { forward, two_pass, one_pass };

// Four lanes hold a row of up to 16 columns, and a step serves 16 entries instead of 8, half of whose lanes were idle.  On few entries a launch is the time
// of its chains.  With hub rows (n_hub of them) that is a segment's, which 16 runs finish in half the steps; without, the longer start of 16 runs.

// SDDMM (w columns in this launch): everywhere with hub rows, else from 64 Ki entries.  us with 8 / 4 lanes, 8 columns: R-MAT: 800 rows, 8 k entries 4.1 / 3.8; 4 k, 36 k: 4.2 / 4.0; 12 k, 100 k:
// 4.6 / 4.3; 40 k, 300 k: 7.1 / 5.7; 100 k, 1 M: 13.0 / 10.5; 60 k, 2.8 M: 27.8 / 22.6, 16 columns 28.1 / 24.1; 200 k, 8 M: 75.9 / 63.8; 230 k, 60 M: 469 / 398; uniform: 4 k, 36 k:
// 4.15 / 4.24; 9 k, 60 k: 4.37 / 4.48; 3 k, 64 k: 4.35 / 4.32; 12 k, 100 k: 4.7 / 4.6; 8 k, 180 k: 5.5 / 4.9; 500 k, 8 M: 118.4 / 119.6.
inline bool sddmm_four_lanes(int64_t w, int64_t nnz, int64_t n_hub) { return w <= 16 && (n_hub > 0 || nnz >= 64 << 10); }

// FusedMM: from 64 Ki entries with hub rows, else from 120 Ki (forward) and 96 Ki (backward).  us with 8 / 4 lanes, 8 columns, forward and backward: R-MAT, directed: 4 k, 36 k: 5.4 / 5.6,
// 12.2 / 12.1; 9 k, 60 k: 6.0 / 6.0, 13.6 / 13.1; 6 k, 80 k: 6.0 / 5.8, 14.0 / 12.8; 12 k, 100 k: 6.3 / 6.3, 14.9 / 13.5; 3.8 k, 120 k: 6.2 / 5.8, 14.9 / 12.9; 8 k, 180 k: 7.0 / 6.4,
// 17.1 / 14.9; 40 k, 300 k: 9.7 / 8.2, 24.8 / 20.2; 100 k, 1 M: 17.9 / 14.7, 49.5 / 41.3; 60 k, 2.8 M: 35.2 / 28.0, 96.6 / 77.5 (16 columns 36.0 / 29.8, 99.1 / 81.0;
// symmetric 65.4 / 47.3); 200 k, 8 M: 91.7 / 73.5, 250 / 199; 230 k, 60 M: 521 / 413, 1489 / 1140; uniform: 4 k, 36 k: 5.0 / 5.5, 10.9 / 11.7; 6 k, 80 k: 5.5 / 6.2, 12.5 / 13.1; 12 k, 100 k:
// 5.7 / 5.9, 13.2 / 12.5; 3.8 k, 120 k: 6.2 / 6.6, 14.3 / 14.1; 20 k, 130 k: 6.0 / 5.7, 14.2 / 12.8; 30 k, 200 k: 6.7 / 6.0, 16.6 / 14.1; 500 k, 8 M, which waits for its gathers: 117.2 /
// 116.6, 385 / 386.
inline bool fused_four_lanes(fused_pass pass, int64_t d, int64_t nnz, int64_t n_hub) {
  return d <= 16 && nnz >= (n_hub > 0 ? 64 << 10 : pass == fused_pass::forward ? 120 << 10 : 96 << 10);
}

// The min / max backward (w columns in this launch, hub rows of the transpose): below 32 Mi entries with hub rows, else from 256 Ki.  us with 8 / 4 lanes, 8 and 16 columns: R-MAT: 4 k, 36 k: 11.0 / 10.7,
// 11.0 / 10.9; 3.8 k, 120 k: 11.6 / 11.5, 12.1 / 11.8; 8 k, 180 k: 12.7 / 12.2, 12.4 / 12.2; 60 k, 500 k: 19.4 / 18.7, 20.9 / 20.5; 400 k, 4 M: 66.9 / 64.4, 76.7 / 75.4; 1 M, 17 M: 264 / 253,
// 292 / 281; but 230 k, 60 M: 534 / 539, 581 / 584; uniform: 4 k, 36 k: 10.7 / 11.2, 10.4 / 11.4; 8 k, 180 k: 11.8 / 12.5, 11.8 / 12.5; 12 k, 300 k: 12.4 / 12.6, 12.8 / 12.8; 30 k, 400 k:
// 13.6 / 13.3, 16.3 / 15.9.
inline bool select_four_lanes(int64_t w, int64_t nnz, int64_t n_hub) { return w <= 16 && nnz < (32 << 20) && (n_hub > 0 || nnz >= (256 << 10)); }

// FusedMM beyond 32 columns: one or two float4 per lane.  Two halve the lanes per dot product, so a step covers twice the entries with one
// lane-reduction stage and one evaluation of the edge function less per entry, but hold twice the registers and load
// the row operand with every step.  Large matrices have one everywhere (128 columns, us, one / two: forward on 2.4 M entries
// 113 / 116, on 16.9 M 823 / 858, backward 240 / 266, 2830 / 2936) except where rows average 200 entries and nearly
// all work lies in hub segments (115 M entries: 3077 / 2764, backward 7697 / 6860).  With as few entries as the chip's wavefronts finish in a few rounds
// the length of their runs counts, and two it is: beyond 128 columns below 1 Mi entries, beyond 64 below 3/4 Mi - in a directed graph's
// backward, whose passes take two entries at a time with one vector and have too short a ring for it with two, only with operands that the caches
// hold (6 MB; from 129 to 160 columns, where two vectors gain most, 48 MB); in a symmetric pattern's from 512 Ki entries on only with operands of 20 MB, beyond 160 columns 32 MB.
// us, one (in pairs where the pass has them) / two:
//   forward: uniform, 7 k rows, 406 k entries: 72 columns 19.7 / 18.0, 144 34.8 / 25.1, 256 35.9 / 30.8; 30 k, 600 k: 26.9 / 26.4, 53.3 / 49.5, 85.9 / 88.4; 50 k, 1 M: 144 102 / 110; R-MAT, 15 k,
//   600 k: 29.9 / 25.5, 53.4 / 43.9, 54.2 / 49.4; 80 k, 800 k: 36.9 / 36.1, 67.4 / 58.2, 90.5 / 83.5 (100 39.5 / 42.7); 68 k, 1.3 M: 128 60.0 / 59.8, 256 113.6 / 117.9;
//   two passes: uniform, 7 k, 406 k: 72 (2 MB) 58.1 / 52.7, 128 (3.6) 58.9 / 57.7, 200 (5.6) 120.6 / 120.6, 256 (7.2) 133 / 143; 30 k, 600 k: 72 (8.6) 92.0 / 97.0, 128 (15) 128 / 139, 256 265 / 284;
//   R-MAT, 3.8 k, 120 k: 128 27.0 / 26.5, 144 44.1 / 41.2; 12 k, 482 k: 72 (3.5) 60.8 / 60.6, 128 (6.1) 61.7 / 63.4, 200 (9.6) 105 / 109; 15 k, 600 k: 144 (8.6) 144 / 131, 256 (15) 156 / 159; 60 k,
//   600 k: 72 (17) 79.4 / 85.4, 128 92.6 / 101.3, 144 (35) 147 / 144, 256 215 / 233; 80 k, 800 k: 100 (32) 124 / 137, 144 (46) 202 / 195, 256 281 / 300; 150 k, 750 k: 144 (86) 213 / 222; uniform, 60 k,
//   600 k: 144 (35) 186 / 195;
//   one pass: R-MAT, 12 k, 482 k: 72 45.0 / 34.6, 128 45.4 / 36.7, 256 77.6 / 71.1; 15 k, 600 k: 128 (7.7 MB) 60.8 / 52.0, 200 (12) 115 / 99, 256 (15) 117 / 108; 30 k, 600 k, uniform: 128 (15) 83.5 / 82.8, 256 (31)
//   177 / 169; 60 k, 800 k: 144 136 / 122; 100 k, 500 k: 128 (51) 75.2 / 69.0, 256 (102) 162 / 151; but 60 k, 600 k: 72 (17) 57.5 / 50.7, 100 (24) 58.9 / 64.2, 128 60.9 / 66.0, 200 (48) 125 / 131; 133 k, 1.04 M: 144
//   178 / 159, 256 265 / 278; 200 k, 1 M: 200 255 / 273.  (Beyond these numbers of entries two would still gain on small operands: 20 k, 900 k: 72 82.4 / 59.5, 128 83.0 / 63.0.)
// live_rows: rows with entries.
inline bool fused_two_vectors(fused_pass pass, int64_t d, int64_t n_rows, int64_t live_rows, int64_t nnz) {
  if (live_rows > 0 && nnz >= 200 * live_rows) return true;
  const bool wide = d > 160, between = d > 128 && !wide;
  if (pass == fused_pass::two_pass && n_rows * d > (between ? 12 << 20 : 3 << 19)) return false;
  if (pass == fused_pass::one_pass && !between && nnz >= (512 << 10) && n_rows * d > (wide ? 8 << 20 : 5 << 20)) return false;
  return d > 128 ? nnz < (1 << 20) : d > 64 && nnz < (3 << 18);
}

}  // namespace isp_dev
