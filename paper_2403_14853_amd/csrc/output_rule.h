// Which outputs SpMM writes past the caches: host arithmetic only, so that the rule can be checked without a device.
#pragma once
#include <stdint.h>

namespace isp_dev {

// From 160 MB on.  The launch itself gains at any size from some 64 MB, as its output no longer pushes out of the Infinity Cache (256 MB) what it
// still gathers; but whoever reads the output next then finds nothing of it there, and up to half the cache's size that costs as much or more.  us with
// ordinary / these stores, R-MAT, 8 to 12 entries a row; the launch alone, with a dense product on its output, a training step of a two-layer GCN of that hidden width:
//    32 columns:  66 MB 54.5 / 53.8, 135 / 142, 2455 / 2793;  130 MB 105 / 102, 218 / 214, 4223 / 4229;  160 MB 135 / 132, 262 / 259, 5231 / 5208
//    64:          66 MB 57.1 / 56.4, 114 / 124, 1586 / 1750;  90 MB 80.5 / 79.7, 158 / 171, 2226 / 2387;  130 MB 114 / 112, 245 / 252, 2912 / 2935;
//                160 MB 149 / 144, 317 / 313, 3654 / 3635;  300 MB 301 / 291, 473 / 470
//   100:          90 MB 103 / 101, 224 / 232, 2109 / 2175;  160 MB 203 / 199, 401 / 397, 4099 / 4088
//   128:          90 MB 80.6 / 80.5, 145 / 146, 1623 / 1690;  130 MB 115 / 113, 261 / 254, 2211 / 2173;  160 MB 150 / 144, 319 / 312, 2744 / 2705;  300 MB 321 / 296, 542 / 530
// Rows narrower than a line (their parts are stored by several lane groups), alone and with the product: 8 columns 66 MB 114 / 112, 261 / 273; 160 MB 309 / 292, 677 / 677; 300 MB 611 / 573,
// 1314 / 1291; 16 columns 160 MB 159 / 152, 407 / 409; 24 columns 154 / 149, 349 / 344.  Launches on the small LDS tables (run_stream.h), whose operand the L2s hold,
// store as ever.
inline bool streams_output(int64_t rows, int64_t d) { return rows * d >= (int64_t)40 << 20; }

// The packed layout's partial rows, `pieces` of them and `width` columns in this launch: from 96 MB on, of which the fix-up would find less in
// the caches than they cost the gathers.  us with ordinary / these stores: 233 k columns, 115 M entries, some 370 k pieces, 128 columns (190 MB) 2438 / 2413,
// 602 in five launches 11960 / 11865; 2.4 M, 124 M: 4586 / 4567; 800 k, 40 M, 247 k pieces: 50 columns (49 MB) 763 / 760, 100 (99 MB) 1431 / 1402, 128 1377 /
// 1366; 120 k, 40 M, 305 k: 32 (39 MB) 281 / 285, 64 (78 MB) 469 / 470, 100 (122 MB) 838 / 835; 100 k, 16 M, 112 k: 32 122 / 124, 64 (29 MB) 202 / 204, 128 (57 MB) 374 / 376.
inline bool streams_pieces(int64_t pieces, int64_t width) { return pieces * width >= (int64_t)24 << 20; }

}  // namespace isp_dev
