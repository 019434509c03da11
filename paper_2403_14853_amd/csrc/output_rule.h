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

// The packed layout's partial rows, `pieces` of them and `width` columns in this launch: from 88 MB on, of which the fix-up would find less in
// the caches than they cost the gathers.  us with ordinary / these stores, MB in brackets: 233 k columns, 115 M entries, 863 k pieces: 48 columns (166) 1203 / 1197, 64 (221) 1217 / 1210,
// 68 (235) 1917 / 1907; 800 k, 40 M, 247 k pieces: 88 (87) 1191 / 1181, 92 (91) 1168 / 1159, 96 (95) 1046 / 1040, 100 (99) 1394 / 1389, with values 1419 / 1415, 128 (127) 1318 / 1307;
// 120 k, 40 M, 305 k: 64 (78) 427.0 / 426.1, 76 (93) 689.6 / 688.6, 100 (122) 806 / 802; 1.2 M, 60 M, 366 k: 64 (94) 1026 / 1018, 72 (106) 1605 / 1595; 400 k, 30 M, 194 k: 120 (93) 1016 /
// 1014.  Below, matrices of many columns still gain (800 k: 80 (79) 1007 / 996) and of few lose (100 k, 16 M, 112 k: 150 (67) 501.8 / 503.4, 192 (86) 555.3 / 558.5, where 256 (114)
// loses too, 728.7 / 731.2).
inline bool streams_pieces(int64_t pieces, int64_t width) { return pieces * width >= 22000000; }

}  // namespace isp_dev
