// Where a launch puts its hub rows together itself (hub_finish.h), and what it counts their segments in: host arithmetic only, so
// that the rule can be checked without a device.
#pragma once
#include "isp_internal.h"

namespace isp_dev {

constexpr int HF_SLICES = 2;     // counters per hub row: one per column slice of a launch
// Counters from one hub row's to the next: a line of 128 bytes each.  Segments that count in at one line are served one after the
// other, some 10 ns each, whichever row is theirs: 8 rows of 515 segments, SpMM, 16 columns, us with a fix-up launch / rows sharing a line / lines
// of their own 26.6 / 62.3 / 24.2, 128 columns 74 / 141 / 72; 20 rows of 138, 16 columns 13.5 / 21.8 / 10.9.
constexpr int HF_STRIDE = 32;

// Whether a launch finishes its hub rows itself: not where it has more than two segments for every wavefront slot.  The fix-up's
// wavefronts then have enough rows to fill the chip, and the launch spends longer in the chains (store, count, load) at the end
// of its segments.  us with the fix-up / without, segments in brackets: SpMM, 16 and 128 columns: 2 k rows, 20 k entries (52) 7.5 / 5.3, 9.1 / 6.6;
// 10 k, 300 k (2,523) 10.1 / 7.4, 16.1 / 14.0; 170 k, 1.7 M (6,583) 24.1 / 23.2, 68.4 / 67.9; 100 k, 4 M (8,192) 35.5 / 34.7, 112.1 /
// 111.8; 10 k, 1 M (13,911) 16.1 / 15.1, 31.3 / 31.4; 20 k, 3 M (16,000) 26.0 / 26.1, 72.8 / 72.7; 60 k, 18 M (72,304) 114.8 / 122.4, 380 / 380;
// FusedMM, 16 and 64 columns: 10 k, 300 k 12.3 / 9.3, 15.6 / 11.6; 20 k, 3 M 35.7 / 36.6, 56.5 / 56.5; 1 M, 17 M (39,440) 188 / 196, 375 / 373.
inline bool hf_few(const isp_csr* A, const isp_view& v) { return v.n_seg <= 2 * A->wave_slots; }
inline bool hf_pays(const isp_csr* A, const isp_view& v) { return v.hub_done && v.n_hub > 0 && hf_few(A, v); }

}  // namespace isp_dev
