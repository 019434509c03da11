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
// Nor where the longest row has more segments than a wavefront adds in a fix-up launch's time: the one that counts last adds the row alone,
// past the L2s, with nothing else left to run, where the fix-up has four wavefronts for it.  Of a wavefront's lane groups up to four
// work side by side, so the limit goes by the lanes per group (lpg).  us with the fix-up / without, one row of so many segments among 20 k (from 325: 50 k,
// 515: 200 k) of 8 entries, forward: 4 groups: SpMM, 16 columns 256 11.8 / 10.4, 452 16.6 / 15.8, 640 19.3 / 19.4, 64 columns 256 13.1 / 12.1, 640 29.1 / 26.1; FusedMM, 64 columns 256
// 14.6 / 14.0, 452 28.0 / 25.4, 16 columns 640 21.5 / 22.5;  2 groups: SpMM, 128 columns 103 17.0 / 16.6, 136 17.7 / 17.5, 196 18.4 / 19.5; FusedMM 76
// 18.5 / 17.9, 136 19.4 / 19.8;  1 group: SpMM, 200 columns 44 25.2 / 24.7, 76 26.1 / 25.9, 103 26.6 / 27.2; FusedMM 44 28.3 / 27.9, 76 29.3 / 29.5.
constexpr int hf_longest(int lpg) { return lpg <= ISP_WAVE / 4 ? 512 : lpg <= ISP_WAVE / 2 ? 128 : 64; }
inline bool hf_pays(const isp_csr* A, const isp_view& v, int lpg) {
  return v.hub_done && v.n_hub > 0 && hf_few(A, v) && A->longest_row_segs <= hf_longest(lpg);
}

}  // namespace isp_dev
