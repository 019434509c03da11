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
// work side by side, so the limit goes by the lanes per group (lpg; segments as row_segments counts them, 96 for
// the rows of 76 below).  us with the fix-up / without, one row of so many segments among 20 k (from 325: 50 k,
// 515: 200 k) of 8 entries, forward: 4 groups: SpMM, 16 columns 256 11.8 / 10.4, 452 16.6 / 15.8, 640 19.3 / 19.4, 64 columns 256 13.1 / 12.1, 640 29.1 / 26.1; FusedMM, 64 columns 256
// 14.6 / 14.0, 452 28.0 / 25.4, 16 columns 640 21.5 / 22.5;  2 groups: SpMM, 128 columns 103 17.0 / 16.6, 136 17.7 / 17.5, 196 18.4 / 19.5; FusedMM 76
// 18.5 / 17.9, 136 19.4 / 19.8;  1 group: SpMM, 200 columns 44 25.2 / 24.7, 76 26.1 / 25.9, 103 26.6 / 27.2; FusedMM 44 28.3 / 27.9, 76 29.3 / 29.5.
constexpr int hf_longest(int lpg) { return lpg <= ISP_WAVE / 4 ? 512 : lpg <= ISP_WAVE / 2 ? 128 : 96; }
inline bool hf_pays(const isp_csr* A, const isp_view& v, int lpg) {
  return v.hub_done && v.n_hub > 0 && hf_few(A, v) && A->longest_row_segs <= hf_longest(lpg);
}

// The min / max forward, whose fold of (value, position) pairs is longer than the sum's: up to a segment for every third wavefront slot, 32 segments
// to a row (96 with eight lanes to a group; as row_segments counts them), and only where the row blocks hold rows (of 33 entries to the hub threshold, on average) of half
// a segment and more: the segments, which start last, then don't end last, and the fold is hidden.  us with the fix-up / without: R-MAT, segments in
// brackets: 2 k rows, 20 k entries (48) 16 columns 11.9 / 9.7, 128 16.7 / 13.6; 20 k, 108 k (220) 13.5 / 11.3, 20.6 / 17.1; 10 k, 100 k (488) 64 13.1 / 11.6; 50 k, 300 k
// (897, the longest row 32) 64 19.8 / 16.6, 128 31.8 / 28.4; 5 k uniform rows of 50 and 40 of 1,300 (1,280, 32) 64 14.4 / 12.5, 128 18.4 / 17.9; 20 k, 100 k and one of 2,500 (44) 16 14.3 / 11.7, 64
// 16.3 / 15.7, 128 21.4 / 21.2, of 5,000 (64) 16 17.1 / 14.6, 128 23.9 / 27.6;  but without rows of such a length 20 k
// of 8 entries and 8 of 512 (64) 16 10.2 / 11.2, 128 18.2 / 19.2, of 2,511 (358) 128 22.8 / 26.4; 5 k, 40 k and 16 of 1,013 (258) 128 13.1 / 16.8; R-MAT 10 k, 300 k (2,526)
// 16 14.6 / 15.7, 128 21.2 / 26.8.
inline bool hf_minmax_pays(const isp_csr* A, const isp_view& v, int lpg) {
  const isp_csr_info_t& I = A->info;
  return hf_pays(A, v, lpg) && 3 * (int64_t)v.n_seg <= A->wave_slots && A->longest_row_segs <= (lpg <= 8 ? 96 : 32) && I.bin_rows[3] > 0 &&
         2 * I.bin_nnz[3] >= v.seg_len * I.bin_rows[3];
}

}  // namespace isp_dev
