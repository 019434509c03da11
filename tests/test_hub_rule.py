"""Hub rows put together by the launch of their segments, on the CPU (csrc/hub_rule.h): what their counters share, and which launches
do it."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HEAD = r"""
#include <stdio.h>
#include "hub_rule.h"
#include "partition_sizes.h"
using namespace isp_dev;
using namespace isp_part;
#define FAIL(...) do { printf(__VA_ARGS__); return 1; } while (0)
"""


def _run(tmp_path, program):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(HEAD + program)
    subprocess.check_call(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__=1", "-I" + os.path.join(ROOT, "include"),
                           "-I" + os.path.join(ROOT, "paper_2403_14853_amd", "csrc"), "-isystem", "/opt/rocm/include",
                           str(src), "-o", str(exe)])
    env = {k: v for k, v in os.environ.items() if not k.startswith("ISP_")}
    res = subprocess.run([str(exe)], env=env, stdout=subprocess.PIPE, text=True)
    print(res.stdout)
    assert res.returncode == 0, res.stdout


def test_counters_share_no_line(tmp_path):
    """Atomics on one line are served one after the other: a hub row's counters lie on a line that no other row's touch."""
    _run(tmp_path, r"""
int main() {
  if (HF_STRIDE * sizeof(unsigned) % 128 != 0) FAIL("rows share lines\n");  // (the first counter lies on a line: offsets are multiples of 256)
  if (HF_SLICES > HF_STRIDE) FAIL("rows overlap\n");
  return 0;
}
""")


def test_long_rows_keep_the_fix_up(tmp_path):
    """One wavefront adds the row that counts last, the fix-up's workgroup four times as fast: a matrix with a row of hundreds or
    thousands of segments, few as they are together, is left to the fix-up, the sooner the fewer lane groups share the row."""
    _run(tmp_path, r"""
int main() {
  unsigned done = 0;
  int finished = 0, left = 0;
  for (int64_t deg = 161; deg <= 600000; deg += deg / 7 + 1) {  // one such row among 20,000 of 8 entries
    const int64_t nnz = 160000 + deg;
    const partition_params p = get_params(20001, nnz, 4096, 20001);
    isp_csr A{};
    A.wave_slots = 4096;
    A.longest_row_segs = (int32_t)row_segments(deg, p);
    A.v.n_hub = 1;
    A.v.n_seg = A.longest_row_segs;
    if (A.v.n_seg > 8192) break;
    // (the estimate: full segments at least, at most three more to a band)
    if (A.v.n_seg < deg / p.seg_len || A.v.n_seg > deg / p.seg_len + 3 * p.bands) FAIL("%d segments of %lld\n", A.v.n_seg, (long long)deg);
    for (int lpg : {4, 8, 16, 32, 64}) {
      const int limit = lpg == 64 ? 96 : lpg == 32 ? 128 : 512;
      if (hf_pays(&A, A.v, lpg)) FAIL("without counters\n");
      A.v.hub_done = &done;
      const bool pays = hf_pays(&A, A.v, lpg);
      A.v.hub_done = nullptr;
      if (pays != (A.v.n_seg <= limit)) FAIL("%d lanes, %d segments: %d\n", lpg, A.v.n_seg, (int)pays);
      (pays ? finished : left) += 1;
    }
    if (!hf_few(&A, A.v)) FAIL("the order of the sums follows the segments of all rows\n");
  }
  printf("%d finished, %d left\n", finished, left);
  return finished > 20 && left > 20 ? 0 : 1;
}
""")


def test_min_max_keeps_the_fix_up_where_nothing_hides_the_fold(tmp_path):
    """Hub rows among rows too short for any row block to run as long as a segment, or of many segments."""
    _run(tmp_path, r"""
int main() {
  unsigned done = 0;
  isp_csr A{};
  A.wave_slots = 4096;
  A.v.hub_done = &done;
  A.v.n_hub = 8;
  A.v.n_seg = 64;
  A.v.seg_len = 80;
  A.longest_row_segs = 8;
  if (hf_minmax_pays(&A, A.v, 16)) FAIL("no rows of 33 entries and more\n");
  A.info.bin_rows[3] = 87;
  A.info.bin_nnz[3] = 87 * 35;
  if (hf_minmax_pays(&A, A.v, 16)) FAIL("rows of 35 entries\n");
  A.info.bin_nnz[3] = 87 * 40;
  for (int lpg : {8, 16, 32})
    for (int n : {1, 8, 32, 33, 96, 97, 500}) {
      A.longest_row_segs = n;
      if (hf_minmax_pays(&A, A.v, lpg) != (n <= (lpg == 8 ? 96 : 32))) FAIL("%d lanes, %d segments\n", lpg, n);
    }
  A.longest_row_segs = 8;
  A.v.n_seg = 1365;
  if (!hf_minmax_pays(&A, A.v, 32)) FAIL("a segment for every third slot\n");
  A.v.n_seg = 1366;
  if (hf_minmax_pays(&A, A.v, 32)) FAIL("too many segments\n");
  return 0;
}
""")
