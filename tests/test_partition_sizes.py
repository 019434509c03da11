"""Sizes of the work partitions, on the CPU (csrc/partition_sizes.h): on both sides of the numbers of units per wavefront slot where
they change."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HEAD = r"""
#include <stdio.h>
#include "partition_sizes.h"
using namespace isp_part;
constexpr int64_t SLOTS = 4096;
#define FAIL(...) do { printf(__VA_ARGS__); return 1; } while (0)
// the sizes of a matrix of that many rows and columns with `share` units per slot, `more` units on top
static partition_params sizes(int64_t share, int64_t more, int64_t n, int64_t n_cols) { return get_params(n, share * SLOTS + more - n, SLOTS, n_cols); }
"""


def run(tmp_path, program):
    src, exe = tmp_path / "sizes.cpp", tmp_path / "sizes"
    src.write_text(HEAD + program)
    subprocess.check_call(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__=1", "-I" + os.path.join(ROOT, "include"),
                           "-I" + os.path.join(ROOT, "paper_2403_14853_amd", "csrc"), "-isystem", "/opt/rocm/include",
                           str(src), "-o", str(exe)])
    env = {k: v for k, v in os.environ.items() if not k.startswith("ISP_")}
    res = subprocess.run([str(exe)], env=env, stdout=subprocess.PIPE, text=True)
    print(res.stdout)
    assert res.returncode == 0, res.stdout


def test_segments_and_longest_rows_of_a_block(tmp_path):
    run(tmp_path, r"""
int main() {
  struct { int64_t share, more; int hub, seg; } want[] = {{1, 0, 64, 48}, {28, 0, 64, 48}, {28, 1, 96, 64}, {128, 0, 96, 64}, {128, 1, 160, 80},
                                                          {323, 0, 160, 80}, {324, 0, 162, 81}, {1280, 0, 512, 320}, {9000, 0, 512, 320}};
  for (auto& w : want) {
    const partition_params p = sizes(w.share, w.more, 3000, 3000);
    if (p.hub_t != w.hub || p.seg_len != w.seg) FAIL("%lld + %lld units: %d, %d\n", (long long)w.share, (long long)w.more, p.hub_t, p.seg_len);
  }
  return 0;
}
""")


def test_equal_segments_or_column_bands(tmp_path):
    run(tmp_path, r"""
int main() {
  struct { int64_t share, more, n, n_cols; int bands; } want[] = {
    {320, 0, 70000, 70000, 1}, {320, 1, 70000, 70000, 32}, {320, 0, 3000, 2000000, 1}, {320, 0, 600000, 3000, 1}, {321, 0, 65535, 65535, 1}, {321, 0, 3000, 65536, 32},
    {400, 0, 100000, 65535, 1}, {1024, 0, 65535, 65535, 1}, {1024, 1, 65535, 65535, 32}, {1024, 0, 100, 65536, 32}, {1024, 1, 12000, 12000, 32}, {5000, 0, 5000, 5000, 32}};
  for (auto& w : want) {
    const partition_params p = sizes(w.share, w.more, w.n, w.n_cols);
    if (p.bands != w.bands) FAIL("%lld + %lld units, %lld x %lld: %d bands\n", (long long)w.share, (long long)w.more, (long long)w.n, (long long)w.n_cols, p.bands);
  }
  return 0;
}
""")


def test_bounds_hold_the_segments(tmp_path):
    """What the workspace is laid out for, against rows that are all of one length: as many segments as such rows can have, with equal segments and with bands,
    whose pieces may all end in a short one."""
    run(tmp_path, r"""
int main() {
  long equal = 0, banded = 0;
  for (int64_t share : {1, 8, 28, 29, 64, 65, 200, 320, 321, 400, 512, 700, 1024, 1025, 1400, 5000})
    for (int64_t n_cols : {100, 3000, 32768, 65535, 65536, 2000000})
      for (int64_t per : {65, 97, 128, 129, 161, 320, 321, 513, 1000, 5000, 70000}) {
        const int64_t units = share * SLOTS, n = units / (per + 1), nnz = n * per;
        if (n == 0) continue;
        const partition_params p = get_params(n, nnz, SLOTS, n_cols);
        if (per <= p.hub_t) continue;
        const int64_t rows = max_hub_rows(n, nnz, p), most = max_segments(n, nnz, p);
        const int64_t each = p.bands == 1 ? (per + p.seg_len - 1) / p.seg_len : per / p.seg_len + hub_bands(per, p);
        if (rows < n || most < n * each) FAIL("%lld rows of %lld, %lld columns, %d bands: %lld segments, laid out for %lld\n", (long long)n, (long long)per, (long long)n_cols, p.bands, (long long)(n * each), (long long)most);
        (p.bands == 1 ? equal : banded) += share > 320 && n_cols < 65536;
      }
  return equal > 0 && banded > 0 ? 0 : 1;  // (both where the number of columns decides)
}
""")
