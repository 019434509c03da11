"""Places of SpMM's copies of ragged operands in the workspace, on the CPU (csrc/stage_rule.h): over rooms of every relative
size a copy lies in a room, the one for the static-scratch entry point only where no other call writes, and the two apart;
and the workspace that the sizes ask for always holds the copies where the packed layout exists."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include "stage_rule.h"
using namespace isp_part;
using isp_stage::room;

static char* at(int64_t kib) { return (char*)((1 << 20) + kib * 1024); }
static bool in(const float* p, size_t b, char* lo, char* hi) { return (char*)p >= lo && (char*)p + b <= hi; }
static bool apart(const float* p, const float* q, size_t b) { return (char*)p + b <= (char*)q || (char*)q + b <= (char*)p; }
#define FAIL(...) do { printf(__VA_ARGS__); return 1; } while (0)

int main() {
  long copies = 0, both = 0, shared = 0;
  // rows [0, busy) of a partition are written by other calls, of which a SpMM writes the first `used`; `cut` idle rows elsewhere
  for (int64_t n_cols : {100000, 200000})
    for (int64_t cut = 0; cut <= 320000; cut += 40000)
      for (int64_t end = 0; end <= 320000; end += 20000)
        for (int64_t busy = 0; busy <= end; busy += 20000)
          for (int64_t used : {(int64_t)0, busy / 4, busy})
            for (int64_t rows : {100, 40000}) {
              isp_csr A{};
              A.v.n_cols = n_cols; A.v.nnz = 40 * n_cols; A.spmm_rows = rows;
              const size_t b = isp_stage::wanted(n_cols, A.v.nnz);
              room r[3] = {{at(1000000), at(1000000 + cut)}, {at(busy), at(end)}, {at(used), at(end)}};
              isp_stage::place(&A, r + (cut ? 0 : 1), cut ? 3 : 2);
              const bool fits = (size_t)cut * 1024 >= b || (size_t)(end - used) * 1024 >= b;
              if (A.stages != fits || (A.stage != nullptr) != fits || (fits && A.stage_cols != 128)) FAIL("place missed\n");
              if (!fits) { if (A.static_stage) FAIL("static copy alone\n"); continue; }
              ++copies;
              if (!in(A.stage, b, at(1000000), at(1000000 + cut)) && !in(A.stage, b, at(used), at(end))) FAIL("copy outside\n");
              shared += !in(A.stage, b, at(1000000), at(1000000 + cut)) && !in(A.stage, b, at(busy), at(end));
              if (!A.static_stage) continue;
              ++both;
              if (rows > ISP_STATIC_SCRATCH_ROWS) FAIL("static copy of a handle that the entry point refuses\n");
              if (!in(A.static_stage, b, at(1000000), at(1000000 + cut)) && !in(A.static_stage, b, at(busy), at(end)))
                FAIL("static copy where other calls write\n");
              if (!apart(A.stage, A.static_stage, b)) FAIL("copies overlap\n");
            }
  if (!copies || !both || !shared) FAIL("%ld %ld %ld\n", copies, both, shared);
  // with the packed layout the rows of the ordinary partition and what is added always hold the copies
  for (int64_t n : {65536, 100003, 262144, 1000000, 2449029, 8000000})
    for (int64_t per = 4; per <= 4000; per += per / 4 + 1) {
      const int64_t nnz = n * per;
      if (nnz < (8 << 20) || nnz > (256 << 20)) continue;
      const partition_params p1 = get_params(n, nnz, 4096, n);
      const size_t rows = (size_t)(max_segments(n, nnz, p1) + 1) * 1024, own = isp_stage::own_bytes(n, nnz, rows, true);
      if (rows + own < isp_stage::wanted(n, nnz)) FAIL("no place: %lld x %lld\n", (long long)n, (long long)per);
    }
  for (int ld = 1; ld <= 140; ++ld)  // lines touched, row by row
    for (int w = 1; w <= ld; w += 3)
      for (uintptr_t at : {(uintptr_t)0, (uintptr_t)4, (uintptr_t)64, (uintptr_t)(4096 + 124)}) {
        int64_t sum = 0;
        for (int r = 0; r < 32; ++r) {
          const uintptr_t first = at + (uintptr_t)r * ld * 4, last = first + (uintptr_t)w * 4 - 1;
          sum += (int64_t)(last / 128 - first / 128 + 1);
        }
        if (isp_stage::line_sum(at, ld, w) != sum) FAIL("lines of %d floats, pitch %d\\n", w, ld);
      }
  // from 128 columns up a copy changes the launches, hence the order of the sums: X's address has no say in it, but where
  // rows are whole lines and run 128 columns at a time with and without
  long by_base = 0;
  for (int d = 12; d <= 640; ++d)
    for (int64_t ld = d; ld <= d + 24; ++ld)
      for (uintptr_t at = 4; at < 128; at += 4)
        if (isp_stage::operand_lines(4096 + at, ld, d, 256, 100000) != isp_stage::operand_lines(4096, ld, d, 256, 100000)) {
          if (d >= 128 && ld % 32 != 0) FAIL("%d columns, pitch %d, base %d\n", d, (int)ld, (int)at);
          ++by_base;
        }
  if (!by_base) FAIL("no call looks at the address\n");
  // a copy's rows begin at lines in every tile
  for (int d = 4; d <= 640; ++d) {
    int64_t sum = d < 128 ? (d + 31) / 32 : d / 128 * 4 + (d % 128 == 0 ? 0 : d % 128 < 4 ? 1 : (d % 128 + 31) / 32);
    if (isp_stage::copied_lines(d) != 32 * sum) FAIL("copied lines of %d columns\n", d);
  }
  for (int d : {257, 258, 259, 385, 387})  // (measured: 4 to 14 % faster with copies)
    if (!isp_stage::call_pays({20000000, 200000, d, d, isp_stage::operand_lines(0, d, d, 256, 200000), isp_stage::copied_lines(d), true, false, false}))
      FAIL("%d columns are not copied\n", d);
  // the rule on calls whose both sides are measured: packed X of d columns, `lines` of it per row and in its copy
  struct { int64_t n, nnz; int d, long_rows; bool pays; } calls[] = {
      {500000, 16500000, 500, 0, false}, {500000, 16500000, 602, 0, false}, {500000, 22000000, 602, 0, true}, {1000000, 33000000, 500, 0, true},
      {232965, 114600001, 602, 0, true}, {233000, 115000000, 100, 0, false}, {1000000, 40000000, 12, 0, true}, {1000000, 40000000, 9, 0, false},
      {350000, 105000000, 17, 1, false}, {350000, 105000000, 17, 0, true}, {350000, 105000000, 22, 1, true}, {350000, 105000000, 13, 1, true}};
  for (auto& q : calls) {
    int64_t lines = 0, copied = 0;
    for (int k = 0; k < q.d; k += 256) lines += isp_stage::line_sum(4 * k, q.d, q.d - k < 256 ? q.d - k : 256);
    for (int k = 0; k < q.d; k += 128) copied += isp_stage::line_sum(0, 32, q.d - k < 128 ? q.d - k : 128);
    if (isp_stage::call_pays({q.nnz, q.n, q.d, q.d, lines, copied, true, q.n >= 512 << 10, q.long_rows != 0}) != q.pays)
      FAIL("%d columns of %lld\\n", q.d, (long long)q.n);
  }
  struct { int64_t n, nnz; int d; bool pays; } sliced[] = {
      {524300, 17000000, 200, false}, {524300, 17000000, 500, false}, {524300, 17000000, 140, true}, {560000, 20000000, 200, false}, {560000, 20000000, 602, true},
      {640000, 21000000, 200, false}, {640000, 21000000, 301, true}, {800000, 26000000, 200, true}, {1400000, 46000000, 500, true},
      {881974, 29733124, 592, false}, {1106926, 36734308, 304, false}, {1060161, 36415778, 208, false}, {1400000, 70000000, 592, true}, {1000000, 40000000, 301, true}};
  for (auto& q : sliced)
    if (isp_stage::call_pays({q.nnz, q.n, q.d, q.d, isp_stage::operand_lines(0, q.d, q.d, 256, q.n), isp_stage::copied_lines(q.d), true, true, false}) != q.pays)
      FAIL("two slices: %d columns of %lld\n", q.d, (long long)q.n);
  struct { int64_t n, nnz; int d; bool pays; } uniform[] = {
      {91342, 8901716, 18, false}, {75751, 12442518, 18, false}, {114609, 9299487, 17, false}, {166803, 14124212, 12, false}, {84990, 12035986, 13, true},
      {91342, 8901716, 24, true}, {183756, 11407391, 18, true}, {221850, 24848037, 12, true}};
  for (auto& q : uniform)
    if (isp_stage::call_pays({q.nnz, q.n, q.d, q.d, isp_stage::operand_lines(0, q.d, q.d, 256, q.n), isp_stage::copied_lines(q.d), false, false, true}) != q.pays)
      FAIL("equally long rows: %d columns of %lld\n", q.d, (long long)q.n);
  for (int d : {272, 304, 528, 560, 592, 140, 301, 602})  // (five of half lines, three of any)
    for (int even : {0, 1}) {
      const bool pays = isp_stage::call_pays({8500000, 98496, d, d, isp_stage::operand_lines(0, d, d, 256, 98496), isp_stage::copied_lines(d), false, true, even != 0});
      if (pays != (even || d == 140 || d == 301 || d == 602)) FAIL("hub rows %d: %d columns\n", !even, d);
    }
  for (int w = 1, last = 0; w <= 128; ++w) {  // an alias for max_d columns has room for every narrower call
    const int p = isp_stage::pitch(w);
    if (p < w || p < last || p > isp_stage::pitch_up_to(w, true) + (w < 4 ? 8 : 0)) FAIL("pitch of %d\n", w);
    last = p;
  }
  return 0;
}
"""


def test_places(tmp_path):
    src, exe = tmp_path / "places.cpp", tmp_path / "places"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__=1", "-I" + os.path.join(ROOT, "include"),
                           "-I" + os.path.join(ROOT, "paper_2403_14853_amd", "csrc"), "-isystem", "/opt/rocm/include",
                           str(src), "-o", str(exe)])
    env = {k: v for k, v in os.environ.items() if not k.startswith("ISP_")}
    res = subprocess.run([str(exe)], env=env, stdout=subprocess.PIPE, text=True)
    assert res.returncode == 0, res.stdout
