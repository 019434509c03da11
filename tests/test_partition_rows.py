"""Partial rows of the shared transpose, on the CPU: the sizes that the partitions are laid out by (csrc/partition_sizes.h)
against the pieces that the packed SpMM layout cuts, over row lengths on both sides of every step in the piece count."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include "partition_sizes.h"
using namespace isp_part;
int main() {
  const int64_t sizes[] = {65536, 70000, 100003, 400000};
  long checked = 0, beyond = 0;
  for (int64_t n : sizes)
    for (int64_t deg = 200; deg <= 3000; ++deg) {
      const int64_t nnz = n * deg;
      if (nnz < (8 << 20) || nnz > (256 << 20)) continue;  // (where the layout is chosen)
      const partition_params p1 = get_params(n, nnz, 4096, n), pc = cut_params(p1, 256);
      // columns spread evenly over the bands: every band holds a piece, as many segments as its length needs
      auto cut = [&](const partition_params& p) -> int64_t {
        if (deg <= p.hub_t) return 0;
        const int64_t br = hub_bands(deg, p), len = (deg + br - 1) / br;
        return n * br * ((len + p.seg_len - 1) / p.seg_len);
      };
      isp_csr A{};
      A.v.n_seg = (int32_t)cut(p1);
      A.partial_rows = max_segments(n, nnz, p1) + 1;  // what the handle's own scratch has
      const int64_t pieces = cut(pc);
      A.spmm_rows = pieces > A.v.n_seg ? pieces : A.v.n_seg;
      ++checked;
      beyond += pieces > A.partial_rows;
      const int64_t own = max_segments(n, nnz, pc) + 1;  // the scratch a partition of its own would have for the pieces
      if (isp_shared_rows(&A) < pieces || isp_shared_rows(&A) < A.v.n_seg || pieces > own || A.v.n_seg > A.partial_rows) {
        printf("rows %lld of %lld entries: %lld pieces, %d segments, %lld shared rows, %lld + %lld laid out\n", (long long)n,
               (long long)deg, (long long)pieces, A.v.n_seg, (long long)isp_shared_rows(&A), (long long)A.partial_rows,
               (long long)own);
        return 1;
      }
    }
  printf("%ld shapes, %ld with more pieces than rows of the ordinary partition\n", checked, beyond);
  return checked > 0 && beyond > 0 ? 0 : 1;  // (the lengths are there where the two differ)
}
"""


def test_shared_scratch_holds_the_pieces(tmp_path):
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__=1", "-I" + os.path.join(ROOT, "include"),
                           "-I" + os.path.join(ROOT, "paper_2403_14853_amd", "csrc"), "-isystem", "/opt/rocm/include",
                           str(src), "-o", str(exe)])
    env = {k: v for k, v in os.environ.items() if not k.startswith("ISP_")}
    res = subprocess.run([str(exe)], env=env, stdout=subprocess.PIPE, text=True)
    print(res.stdout)
    assert res.returncode == 0, res.stdout
