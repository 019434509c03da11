"""Outputs that SpMM writes past the caches, on the CPU (csrc/output_rule.h): not those that the Infinity Cache keeps for their reader."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <initializer_list>
#include <stdio.h>
#include "output_rule.h"
int main() {
  for (int64_t d : {1, 8, 37, 128, 602}) {
    const int64_t mb = (1 << 18) / d + 1;  // rows of a megabyte
    for (int64_t n : {1, 64, 90, 128, 150, 159})
      if (isp_dev::streams_output(n * mb - n, d)) { printf("%lld MB, %lld columns\n", (long long)n, (long long)d); return 1; }
    for (int64_t n : {160, 300, 5000})
      if (!isp_dev::streams_output(n * mb, d)) { printf("%lld MB, %lld columns: not\n", (long long)n, (long long)d); return 1; }
  }
  return isp_dev::streams_output(2147483646, 1 << 20) ? 0 : 1;
}
"""


def test_outputs_that_a_reader_finds_in_the_cache(tmp_path):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-I" + os.path.join(ROOT, "paper_2403_14853_amd", "csrc"), str(src), "-o", str(exe)])
    res = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert res.returncode == 0, res.stdout
