"""Outputs and partial rows that SpMM writes past the caches, on the CPU (csrc/output_rule.h): not those that the Infinity Cache keeps for their
reader."""
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

PIECES = r"""
#include <stdio.h>
#include "output_rule.h"
int main() {
  // (800 k rows, 40 M entries are 247,219 pieces: 100 columns gain by it; 1.2 M, 60 M: 366 k, 64 columns; 120 k, 40 M: 305 k, 64 columns gain nothing, nor 100 k, 16 M: 112 k, 192)
  const struct { int64_t pieces, width; bool past; } want[] = {{247219, 100, true}, {247219, 92, true}, {366000, 64, true}, {863345, 48, true}, {304847, 64, false}, {111710, 192, false},
                                                               {22000000, 1, true}, {21999999, 1, false}, {2147483646, 256, true}, {0, 256, false}};
  for (auto& w : want)
    if (isp_dev::streams_pieces(w.pieces, w.width) != w.past) { printf("%lld pieces, %lld columns\n", (long long)w.pieces, (long long)w.width); return 1; }
  return 0;
}
"""


def run(tmp_path, program):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(program)
    subprocess.check_call(["g++", "-std=c++17", "-I" + os.path.join(ROOT, "paper_2403_14853_amd", "csrc"), str(src), "-o", str(exe)])
    res = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert res.returncode == 0, res.stdout


def test_outputs_that_a_reader_finds_in_the_cache(tmp_path):
    run(tmp_path, PROGRAM)


def test_partial_rows(tmp_path):
    run(tmp_path, PIECES)
