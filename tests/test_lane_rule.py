"""How many lanes hold a row, on the CPU (csrc/lane_rule.h): on both sides of the sizes where the choice changes."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HEAD = r"""
#include <stdio.h>
#include <initializer_list>
#include "lane_rule.h"
using namespace isp_dev;
#define CHECK(...) do { if (!(__VA_ARGS__)) { printf("%s\n", #__VA_ARGS__); return 1; } } while (0)
constexpr int64_t Ki = 1 << 10, Mi = 1 << 20;
"""


def run(tmp_path, program):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(HEAD + program)
    subprocess.check_call(["g++", "-std=c++17", "-I" + os.path.join(ROOT, "paper_2403_14853_amd", "csrc"), str(src), "-o", str(exe)])
    res = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert res.returncode == 0, res.stdout


def test_four_lanes(tmp_path):
    """(Without hub rows, few entries took 2 to 13 % longer with four lanes.)"""
    run(tmp_path, r"""
int main() {
  for (int64_t hubs : {0, 1, 50}) {
    for (fused_pass p : {fused_pass::two_pass, fused_pass::one_pass}) {
      const int64_t from = hubs ? 64 * Ki : 96 * Ki;
      CHECK(!fused_four_lanes(p, 16, from - 1, hubs) && fused_four_lanes(p, 16, from, hubs));
      CHECK(!fused_four_lanes(p, 17, from, hubs) && fused_four_lanes(p, 4, 2147483646, hubs));
    }
    const int64_t from = hubs ? 64 * Ki : 120 * Ki;
    CHECK(!fused_four_lanes(fused_pass::forward, 16, from - 1, hubs) && fused_four_lanes(fused_pass::forward, 16, from, hubs));
    CHECK(!fused_four_lanes(fused_pass::forward, 17, from, hubs));
    CHECK(sddmm_four_lanes(16, 64 * Ki - 1, hubs) == (hubs > 0) && sddmm_four_lanes(16, 64 * Ki, hubs) && !sddmm_four_lanes(17, 64 * Ki, hubs));
    CHECK(select_four_lanes(16, 256 * Ki - 1, hubs) == (hubs > 0) && select_four_lanes(16, 256 * Ki, hubs) && !select_four_lanes(17, 256 * Ki, hubs));
    CHECK(select_four_lanes(16, 32 * Mi - 1, hubs) && !select_four_lanes(16, 32 * Mi, hubs));
  }
  CHECK(!fused_four_lanes(fused_pass::forward, 16, 120000, 0));  // (3.8 k rows, uniform: 6.2 -> 6.6 us with four)
  CHECK(!fused_four_lanes(fused_pass::two_pass, 16, 80000, 0));  // (6 k: 12.5 -> 13.1)
  CHECK(!select_four_lanes(16, 20000, 0) && !select_four_lanes(8, 120000, 0));  // (2 k and 3.8 k: 10.3 -> 11.1, 11.7 -> 12.5)
  CHECK(!sddmm_four_lanes(16, 60000, 0));  // (9 k: 4.4 -> 4.5)
  return 0;
}
""")


def test_two_vectors(tmp_path):
    """(The two passes of a directed graph's backward, which one vector runs in pairs of entries, took up to 13 % longer with two beyond the L2s.)"""
    run(tmp_path, r"""
int main() {
  for (fused_pass p : {fused_pass::forward, fused_pass::one_pass, fused_pass::two_pass}) {
    CHECK(!fused_two_vectors(p, 64, 1000, 900, 20000) && fused_two_vectors(p, 65, 1000, 900, 20000) && fused_two_vectors(p, 256, 1000, 900, 20000));
    CHECK(fused_two_vectors(p, 128, 6000, 5000, 3 * Mi / 4 - 1) && !fused_two_vectors(p, 128, 6000, 5000, 3 * Mi / 4));
    CHECK(fused_two_vectors(p, 129, 6000, 5500, Mi - 1) && !fused_two_vectors(p, 129, 6000, 5500, Mi));
    CHECK(fused_two_vectors(p, 40, 233000, 233000, 115000000));  // (rows of 200 entries and more)
    CHECK(fused_two_vectors(p, 128, 12288, 12000, 300000) && fused_two_vectors(p, 128, 12289, 12000, 300000) == (p != fused_pass::two_pass));
  }
  for (int64_t nnz : {512 * Ki - 1, 512 * Ki}) {
    const bool few = nnz < 512 * Ki;
    CHECK(fused_two_vectors(fused_pass::one_pass, 128, 40960, 40000, nnz) && fused_two_vectors(fused_pass::one_pass, 128, 40961, 40000, nnz) == few);  // (5 Mi floats)
    CHECK(fused_two_vectors(fused_pass::one_pass, 256, 32768, 30000, nnz) && fused_two_vectors(fused_pass::one_pass, 256, 32769, 30000, nnz) == few);  // (8 Mi)
    CHECK(fused_two_vectors(fused_pass::one_pass, 160, 90000, 80000, nnz) && fused_two_vectors(fused_pass::one_pass, 161, 90000, 80000, nnz) == few);
    CHECK(fused_two_vectors(fused_pass::forward, 256, 90000, 80000, nnz));
  }
  CHECK(!fused_two_vectors(fused_pass::one_pass, 100, 60000, 60000, 600000));  // (58.9 -> 64.2 us with two)
  CHECK(fused_two_vectors(fused_pass::two_pass, 144, 87381, 80000, 800000) && !fused_two_vectors(fused_pass::two_pass, 144, 87382, 80000, 800000));  // (12 Mi floats)
  CHECK(fused_two_vectors(fused_pass::two_pass, 160, 50000, 40000, 800000) && !fused_two_vectors(fused_pass::two_pass, 161, 50000, 40000, 800000));
  CHECK(!fused_two_vectors(fused_pass::two_pass, 100, 60000, 33000, 600000) && !fused_two_vectors(fused_pass::two_pass, 256, 80000, 45000, 800000));  // (90.8 -> 101, 281 -> 300 us with two)
  CHECK(!fused_two_vectors(fused_pass::two_pass, 128, 30000, 30000, 600000));  // (uniform: 128 -> 139)
  return 0;
}
""")
