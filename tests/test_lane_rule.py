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
