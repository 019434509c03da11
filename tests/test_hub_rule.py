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
