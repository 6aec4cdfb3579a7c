"""The SGEMM tiles picked for a masked partition (csrc/gemm_choice.hpp, compiled
here): the whole chip's choice where no CU is taken away, and by the formula no
slower than that choice on the CUs that are left."""

import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1511_07658_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "gemm_choice.hpp"
using namespace gvm;
static const GemmCost& cost(int config) {
  for (const GemmCost& c : kGemmCosts) if (c.config == config) return c;
  return kGemmCosts[0];
}
int main() {
  for (int cus : {32, 64, 96, 128, 192, 256})
    for (uint32_t n : {1u, 33u, 256u, 517u, 1024u, 2048u, 4096u, 65536u}) {
      const int whole = gemm_cheapest(1, &n), part = gemm_cheapest(1, &n, cus);
      printf("%d %u %d %d %.9g %.9g\n", cus, n, whole, part, gemm_launch_us(cost(whole), 1, &n, cus),
             gemm_launch_us(cost(part), 1, &n, cus));
    }
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_partition_choice(tmp_path):
    src, exe = tmp_path / "p.cpp", str(tmp_path / "p")
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", f"-I{CSRC}", str(src), "-o", exe], check=True)
    rows = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=60, check=True).stdout.splitlines()
    assert len(rows) == 6 * 8
    for row in rows:
        cus, n, whole, part, t_whole, t_part = row.split()
        assert float(t_part) <= float(t_whole), row
        if cus == "256":
            assert whole == part, row
