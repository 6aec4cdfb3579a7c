"""CUs that a launch in a masked partition is counted over (csrc/common.cpp,
compiled here): as many as the shader engine with the fewest has, in every engine
that has any, and never more than the mask."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1511_07658_amd", "csrc")

PROGRAM = r"""
#include "common.hpp"
using namespace gvm;
int main() {
  uint32_t lat[kPartitionCus / 32], bulk[kPartitionCus / 32];
  for (uint32_t cus = 32; cus < 256; cus += 32)
    if (cu_partition_masks(cus, lat, bulk) == GVM_OK)
      printf("%u %d %d\n", cus, partition_carrying_cus(lat), partition_carrying_cus(bulk));
  for (uint32_t& w : bulk) w = ~0u;
  printf("256 %d 0\n", partition_carrying_cus(bulk));
  for (uint32_t& w : bulk) w = 0x00010003u;   // 16 CUs of engine 0 and 8 of engine 2
  printf("24 %d 0\n", partition_carrying_cus(bulk));
  for (uint32_t& w : bulk) w = 0;
  printf("0 %d 0\n", partition_carrying_cus(bulk));
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_carrying_cus(tmp_path):
    src, exe = tmp_path / "p.cpp", str(tmp_path / "p")
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", f"-I{CSRC}", f"-I{ROOT}/include", str(src),
                    os.path.join(CSRC, "common.cpp"), "-o", exe], check=True)
    got = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=60, check=True).stdout.splitlines()
    # 64 CUs an engine; an odd multiple of 32 halves one engine in both partitions
    assert got == ["32 32 128", "64 64 192", "96 64 96", "128 128 128", "160 96 64", "192 192 64", "224 128 32",
                   "256 256 0", "24 16 0", "0 0 0"]
