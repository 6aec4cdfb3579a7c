"""Which batches have their timed span recorded on the copy FIFOs
(csrc/batch_plan.cpp, compiled here): those whose kernels all follow a whole
copy-in of the batch and precede a copy-out of it."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1511_07658_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "batch_plan.hpp"
#include "gvm.h"
using namespace gvm;
int main() {
  const PlanJob whole{GVM_K_VECADD, 1 << 20, true, true, false, false, false};
  PlanJob local = whole, resident = whole, kept = whole, pieces = whole, out_pieces = whole;
  local.local = true;
  resident.copy_in = false;
  kept.copy_out = false;
  pieces.pieces = true;
  out_pieces.out_pieces = true;
  const std::vector<PlanJob> cases[] = {{whole}, {whole, whole}, {local}, {whole, local}, {resident}, {kept},
                                        {whole, resident}, {whole, kept}, {resident, kept}, {pieces},
                                        {whole, pieces}, {out_pieces}};
  for (const int policy : {GVM_POLICY_PS1, GVM_POLICY_PS2, GVM_POLICY_GROUPED, GVM_POLICY_AUTO}) {
    for (const auto& c : cases) printf("%d", span_on_fifos(policy, c));
    printf("\n");
  }
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_span_marks(tmp_path):
    src, exe = tmp_path / "t.cpp", str(tmp_path / "t")
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", f"-I{ROOT}/include", f"-I{CSRC}", str(src),
                    os.path.join(CSRC, "batch_plan.cpp"), "-o", exe], check=True)
    got = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=60, check=True).stdout.split()
    # PS-1 routes small copies over the FIFOs too, and its phases hold for any
    # mix; PS-2 needs both copies of every job there; never with queued pieces
    assert got == ["111100111001", "110000000001", "000000000000", "000000000000"]
