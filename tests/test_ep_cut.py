"""CPU check of the EP-like kernel's cut into units (tests/cpp/test_ep_cut.cpp)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_records_fit_the_scratch_for_every_size(tmp_path):
    exe = str(tmp_path / "test_ep_cut")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", f"-I{ROOT}/paper_1511_07658_amd/csrc",
                    f"-I{ROOT}/include", f"{ROOT}/tests/cpp/test_ep_cut.cpp", "-o", exe], check=True)
    p = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert p.returncode == 0 and p.stdout.strip().endswith("ok: 0 failures"), p.stdout[-2000:]
