"""The cut of a host copy into chunks (tests/cpp/test_copy_chunks.cpp, compiled with csrc/copy_pool.cpp)."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1511_07658_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_copy_chunks(tmp_path):
    exe = str(tmp_path / "t")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-pthread", f"-I{CSRC}",
                    os.path.join(HERE, "cpp", "test_copy_chunks.cpp"), os.path.join(CSRC, "copy_pool.cpp"), "-o", exe],
                   check=True)
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
