"""CPU checks of the SGEMM launch: the choice of tiles (csrc/gemm_choice.hpp,
compiled here), the k-step's LDS schedule restated, and the fetch addresses
of every tile inside the matrices."""

import os
import re
import shutil
import subprocess

import pytest

from test_sgemm_lds_schedule import JUNK, races

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1511_07658_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "gemm_choice.hpp"
int main() {
  using namespace gvm;
  for (const GemmCost& c : kGemmCosts) printf("cost %d %u %u\n", c.config, c.bm, c.bn);
  for (uint32_t count : {1u, 2u, 5u, 8u, 32u})
    for (uint32_t n : {1u, 31u, 33u, 256u, 517u, 1024u, 1536u, 2048u, 4096u, 65536u}) {
      std::vector<uint32_t> v(count, n);
      printf("pick %u %u %d\n", count, n, gemm_cheapest(count, v.data()));
    }
  const uint32_t mix[4] = {1920, 704, 160, 1};
  printf("mix %d\n", gemm_cheapest(4, mix));
}
"""


def configs():
    src = open(os.path.join(CSRC, "sgemm.hip")).read()
    return {int(r[0]): tuple(int(x) for x in r[1:])
            for r in re.findall(r"\{(\d+), (\d+), (\d+), (\d+), (\d+), (\d+), (?:true|false)\}", src)}


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_choice_names_compiled_tiles_and_fills_the_chip(tmp_path):
    src = tmp_path / "choice.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "choice")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", f"-I{CSRC}", str(src), "-o", exe], check=True)
    out = subprocess.run([exe], stdout=subprocess.PIPE, text=True, timeout=60, check=True).stdout
    cfg = configs()
    costs = {int(a): (int(b), int(c)) for a, b, c in re.findall(r"cost (\d+) (\d+) (\d+)", out)}
    assert all(cfg[i][:2] == t for i, t in costs.items())
    for count, n, pick in ((int(a), int(b), int(c)) for a, b, c in re.findall(r"pick (\d+) (\d+) (\d+)", out)):
        bm, bn = costs[pick]
        tiles = count * -(-n // bm) * -(-n // bn)
        smallest = count * -(-n // 32) * -(-n // 32)
        # at least half of the 256 CUs have a tile where 32x32 tiles would
        # give them one (517: 153 tiles of 64x32, faster than 289 of 32x32)
        assert tiles >= min(smallest, 128), (count, n, pick, tiles)
    assert int(re.search(r"mix (\d+)", out).group(1)) in costs


def step_loop(ktiles, pipe):
    """Events of one tile's k-loop: the next k-tile is written in the first
    half of a step, and with PIPE its fragments are read after the barrier;
    the remainder of k, if any, is the last k-tile."""
    ev = [("W", 0, 0), ("B",)]
    if pipe:
        ev.append(("R", 0, 0))
    for kt in range(ktiles - 1):
        nxt = kt + 1
        if pipe:
            ev += [("W", nxt & 1, nxt), ("B",), ("R", nxt & 1, nxt)]
        else:
            ev += [("R", kt & 1, kt), ("W", nxt & 1, nxt), ("B",)]
    if not pipe:
        ev.append(("R", (ktiles - 1) & 1, ktiles - 1))
    return ev


@pytest.mark.parametrize("pipe", [True, False])
@pytest.mark.parametrize("ktiles", [1, 2, 3, 4, 5, 9, 32])
def test_step_loop_has_no_lds_race(pipe, ktiles):
    assert JUNK is None
    assert races(step_loop(ktiles, pipe)) == []


def test_the_check_catches_a_missing_barrier():
    ev = step_loop(6, True)
    barriers = [i for i, e in enumerate(ev) if e == ("B",)]
    del ev[barriers[3]]
    assert races(ev)


@pytest.mark.parametrize("n", [1, 3, 16, 31, 32, 33, 35, 63, 64, 65, 97, 130, 255, 257])
def test_fetches_stay_inside_the_matrices(n):
    # the offsets of the unmasked 16-byte fetches of every full k-tile of
    # every tile, restated from the kernel: floats 0 .. n*n - 1 of A and of B
    for idx, (bm, bn, bk, wm, wn) in configs().items():
        nt = wm * wn * 64
        assert bm * bk % (4 * nt) == 0 and bk * bn % (4 * nt) == 0, idx
        nfull = n // bk
        if nfull == 0:
            continue
        for row0 in range(0, n, bm):
            top = min(bm - 1, n - 1 - row0)
            last = (row0 + top) * n + (nfull - 1) * bk + bk - 4 + 3
            assert last < n * n, (idx, n, row0)
        for col0 in range(0, n, bn):
            c = max(c if col0 + c < n else 0 for c in range(0, bn, 4))
            last = col0 + (nfull * bk - 1) * n + c + 3
            assert last < n * n, (idx, n, col0)
