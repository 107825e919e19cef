"""The work list of the large-prompt similarity kernel (csrc/equiv_tiles.hpp), on the CPU: every tile
of every prompt's upper triangle once, and no XCD with more than its share of the work."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_18954_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"
XCDS, RESIDENT = 8, 4 * 256


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    exe = str(tmp_path_factory.mktemp("tiles") / "tiles_driver")
    r = subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", CSRC,
                        os.path.join(ROOT, "tests", "host", "tiles_driver.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


@pytest.mark.parametrize("sizes", [[], [257], [321, 320], [517] * 64, [517] * 65, [4000] + [300] * 7,
                                   [300] * 7 + [4000], [1500] + [500] * 7, [2000] * 9, [300] * 100,
                                   list(range(260, 1260, 50)), [257] * 68, [257] * 69, [20000, 257]])
def test_tiles_cover_and_balance(driver, sizes):
    r = subprocess.run([driver, *map(str, sizes)], capture_output=True, text=True)
    assert r.returncode == 0
    side, *lines = r.stdout.splitlines()
    side, tiles = int(side), [tuple(map(int, l.split())) for l in lines]
    small = sum((n + 63) // 64 * ((n + 63) // 64 + 1) // 2 for n in sizes)
    assert side == (64 if small <= RESIDENT else 128)     # small tiles while all run at once
    assert len(tiles) % XCDS == 0
    want, at = [], 0
    for n in sizes:
        want += [(at + i, at + j, at + n) for i in range(0, n, side) for j in range(i, n, side)]
        at += n
    assert sorted(t for t in tiles if t[2] > 0) == sorted(want)
    # a tile of at most half the columns counts a third; at most a sixteenth, or one tile, beyond
    # an eighth
    load = [sum(3 if t[2] - t[1] > side // 2 else 1 for t in tiles[x::XCDS] if t[2] > 0)
            for x in range(XCDS)]
    mean = sum(load) / XCDS
    assert max(load) <= max(mean + 3, mean * 17 / 16)
