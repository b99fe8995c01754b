"""The deal of tiles to XCDs (csrc/deal.h), run on the CPU (host_deal.cpp): every tile once, no XCD more than a tile
ahead where tiles are shared out one by one, and a grid that holds the fullest XCD for the worst routing."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("deal") / "host_deal")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-w", os.path.join(HERE, "host_deal.cpp"), "-o", exe])
    return exe


def run(exe, *args):
    out = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0
    lines = out.stdout.split("\n")
    return [[int(v) for v in l.split()] for l in lines[:8]], int(lines[8])


# one tile; a few; groups of 4, 8 or 32 row tiles just full and one over; 128 groups of 4 (the line of the whole deal) and around
@pytest.mark.parametrize("BM,streamed", [(32, 0), (32, 1), (128, 0), (128, 1), (256, 0)])
@pytest.mark.parametrize("tm", [1, 3, 4, 7, 8, 9, 31, 32, 33, 65, 263, 508, 509, 511, 512, 513, 1057])
@pytest.mark.parametrize("tn", [1, 3, 12])
def test_row_tiles(program, BM, streamed, tm, tn):
    tiles, most = run(program, "rows", BM, tm, tn, tm + 5, streamed)
    assert sorted(sum(tiles, [])) == list(range(tm * tn))
    counts = [len(t) for t in tiles]
    assert max(counts) <= most
    group = 1024 // BM
    if BM != 256 or -(-tm // group) < 128:
        assert max(counts) - min(counts) <= 1
    else:
        assert max(counts) - min(counts) <= group * tn


# an XCD's rest of 0, 1, 12, 13, 16 and 31 tiles behind no, one and several whole rounds of 32
@pytest.mark.parametrize("tm,tn", [(8, 1), (1, 9), (128, 1), (128, 2), (129, 2), (384, 1), (385, 1), (392, 1), (31, 8), (81, 4), (96, 1), (104, 1), (103, 1),
                                   (263, 3), (263, 12), (1057, 8), (1057, 3)])
def test_quarters(program, tm, tn):
    dealt, _ = run(program, "quarters", tm, tn, tm + 5)
    whole, _ = run(program, "rows", 256, tm, tn, tm + 5, 0)
    for got, mine in zip(dealt, whole):
        rest = len(mine) % 32
        cut = mine[len(mine) - rest:] if rest <= 12 else []
        assert got == [5 * t for t in mine[:len(mine) - len(cut)]] + [5 * t + 1 + q for t in cut for q in range(4)]


@pytest.mark.parametrize("tiles", [1, 2, 7, 8, 9, 12, 36, 256])
@pytest.mark.parametrize("items", [0, 1, 2, 7, 8, 9, 17, 64])
def test_token_tiles(program, tiles, items):
    dealt, most = run(program, "tokens", tiles, items, items + 3)
    assert sorted(sum(dealt, [])) == list(range(tiles * items))
    counts = [len(t) for t in dealt]
    assert max(counts) <= most
    assert max(counts) - min(counts) <= min(8, items)
