"""The kernel that builds the work lists of the 256x256 contractions, run on the CPU (host_worklists.cpp) in two
orders of its wavefronts and lanes: a thread that reads or overwrites what another thread writes between the same
two barriers gives lists that depend on the order."""
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("worklists") / "host_worklists")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-w", os.path.join(HERE, "host_worklists.cpp"), "-o", exe])
    return exe


def run(exe, order, offsets, L, d, f, rt_cap):
    text = " ".join(map(str, [order, len(offsets) - 1, L, rt_cap, d, f, *offsets]))
    out = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stderr
    return np.array(out.stdout.split(), dtype=np.int64)


def expected(offsets, L, d, f):
    """(row tiles, items, flags) as the header and the lists should hold them."""
    tiles, items, slots, longest = [], [], 0, 0
    for e, (b, end) in enumerate(zip(offsets[:-1], offsets[1:])):
        n = end - b
        tiles += [(e, r, min(end, r + 256), -1) for r in range(b, end, 256)]
        if n == 0:
            continue
        nc = max(0, n - L // 8 - 1) // L + 1     # as few chunks as keep them at 9/8 L, equal up to blocks of 64 rows
        starts = [(c * (n // nc) + min(c, n % nc)) // 64 * 64 for c in range(nc)] + [n]
        items += [(e, b + starts[c], b + starts[c + 1], slots + c if nc > 1 else -1) for c in range(nc)]
        slots += nc if nc > 1 else 0
        longest = max(longest, n // nc)
    return tiles, items, (int(longest >= 8 * d), int(longest >= 8 * f))


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("E", [1, 2, 63, 64, 65, 128, 192, 640, 960, 1000, 1023, 1024])
def test_lists_do_not_depend_on_the_order_of_the_wavefronts(program, E, order):
    rng = np.random.default_rng(E)
    L, d, f = 1024, 64, 512
    counts = np.minimum(rng.zipf(1.3, E) * 37, 20000)
    counts[rng.random(E) < 0.2] = 0
    counts[E - 1] = 4999                          # the last segment: several row tiles and chunks
    offsets = [0, *np.cumsum(counts).tolist()]
    rt_cap = offsets[-1] // 256 + E
    got = run(program, order, offsets, L, d, f, rt_cap)
    tiles, items, flags = expected(offsets, L, d, f)
    assert got[:4].tolist() == [len(tiles), len(items), *flags]
    quads = got[8:].reshape(-1, 4)
    assert quads[:len(tiles)].tolist() == [list(t) for t in tiles]
    assert quads[rt_cap:rt_cap + len(items)].tolist() == [list(i) for i in items]
