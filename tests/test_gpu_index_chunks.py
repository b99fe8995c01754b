"""The index build against the oracle, bit for bit, at the edges of its launch plan: one workgroup or several, rows and
runs that are not full, expert counts around the wavefront and workgroup sizes, ids outside [0, E)."""
import numpy as np
import pytest
import torch

from paper_2411_01288_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("T,k,E,drop", [
    (1, 1, 1, False), (63, 1, 2, True), (65, 1, 64, False), (1023, 1, 65, True), (1025, 1, 3, False),
    (8192, 1, 64, False), (8191, 1, 512, True), (8193, 1, 64, False), (4097, 2, 17, True), (8192, 1, 513, False),
    (16400, 1, 1024, True), (131072, 1, 5, False), (131073, 2, 33, True), (400000, 1, 600, False),
    (1200000, 1, 40, True), (600000, 2, 1, False),      # more rows than a wavefront keeps in registers
])
def test_index_plans(oracle, T, k, E, drop):
    rng = np.random.default_rng(T + E)
    p = rng.random(E) ** 3
    ids = rng.choice(E, size=T * k, p=p / p.sum()).astype(np.int32)
    if drop:
        ids[rng.random(T * k) < 0.1] = E
        ids[rng.random(T * k) < 0.1] = -1
    check(oracle, ids, T, k, E, drop)


@pytest.mark.parametrize("T,E", [(1, 3), (64, 1), (65, 7), (511, 1), (512, 600), (8192, 64), (8193, 64), (70001, 2), (393216, 5), (393217, 5),
                                 (400000, 1024), (1100000, 16)])
@pytest.mark.parametrize("ids_of", ["last", "stray", "dropped"])
def test_collapsed_routing(oracle, T, E, ids_of):
    # rows of equal ids are counted in one addition: all on the last expert; all but a few; none in range
    ids = np.full(T, E if ids_of == "dropped" else E - 1, np.int32)
    if ids_of == "stray":
        ids[np.random.default_rng(T).integers(0, T, 1 + T // 3000)] = 0
        ids[-1] = -1
    check(oracle, ids, T, 1, E, ids_of != "last")


def check(oracle, ids, T, k, E, drop):
    shape = B.make_shape(T, 64, 64, E, k, "f32")
    got = B.alloc_idx(shape, torch.device(DEV))
    for t in got.values():
        t.fill_(-7)
    B.hexa_moe_index(shape, torch.from_numpy(ids.reshape(T, k)).to(DEV), got)
    got = {n: t.cpu().numpy() for n, t in got.items()}
    # ids outside the range are dropped: the stable sort of the others, -1 behind it and in inv
    valid = (ids >= 0) & (ids < E)
    perm = np.flatnonzero(valid)[np.argsort(ids[valid], kind="stable")]
    counts = np.bincount(ids[valid], minlength=E)
    inv = np.full(T * k, -1)
    inv[perm] = np.arange(perm.size)
    assert np.array_equal(got["counts"], counts)
    assert np.array_equal(got["offsets"], np.concatenate([[0], np.cumsum(counts)]))
    assert np.array_equal(got["perm"], np.concatenate([perm, np.full(T * k - perm.size, -1)]))
    assert np.array_equal(got["inv"], inv)
    if not drop:
        want = oracle.index(ids.reshape(T, k), E)
        assert all(np.array_equal(got[n], w) for n, w in zip(("counts", "offsets", "perm", "inv"), want))
