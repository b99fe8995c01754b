"""The two tile classes of the fp32 contractions (64x64 and 32x32) against the oracle, every element: segments
around the edges of a tile, of a wavefront's share of it and of the K-blocks, feature sizes that leave rows at
any dword alignment, and sizes at which the launch rule mixes the classes within a step."""
import pytest
import torch

from paper_2411_01288_amd.workloads import MoEWorkload, generate
from gpu_util import assert_tiles
from test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("T,d,f", [(1, 1, 1), (1, 3, 5), (15, 16, 17), (31, 33, 31), (32, 32, 64), (33, 31, 65),
                                   (63, 64, 66), (65, 67, 130), (129, 97, 191)])
def test_edges_of_a_tile(oracle, T, d, f):
    # one expert: a segment of exactly T rows
    w = MoEWorkload("edge", T, d, f, 1, 1, "f32", "topk", 700 + T)
    data = generate(w, DEV)
    data["gate"] = 0.5 + torch.rand_like(data["gate"])
    full_parity(oracle, w, data, label=f"edge T{T} d{d} f{f}")


@pytest.mark.parametrize("T,d,f,E,k,routing,tiles", [
    (4001, 190, 771, 3, 2, "topk", [64, 32, 64, 32]),
    (9001, 509, 66, 2, 1, "topk", [32, 64, 32, 64]),
    (3001, 258, 1027, 70, 3, "zipf", [64, 64, 64, 64]),   # more experts than lanes
    (500, 40, 50, 200, 2, "zipf", [32, 32, 32, 32]),      # most experts empty
])
def test_mixed_tile_classes(oracle, T, d, f, E, k, routing, tiles):
    w = MoEWorkload("mixed", T, d, f, E, k, "f32", routing, 33 + T)
    assert_tiles(w, tiles)                                # (none of them on 128x64)
    full_parity(oracle, w, generate(w, DEV), label=f"f32 T{T} d{d} f{f} E{E} k{k}")
