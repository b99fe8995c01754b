"""The 128x64 tiles of the fp32 path (operands in three bf16 planes) against the oracle, every element:
segments and feature sizes around the edges of a tile and of a K-step, rows at any dword alignment, the last rows of every tensor, token
contractions of one row to several chunks."""
import pytest
import torch

from paper_2411_01288_amd import binding as B
from paper_2411_01288_amd.workloads import MoEWorkload, generate
from test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def wide(w):
    return B.launch_plan(B.make_shape(w.T, w.d_model, w.d_ff, w.E, w.k, w.dtype))["wide"]


# wide: bits of fc1, fc2, bwd_fc2, bwd_fc1.  Contractions of 576 (the shortest on these tiles) to 1281: whole steps, last steps of one to 31
@pytest.mark.parametrize("T,d,f,E,k,routing,launches", [
    (4097, 640, 703, 1, 1, "topk", 5), (3001, 577, 578, 3, 3, "zipf", 15), (2003, 583, 1281, 5, 3, "topk", 15), (6001, 576, 517, 3, 1, "topk", 5),
    (9001, 517, 607, 2, 1, "topk", 10), (3000, 258, 1027, 70, 3, "zipf", 10), (700, 391, 1030, 90, 1, "zipf", 10),
])
def test_edges(oracle, T, d, f, E, k, routing, launches):
    w = MoEWorkload("wide", T, d, f, E, k, "f32", routing, 900 + d)
    assert wide(w) == launches
    full_parity(oracle, w, generate(w, DEV), label=f"wide T{T} d{d} f{f} E{E} k{k}")


@pytest.mark.parametrize("rows", [1, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128, 129, 300])
def test_segments(oracle, rows):
    w = MoEWorkload("segment", 80 * rows, 578, 605, 80, 1, "f32", "topk", rows)
    assert wide(w) == 15
    data = generate(w, DEV)
    data["topk_idx"] = (torch.arange(w.T, device=DEV, dtype=torch.int32) % 80).view(w.T, 1).contiguous()
    full_parity(oracle, w, data, label=f"segments of {rows}")
