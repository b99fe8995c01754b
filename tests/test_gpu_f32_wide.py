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


# launches: bits of fc2 (2), bwd_fc2 (4) and bwd_fc1 (8).  Contractions of 577 to 1281: whole steps, last steps of one to 31
@pytest.mark.parametrize("T,d,f,E,k,routing,launches", [
    (5001, 577, 578, 3, 1, "zipf", 10), (2003, 583, 1281, 5, 3, "topk", 10), (9001, 517, 607, 2, 1, "topk", 2), (6001, 1030, 509, 3, 1, "topk", 4),
    (3300, 1055, 1030, 3, 1, "zipf", 14), (23000, 70, 601, 2, 1, "topk", 10), (9300, 450, 600, 9, 1, "zipf", 10),
])
def test_edges(oracle, T, d, f, E, k, routing, launches):
    w = MoEWorkload("wide", T, d, f, E, k, "f32", routing, 900 + d)
    assert wide(w) == launches
    full_parity(oracle, w, generate(w, DEV), label=f"wide T{T} d{d} f{f} E{E} k{k}")


@pytest.mark.parametrize("rows,T,d,f,launches", [(r, 5000, 578, 605, 10) for r in (1, 31, 32, 33, 63, 64, 65, 96, 97, 127, 128, 129, 300)] +
                         [(r, 5600, 1030, 509, 4) for r in (1, 33, 64, 129)])
def test_segments(oracle, rows, T, d, f, launches):
    """One expert of `rows` rows, one of one more, one without, one with the rest (in several chunks)."""
    w = MoEWorkload("segment", T, d, f, 4, 1, "f32", "topk", rows)
    assert wide(w) == launches
    data = generate(w, DEV)
    ids = torch.full((T,), 3, device=DEV, dtype=torch.int32)
    at = torch.randperm(T, device=DEV, generator=torch.Generator(device=DEV).manual_seed(rows))
    ids[at[:rows]] = 0
    ids[at[rows:2 * rows + 1]] = 1
    data["topk_idx"] = ids.view(T, 1).contiguous()
    full_parity(oracle, w, data, label=f"segments of {rows}")


# what keeps launches on 64x64 tiles: short contractions, few rows per expert, few rows where the contraction is not 1536 long, one column of tiles,
# an M of which 128-row tiles would pad much
@pytest.mark.parametrize("T,d,f,E,launches", [
    (8192, 512, 575, 2, 0), (3000, 768, 768, 64, 0), (8191, 512, 1024, 8, 0), (8192, 512, 1024, 8, 10), (4095, 768, 1536, 8, 0), (4096, 768, 1536, 8, 10),
    (300000, 64, 600, 4, 0), (16384, 576, 576, 2, 2), (8192, 1023, 512, 4, 0), (8192, 1024, 512, 4, 4), (8192, 1024, 513, 4, 0),
])
def test_rule(T, d, f, E, launches):
    assert wide(MoEWorkload("rule", T, d, f, E, 1, "f32", "topk", 1)) == launches
