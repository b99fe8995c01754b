"""The 32x128 tiles of forward passes with few rows per expert, against the oracle, every element: segments around the 16 and 32
rows of a tile, contractions of two to many 32-k steps (fewer than wavefronts, no multiple of what is on its way), column tails, FC2 in
one share and in several, empty experts, one, four and sixteen experts per lane in the look-up."""
import pytest
import torch

from paper_2411_01288_amd import binding as B
from paper_2411_01288_amd.workloads import MoEWorkload, generate
from test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def plan(w):
    return B.launch_plan(B.make_shape(w.T, w.d_model, w.d_ff, w.E, w.k, w.dtype))


@pytest.mark.parametrize("T,d,f,E,k,dtype,routing,split", [
    (1, 64, 64, 1, 1, "bf16", "topk", False), (3, 128, 192, 5, 2, "f16", "topk", False), (16, 768, 3072, 16, 2, "bf16", "bias", True),
    (40, 320, 448, 14, 2, "bf16", "zipf", True), (64, 576, 832, 48, 4, "bf16", "zipf", True), (200, 192, 704, 104, 3, "f16", "zipf", True),
    (300, 64, 1088, 300, 2, "bf16", "zipf", False), (900, 1024, 320, 160, 1, "bf16", "topk", False),
])
def test_thin(oracle, T, d, f, E, k, dtype, routing, split):
    w = MoEWorkload("thin", T, d, f, E, k, dtype, routing, 40 + T)
    p = plan(w)
    assert p["thin"] and (p["fc2_shares"] > 1) == split
    full_parity(oracle, w, generate(w, DEV), label=f"thin T{T} d{d} f{f} E{E} k{k}")


# From two rows on: a single dgate = <dY, o> is off by up to 2^-9 |dY| |o| (o is rounded), which has no bound relative to a sum that happens
# to cancel (one row, d = 192: z |dY| |o| / sqrt(192) with z = 0.03); two and more are judged by the largest.
@pytest.mark.parametrize("rows", [2, 15, 16, 17, 31, 32, 33, 48, 49, 64, 65])
def test_rows_of_one_expert(oracle, rows):
    w = MoEWorkload("rows", rows, 192, 320, 12, 1, "bf16", "topk", rows)      # the other experts are empty
    assert plan(w)["thin"]
    data = generate(w, DEV)
    data["topk_idx"].fill_(4)
    full_parity(oracle, w, data, label=f"thin, {rows} rows")
