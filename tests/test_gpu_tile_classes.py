"""The two tile classes of the 16-bit contractions (256x256 and 128x128) against the oracle, every element:
segments of one expert around the edges of a 128-row tile and its 64-row halves, and ragged sizes at which
the launch rule gives all or some of a step's launches 256x256 tiles (the named workloads C3, C4, C5 are
covered on samples by test_gpu_full_configs.py)."""
import pytest
import torch

from paper_2411_01288_amd import binding as B
from paper_2411_01288_amd.workloads import MoEWorkload, generate
from gpu_util import assert_tiles
from test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("T", [1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 191, 193, 257])
def test_row_edges_of_a_128_row_tile(oracle, T):
    # a segment of exactly T rows, and one of 193, with which there are too many for 32x128 tiles; feature sizes with column tails of both kinds (64 and
    # 192 of 128)
    w = MoEWorkload("edge", T + 193, 192, 320, 2, 1, "bf16", "topk", 900 + T)
    assert_tiles(w, [128, 128, 128, 128])
    data = generate(w, DEV)
    data["topk_idx"].copy_((torch.arange(w.T, device=DEV) >= T).view(-1, 1))
    data["gate"] = 0.5 + torch.rand_like(data["gate"])
    full_parity(oracle, w, data, label=f"edge T{T}")


@pytest.mark.parametrize("T,d,f,E,k,dtype,tiles", [
    (25003, 192, 960, 3, 2, "bf16", [256, 256, 256, 256]),
    (17001, 448, 576, 5, 2, "bf16", [128, 256, 256, 256]),
    (25003, 384, 448, 1, 2, "f16", [128, 128, 128, 128]),    # (top-1: there is one expert)
    (56250, 320, 192, 9, 2, "f16", [256, 128, 256, 128]),    # the second layer's backward reads the lists, the first's does not
    (25003, 192, 448, 5, 2, "f16", [128, 128, 128, 256]),
])
def test_mixed_tile_classes(oracle, T, d, f, E, k, dtype, tiles):
    w = MoEWorkload("mixed", T, d, f, E, min(k, E), dtype, "topk", 77 + T)
    assert_tiles(w, tiles)
    full_parity(oracle, w, generate(w, DEV), label=f"{dtype} T{T} d{d} f{f} E{E} k{k}")


@pytest.mark.parametrize("E", [1, 64, 65, 256, 257, 1024])
def test_expert_look_up(oracle, E):
    # 128x128 tiles; one, four or sixteen experts per lane in the look-up, many of them empty, some cut into chunks
    w = MoEWorkload("lanes", 6000, 64, 128, E, min(E, 2), "bf16", "zipf", 60 + E)
    assert_tiles(w, [128, 128, 128, 128])
    full_parity(oracle, w, generate(w, DEV), label=f"E{E}")


# more than 256 MB of weights and fewer than 128 rows per expert: the forward pass deals groups of tiles in eighths.  Column tiles
# with a tail, groups of row tiles with a rest, empty experts
# (thin: both on 32x128 tiles, in groups of 32 row tiles; the third and fourth case have a group and a rest of them)
@pytest.mark.parametrize("T,d,f,E,k,dtype,routing,thin", [
    (300, 1024, 2112, 62, 2, "bf16", "zipf", 0), (9, 2048, 3264, 20, 1, "f16", "topk", 3), (60, 704, 3136, 61, 1, "f16", "topk", 3),
    (96, 1024, 1344, 100, 2, "bf16", "bias", 3), (1200, 704, 3136, 61, 1, "bf16", "bias", 0)])
def test_streamed_weights(oracle, T, d, f, E, k, dtype, routing, thin):
    w = MoEWorkload("streamed", T, d, f, E, k, dtype, routing, 31 + T)
    assert w.A < 128 * E and 2 * E * d * f > 256e6
    assert_tiles(w, [128, 128, 128, 128], thin=thin)
    full_parity(oracle, w, generate(w, DEV), label=f"streamed T{T}")


# the look-up divides only where an expert is cut into chunks, which is from L + L / 8 + 1 rows on: the last size without, the first with,
# few rows on many experts (none near it); one, four and sixteen experts per lane
@pytest.mark.parametrize("E", [40, 130, 300])
@pytest.mark.parametrize("over", [0, 1, None])
def test_look_up_with_and_without_cut_experts(oracle, E, over):
    w = MoEWorkload("cut", 3000 if over is not None else 2 * E // 3, 64, 192, E, 1, "bf16", "topk", E)
    assert_tiles(w, [128, 128, 128, 128], thin=3 if w.T < 193 else 0)    # (few rows: the forward pass on 32x128)
    data = generate(w, DEV)
    if over is not None:
        L = B.launch_plan(B.make_shape(w.T, w.d_model, w.d_ff, E, 1, w.dtype))["chunk_rows"]
        n = L + L // 8 + over
        assert n < w.T
        at = torch.randperm(w.T, device=DEV)
        data["topk_idx"][at[:n]] = E - 3
        data["topk_idx"][at[n:]] = (torch.arange(w.T - n, device=DEV, dtype=torch.int32) % (E - 3)).view(-1, 1)
    full_parity(oracle, w, data, label=f"cut E{E} {over}")
