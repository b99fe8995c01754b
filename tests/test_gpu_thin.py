"""The 32x128 tiles of forward passes with few rows per expert, against the oracle, every element: segments around the 16 and 32
rows of a tile, contractions of two to many 32-k steps (fewer than wavefronts, no multiple of what is on its way), column tails, FC2 in
one share and in several, empty experts, one, four and sixteen experts per lane in the look-up; all activations; no valid id; the
rule that takes them."""
import pytest
import torch

from paper_2411_01288_amd import binding as B
from paper_2411_01288_amd.workloads import MoEWorkload, generate
from gpu_util import run_hip_layer
from test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def plan(w):
    return B.launch_plan(B.make_shape(w.T, w.d_model, w.d_ff, w.E, w.k, w.dtype))


# thin: bits of fc1 and fc2
@pytest.mark.parametrize("T,d,f,E,k,dtype,routing,thin,split", [
    (1, 64, 64, 1, 1, "bf16", "topk", 3, False), (3, 128, 192, 5, 2, "f16", "topk", 3, False), (16, 768, 3072, 16, 2, "bf16", "bias", 3, True),
    (40, 320, 448, 14, 2, "bf16", "zipf", 3, True), (40, 576, 832, 48, 4, "f16", "zipf", 3, True), (64, 192, 704, 104, 3, "f16", "zipf", 3, True),
    (90, 64, 1088, 300, 2, "bf16", "zipf", 3, True), (63, 320, 704, 180, 3, "bf16", "zipf", 3, True), (150, 1024, 128, 200, 1, "bf16", "zipf", 1, False), (190, 1024, 320, 260, 1, "f16", "topk", 1, False),
    (96, 192, 2112, 32, 2, "bf16", "bias", 3, True), (64, 192, 448, 1024, 1, "bf16", "topk", 3, True),
])
def test_thin(oracle, T, d, f, E, k, dtype, routing, thin, split):
    w = MoEWorkload("thin", T, d, f, E, k, dtype, routing, 40 + T)
    p = plan(w)
    assert p["thin"] == thin and (p["fc2_shares"] > 1) == split
    full_parity(oracle, w, generate(w, DEV), label=f"thin T{T} d{d} f{f} E{E} k{k}")


# From two rows on: a single dgate = <dY, o> is off by up to 2^-9 |dY| |o| (o is rounded), which has no bound relative to a sum that happens
# to cancel (one row, d = 192: z |dY| |o| / sqrt(192) with z = 0.03); two and more are judged by the largest.
@pytest.mark.parametrize("rows", [2, 15, 16, 17, 31, 32, 33, 48, 49, 64, 65, 191, 192])
def test_rows_of_one_expert(oracle, rows):
    w = MoEWorkload("rows", rows, 192, 320, 32, 1, "bf16", "topk", rows)      # the other experts are empty
    assert plan(w)["thin"] == 3
    data = generate(w, DEV)
    data["topk_idx"].fill_(4)
    full_parity(oracle, w, data, label=f"thin, {rows} rows")


@pytest.mark.parametrize("kind", [B.ACT_RELU, B.ACT_SILU])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_activations(oracle, kind, dtype):
    w = MoEWorkload("act", 40, 192, 704, 20, 1, dtype, "topk", 70 + kind)
    assert plan(w)["thin"] == 3
    oracle.set_activation(kind)
    try:
        full_parity(oracle, w, generate(w, DEV), label=f"thin {dtype} {kind}", activation=kind)
    finally:
        oracle.set_activation(0)


@pytest.mark.parametrize("f", [192, 1088])                                    # fc2 in one share, in several
def test_all_ids_out_of_range(f):
    w = MoEWorkload("none", 20, 128, f, 16, 2, "bf16", "topk", 5)
    assert plan(w)["thin"] == 3 and (plan(w)["fc2_shares"] > 1) == (f > 192)
    data = generate(w, DEV)
    data["topk_idx"].copy_(torch.tensor([16, -1], device=DEV, dtype=torch.int32).expand(20, 2))
    idx, y, g = run_hip_layer(w, data)
    assert int(idx["offsets"][-1]) == 0
    for name, t in {"y": y, **g}.items():
        assert not t.any(), name


# at both sides of each line: 32 rows, 6 per expert, 192 rows in all, 1024 tiles of fc2
@pytest.mark.parametrize("T,d,E,thin", [(32, 192, 1, 3), (33, 192, 1, 0), (36, 192, 6, 3), (37, 192, 6, 0), (192, 192, 32, 3), (193, 192, 33, 0),
                                        (128, 1024, 128, 3), (129, 1024, 129, 1), (16, 8192, 16, 3), (16, 8256, 16, 1)])
def test_rule(T, d, E, thin):
    assert plan(MoEWorkload("rule", T, d, 1024, E, 1, "bf16", "topk", 1))["thin"] == thin
