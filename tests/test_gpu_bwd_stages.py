"""The backward prologue and the backward finish against the oracle, every element: row lengths around the sweeps
of a group of lanes (16 or 64 lanes, one, two or four chunks each, more than one sweep), tiles with fewer rows than
wavefronts, experts cut into chunks whose partial weight gradients have a size that is no multiple of four."""
import pytest
import torch

from paper_2411_01288_amd.workloads import MoEWorkload, generate
from test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f16", 192), ("bf16", 512), ("f16", 576), ("bf16", 1024),
                                     ("bf16", 1088), ("bf16", 2048), ("bf16", 2112), ("f16", 4160),
                                     ("f32", 63), ("f32", 65), ("f32", 256), ("f32", 257), ("f32", 513), ("f32", 1024),
                                     ("f32", 1027), ("f32", 2050)])
def test_row_lengths(oracle, dtype, d):
    w = MoEWorkload("rows", 83, d, 64, 3, 2, dtype, "topk", 500 + d)
    full_parity(oracle, w, generate(w, DEV), label=f"{dtype} d{d}")


@pytest.mark.parametrize("T,d,f,E,k,dtype,routing", [
    (1500, 33, 35, 2, 1, "f32", "zipf"),      # several chunks, one tile each, odd partial tiles
    (4000, 130, 67, 70, 2, "f32", "zipf"),    # some experts cut, some whole, some empty; more experts than lanes
    (9000, 64, 128, 3, 1, "bf16", "zipf"),
    (33000, 128, 64, 66, 1, "f16", "forced"),
])
def test_split_experts(oracle, T, d, f, E, k, dtype, routing):
    w = MoEWorkload("split", T, d, f, E, k, dtype, routing, 40 + T)
    full_parity(oracle, w, generate(w, DEV), label=f"{dtype} T{T} d{d} f{f} E{E}")


@pytest.mark.parametrize("T,dtype", [(287, "f32"), (288, "f32"), (289, "f32"), (545, "f32"), (1919, "f32"),
                                     (1152, "bf16"), (1153, "bf16"), (2177, "f16"), (7000, "bf16")])
def test_chunk_counts(oracle, T, dtype):
    # one expert around the row counts at which it is cut into one more chunk (of about 256 and 1024 rows)
    w = MoEWorkload("cut", T, 64, 64, 1, 1, dtype, "topk", 80 + T)
    full_parity(oracle, w, generate(w, DEV), label=f"{dtype} T{T}")
