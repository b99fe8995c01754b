"""FC2 in shares of its contraction (few rows, long d_ff) against the oracle, every element of forward and backward (which
reads the expert outputs that the split path rounds and stores): shares of unequal length, one row, column tails,
several row tiles per expert, dropped assignments."""
import numpy as np
import pytest
import torch

from paper_2411_01288_amd import binding as B
from paper_2411_01288_amd.workloads import MoEWorkload, generate
from gpu_util import TOL, host32, host_inputs, nrm_err, poisoned
from test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("T,d,f,E,k,dtype", [
    (1, 64, 4096, 1, 1, "bf16"), (5, 64, 2112, 4, 2, "f16"), (16, 192, 1088, 16, 2, "bf16"), (130, 320, 1024, 3, 1, "bf16"),
    (33, 128, 704, 70, 8, "f16"), (300, 64, 2048, 2, 2, "bf16"),
])
def test_split_fc2(oracle, T, d, f, E, k, dtype):
    w = MoEWorkload("shares", T, d, f, E, k, dtype, "topk", 210 + T)
    full_parity(oracle, w, generate(w, DEV), label=f"{dtype} T{T} d{d} f{f} E{E} k{k}")


def test_split_fc2_drops_out_of_range_ids(oracle):
    w = MoEWorkload("shares", 20, 128, 2048, 6, 2, "bf16", "topk", 4)
    data = generate(w, DEV)
    data["topk_idx"][:, 1] = torch.tensor([6, -1] * 10, device=DEV, dtype=torch.int32)
    shape = B.make_shape(w.T, w.d_model, w.d_ff, w.E, w.k, w.dtype)
    idx = B.hexa_moe_index(shape, data["topk_idx"])
    ws = B.alloc_workspace(shape, torch.device(DEV))
    ws.fill_(0xFF)
    y = B.hexa_moe_fwd(shape, data["x"], data["topk_idx"], data["gate"], data["W1"], data["b1"], data["W2"], data["b2"],
                       idx, ws, poisoned((w.T, w.d_model), data["x"].dtype, DEV))
    c = host_inputs(data)
    ref = oracle.fwd(c["x"], np.ascontiguousarray(c["topk_idx"][:, :1]), np.ascontiguousarray(c["gate"][:, :1]),
                     c["W1"], c["b1"], c["W2"], c["b2"])
    assert nrm_err(host32(y), ref) <= TOL["bf16"]
