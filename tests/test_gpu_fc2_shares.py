"""FC2 in shares of its contraction (few rows, long d_ff) against the oracle, every element of forward and backward (which
reads the expert outputs that the split path rounds and stores): shares of unequal length, one row, column tails,
several row tiles per expert, dropped assignments."""
import numpy as np
import pytest
import torch

from paper_2411_01288_amd import binding as B
from paper_2411_01288_amd.workloads import MoEWorkload, generate
from gpu_util import TOL, host32, host_inputs, nrm_err, run_hip_layer
from test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# thin: bits of fc1 and fc2 on 32x128 tiles
@pytest.mark.parametrize("T,d,f,E,k,dtype,thin", [
    (1, 64, 4096, 1, 1, "bf16", 3), (5, 64, 2112, 4, 2, "f16", 3), (16, 192, 1088, 16, 2, "bf16", 3), (130, 320, 1024, 3, 1, "bf16", 0),
    (33, 128, 704, 70, 8, "f16", 0), (300, 64, 2048, 2, 2, "bf16", 0), (5, 1728, 1088, 10, 2, "f16", 3), (33, 64, 2112, 5, 1, "f16", 0),
    (36, 192, 1088, 5, 1, "bf16", 0), (70, 64, 2112, 4, 2, "f16", 0),
])
def test_split_fc2(oracle, T, d, f, E, k, dtype, thin):
    w = MoEWorkload("shares", T, d, f, E, k, dtype, "topk", 210 + T)
    plan = B.launch_plan(B.make_shape(T, d, f, E, k, dtype))
    assert plan["fc2_shares"] > 1 and plan["thin"] == thin
    full_parity(oracle, w, generate(w, DEV), label=f"{dtype} T{T} d{d} f{f} E{E} k{k}")


@pytest.mark.parametrize("E,thin", [(6, 0), (16, 3)])
def test_split_fc2_drops_out_of_range_ids(oracle, E, thin):
    w = MoEWorkload("shares", 20, 128, 2048, E, 2, "bf16", "topk", 4)
    data = generate(w, DEV)
    data["topk_idx"][:, 1] = torch.tensor([E, -1] * 10, device=DEV, dtype=torch.int32)
    plan = B.launch_plan(B.make_shape(w.T, w.d_model, w.d_ff, w.E, w.k, w.dtype))
    assert plan["fc2_shares"] > 1 and plan["thin"] == thin
    _, y, g = run_hip_layer(w, data)     # the backward reads the expert outputs that this path stores
    c = host_inputs(data)
    kept = lambda a: np.ascontiguousarray(a[:, :1])
    args = (c["x"], kept(c["topk_idx"]), kept(c["gate"]), c["W1"], c["b1"], c["W2"])
    dx, dgate = oracle.bwd_tokens(*args, c["b2"], c["dY"])
    dW1, db1, dW2, db2 = oracle.bwd_experts(*args, c["dY"])
    for name, got, ref in (("y", y, oracle.fwd(*args, c["b2"])), ("dx", g["dx"], dx), ("dgate", g["dgate"][:, :1], dgate),
                           ("dW1", g["dW1"], dW1), ("db1", g["db1"], db1), ("dW2", g["dW2"], dW2),
                           ("db2", g["db2"], db2)):
        assert nrm_err(host32(got), ref) <= TOL["bf16"], name
    assert not g["dgate"][:, 1].any()
