"""The 256x256 contractions and their work lists against the oracle, every element, at shapes that the launch rule
sends there (asserted): segments around the edges of a 256-row tile and of its halves, expert counts around the
wavefront size of the list builder (a multiple of 64 puts the end of the last segment in another wavefront's reach),
ReLU and SiLU, dropped ids."""
import numpy as np
import pytest
import torch

from paper_2411_01288_amd import binding as B
from paper_2411_01288_amd.workloads import MoEWorkload, generate
from gpu_util import TOL, assert_tiles, host32, host_inputs, nrm_err, run_hip_layer
from test_gpu_parity import full_parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_row_edges_of_a_256_row_tile(oracle):
    # sixteen experts: fifteen short segments, the rest of the rows on one of them
    w = MoEWorkload("edges", 200000, 192, 192, 16, 1, "bf16", "topk", 31)
    assert_tiles(w, [256, 256, 256, 256])
    data = generate(w, DEV)
    counts = [1, 15, 17, 63, 65, 127, 128, 0, 129, 191, 255, 256, 257, 385, 511]
    counts.insert(9, w.T - sum(counts))
    ids = torch.repeat_interleave(torch.arange(w.E, dtype=torch.int32), torch.tensor(counts))
    gen = torch.Generator().manual_seed(5)
    data["topk_idx"].copy_(ids[torch.randperm(w.T, generator=gen)].reshape(w.T, 1))
    full_parity(oracle, w, data, label="edges")
    # a short segment's weight gradients on their own scale
    _, _, g = run_hip_layer(w, data)
    c = host_inputs(data)
    dW1, db1, dW2, db2 = oracle.bwd_experts(c["x"], c["topk_idx"], c["gate"], c["W1"], c["b1"], c["W2"], c["dY"])
    for e in np.flatnonzero(np.array(counts)):
        for name, ref in (("dW1", dW1), ("db1", db1), ("dW2", dW2), ("db2", db2)):
            assert nrm_err(host32(g[name][e]), ref[e]) <= TOL["bf16"], (name, e, counts[e])


@pytest.mark.parametrize("T,d,f,E,k,dtype", [
    (80000, 256, 256, 64, 2, "bf16"),
    (49000, 448, 448, 70, 1, "f16"),
    (64000, 192, 448, 128, 2, "bf16"),
])
def test_expert_counts(oracle, T, d, f, E, k, dtype):
    w = MoEWorkload("experts", T, d, f, E, k, dtype, "zipf", 12 + E)
    assert_tiles(w, [256, 256, 256, 256])
    full_parity(oracle, w, generate(w, DEV), label=f"{dtype} E{E}")


@pytest.mark.parametrize("kind", [B.ACT_RELU, B.ACT_SILU])
def test_activations(oracle, kind):
    w = MoEWorkload("act", 25003, 192, 960, 3, 2, "bf16", "zipf", 70 + kind)
    assert_tiles(w, [256, 256, 256, 256])
    oracle.set_activation(kind)
    try:
        full_parity(oracle, w, generate(w, DEV), label=f"activation {kind}", activation=kind)
    finally:
        oracle.set_activation(0)


def test_dropped_ids(oracle):
    w = MoEWorkload("drop", 80000, 256, 256, 64, 2, "bf16", "topk", 8)
    assert_tiles(w, [256, 256, 256, 256])
    data = generate(w, DEV)
    gen = torch.Generator().manual_seed(9)
    drop = torch.rand((w.T, w.k), generator=gen) < 0.1
    ids = data["topk_idx"].cpu()
    bad = torch.tensor([w.E, -1, 1000, -2**31], dtype=torch.int32)
    data["topk_idx"].copy_(torch.where(drop, bad[torch.randint(0, 4, (w.T, w.k), generator=gen)], ids))
    idx, y, g = run_hip_layer(w, data)
    drop = drop.numpy()
    assert int(idx["offsets"][-1]) == w.A - int(drop.sum())
    # an equivalent problem without dropped ids: those assignments with gate 0
    c = host_inputs(data)
    ti, gate = np.where(drop, 0, c["topk_idx"]).astype(np.int32), np.where(drop, 0, c["gate"]).astype(np.float32)
    args = (c["x"], ti, gate, c["W1"], c["b1"], c["W2"])
    dx, dgate = oracle.bwd_tokens(*args, c["b2"], c["dY"])
    dW1, db1, dW2, db2 = oracle.bwd_experts(*args, c["dY"])
    for name, got, ref in (("y", y, oracle.fwd(*args, c["b2"])), ("dx", g["dx"], dx),
                           ("dgate", g["dgate"], np.where(drop, 0, dgate)), ("dW1", g["dW1"], dW1),
                           ("db1", g["db1"], db1), ("dW2", g["dW2"], dW2), ("db2", g["db2"], db2)):
        assert nrm_err(host32(got), ref) <= TOL["bf16"], name
    assert not g["dgate"].cpu().numpy()[drop].any()
