"""The fp32 path where x, or a weight matrix, has more bytes than 32-bit offsets reach (its tiles then compute 64-bit addresses), against
fp64 torch: rows at both ends and across the line, and the weight gradients, which read all of them."""
import pytest
import torch

from paper_2411_01288_amd import binding as B
from paper_2411_01288_amd.workloads import MoEWorkload, generate
from gpu_util import TOL, assert_tiles, nrm_err, run_hip_layer

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_x_of_more_than_4_gb():
    w = MoEWorkload("far", 1080001, 1001, 7, 2, 1, "f32", "topk", 3)
    assert 4 * w.T * w.d_model > 2 ** 32
    data = generate(w, DEV)
    _, y, g = run_hip_layer(w, data, activation=B.ACT_RELU)
    W1, b1, W2, b2 = (data[n].double() for n in ("W1", "b1", "W2", "b2"))
    dW1, dW2 = torch.zeros_like(W1), torch.zeros_like(W2)
    line = 2 ** 30 // w.d_model
    for i0 in range(0, w.T, 50000):
        x, dY, gate, e = (data[n][i0:i0 + 50000] for n in ("x", "dY", "gate", "topk_idx"))
        for ex in range(w.E):
            at = (e[:, 0] == ex).nonzero()[:, 0]
            xe, do = x[at].double(), gate[at].double() * dY[at].double()
            pre = xe @ W1[ex] + b1[ex]
            dpre = (do @ W2[ex].t()) * (pre > 0)
            dW1[ex] += xe.t() @ dpre
            dW2[ex] += torch.relu(pre).t() @ do
            if i0 == 0 or i0 + 50000 >= w.T or i0 <= line < i0 + 50000:
                ref = gate[at].double() * (torch.relu(pre) @ W2[ex] + b2[ex])
                assert nrm_err(y[i0:i0 + 50000][at].cpu().numpy(), ref.cpu().numpy()) <= TOL["f32"], (i0, ex)
                assert nrm_err(g["dx"][i0:i0 + 50000][at].cpu().numpy(), (dpre @ W1[ex].t()).cpu().numpy()) <= TOL["f32"], (i0, ex)
    for n, ref in (("dW1", dW1), ("dW2", dW2)):
        assert nrm_err(g[n].cpu().numpy(), ref.cpu().numpy()) <= TOL["f32"], n


def test_weights_of_more_than_4_gb():
    w = MoEWorkload("far", 100, 33001, 32999, 1, 1, "f32", "topk", 4)
    assert 4 * w.d_model * w.d_ff > 2 ** 32
    assert_tiles(w, [64, 64, 64, 64])
    data = generate(w, DEV)
    _, y, g = run_hip_layer(w, data, activation=B.ACT_RELU)
    x, b1, W1, b2 = (data[n].double() for n in ("x", "b1", "W1", "b2"))
    do = data["gate"].double() * data["dY"].double()
    pre = x @ W1[0] + b1[0]
    h = torch.relu(pre)
    W2 = data["W2"][0].double()
    dpre = (do @ W2.t()) * (pre > 0)
    ref = {"y": data["gate"].double() * (h @ W2 + b2[0]), "dx": dpre @ W1[0].t()}
    del W1, W2
    for n, r in ref.items():
        assert nrm_err((y if n == "y" else g[n]).cpu().numpy(), r.cpu().numpy()) <= TOL["f32"], n
    for n, a, b in (("dW1", x, dpre), ("dW2", h, do)):
        r = a.t() @ b
        assert float((g[n][0] - r).abs().max() / r.abs().max()) <= TOL["f32"], n
