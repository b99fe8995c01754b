"""The fp32 path where x has more bytes than 32-bit offsets reach (its tiles then compute 64-bit addresses): rows at both ends and across the
line, and the weight gradient that gathers all of them, against fp64 torch."""
import pytest
import torch

from paper_2411_01288_amd import binding as B
from paper_2411_01288_amd.workloads import MoEWorkload, generate
from gpu_util import TOL, nrm_err, run_hip_layer

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_x_of_more_than_4_gb():
    w = MoEWorkload("far", 1080001, 1001, 7, 2, 1, "f32", "topk", 3)
    assert 4 * w.T * w.d_model > 2 ** 32
    data = generate(w, DEV)
    _, y, g = run_hip_layer(w, data, activation=B.ACT_RELU)
    W1, b1, W2, b2 = (data[n].double() for n in ("W1", "b1", "W2", "b2"))
    dW1 = torch.zeros_like(W1)
    line = 2 ** 30 // w.d_model
    for i0 in range(0, w.T, 50000):
        x, dY, gate, e = (data[n][i0:i0 + 50000] for n in ("x", "dY", "gate", "topk_idx"))
        for ex in range(w.E):
            at = (e[:, 0] == ex).nonzero()[:, 0]
            xe, do = x[at].double(), gate[at].double() * dY[at].double()
            pre = xe @ W1[ex] + b1[ex]
            dW1[ex] += xe.t() @ ((do @ W2[ex].t()) * (pre > 0))
            if i0 == 0 or i0 + 50000 >= w.T or i0 <= line < i0 + 50000:
                ref = gate[at].double() * (torch.relu(pre) @ W2[ex] + b2[ex])
                assert nrm_err(y[i0:i0 + 50000][at].cpu().numpy(), ref.cpu().numpy()) <= TOL["f32"], (i0, ex)
    assert nrm_err(g["dW1"].cpu().numpy(), dW1.cpu().numpy()) <= TOL["f32"]
