"""ReLU and SiLU through the whole layer on the GPU against the oracle (GELU-tanh, the default, is what
every other GPU test runs), fp32 and bf16."""
import numpy as np
import pytest
import torch

from paper_2411_01288_amd.workloads import MoEWorkload, generate
from gpu_util import TOL, host32, host_inputs, nrm_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture
def oracle_act(oracle):
    def choose(kind):
        oracle.set_activation(kind)
        return oracle
    yield choose
    oracle.set_activation(0)


@pytest.mark.parametrize("dtype,T,d,f,E,k", [("f32", 200, 24, 40, 3, 2), ("bf16", 900, 128, 320, 6, 2),
                                             ("bf16", 3000, 256, 512, 7, 2)])
@pytest.mark.parametrize("kind", [1, 2])
def test_activation_parity(oracle_act, kind, dtype, T, d, f, E, k):
    from paper_2411_01288_amd import binding as B
    O = oracle_act(kind)
    w = MoEWorkload("act", T, d, f, E, k, dtype, "zipf", 70 + kind)
    data = generate(w, DEV)
    shape = B.make_shape(w.T, w.d_model, w.d_ff, w.E, w.k, w.dtype, activation=kind)
    idx = B.hexa_moe_index(shape, data["topk_idx"])
    ws = B.alloc_workspace(shape, DEV)
    y = B.hexa_moe_fwd(shape, data["x"], data["topk_idx"], data["gate"], data["W1"], data["b1"],
                       data["W2"], data["b2"], idx, ws)
    g = B.hexa_moe_bwd(shape, data["dY"], data["x"], data["topk_idx"], data["gate"], data["W1"],
                       data["W2"], idx, ws)
    torch.cuda.synchronize()
    c = host_inputs(data)
    args = (c["x"], c["topk_idx"], c["gate"], c["W1"], c["b1"], c["W2"])
    y_ref = O.fwd(*args, c["b2"])
    dx_ref, dg_ref = O.bwd_tokens(*args, c["b2"], c["dY"])
    dW1, db1, dW2, db2 = O.bwd_experts(*args, c["dY"])
    tol = TOL[dtype]
    for name, got, ref in (("y", y, y_ref), ("dx", g["dx"], dx_ref), ("dgate", g["dgate"], dg_ref),
                           ("dW1", g["dW1"], dW1), ("db1", g["db1"], db1), ("dW2", g["dW2"], dW2),
                           ("db2", g["db2"], db2)):
        assert nrm_err(host32(got), ref) <= tol, name
    # the three activations really differ: the GELU result is not within tolerance of this one
    shape0 = B.make_shape(w.T, w.d_model, w.d_ff, w.E, w.k, w.dtype)
    y0 = B.hexa_moe_fwd(shape0, data["x"], data["topk_idx"], data["gate"], data["W1"], data["b1"],
                        data["W2"], data["b2"], idx, ws)
    torch.cuda.synchronize()
    assert nrm_err(host32(y0), y_ref) > 2.5 * tol


@pytest.mark.parametrize("lo,hi", [(-0.1, 0.1), (-1, 1), (-6, -1), (1, 6), (-40, 40)])
def test_f32_gelu_and_its_derivative(lo, hi):
    """One feature, one hidden unit, weights of one: y is F(x) and dx is F'(x), against fp64."""
    from paper_2411_01288_amd import binding as B
    T = 20001
    x = torch.empty(T, 1, device=DEV).uniform_(lo, hi, generator=torch.Generator(device=DEV).manual_seed(3))
    shape = B.make_shape(T, 1, 1, 1, 1, "f32")
    ones, zeros = torch.ones(T, 1, device=DEV), torch.zeros(1, 1, device=DEV)
    ids, W = torch.zeros(T, 1, dtype=torch.int32, device=DEV), ones[:1].view(1, 1, 1)
    idx, ws = B.hexa_moe_index(shape, ids), B.alloc_workspace(shape, DEV)
    y = B.hexa_moe_fwd(shape, x, ids, ones, W, zeros, W, zeros, idx, ws)
    g = B.hexa_moe_bwd(shape, ones, x, ids, ones, W, W, idx, ws)["dx"]
    u = x.double()
    t = 2 * (2 / np.pi) ** 0.5 * (u + 0.044715 * u ** 3)
    s, s1 = torch.sigmoid(t), torch.sigmoid(-t)
    q = 2 * (2 / np.pi) ** 0.5 * (1 + 3 * 0.044715 * u ** 2)
    # the smaller of s and 1 - s is off by 4 roundings of 2^-24 (instructions of 1 ulp) and by those of t, |t| of them; then one or two more
    off = (4 + t.abs()) * torch.minimum(s, s1) + torch.maximum(s, s1)
    assert ((y.double() - u * s).abs() <= 2.0 ** -24 * u.abs() * (off + s) + 1e-26).all()
    assert ((g.double() - (s + u * s * s1 * q)).abs() <= 2.0 ** -24 * (off + u.abs() * q * (off * s + (off + 3 * s) * s1) + 1) + 1e-26).all()


def test_f32_gelu_far_out():
    """Finite pre-activations up to the ends of fp32: F is u or 0, F' 1 or 0; at infinities F' is NaN as in the formula (0 times infinity)."""
    from paper_2411_01288_amd import binding as B
    far = torch.cat([torch.logspace(1.2, 38.5, 3001, device=DEV), torch.tensor([1.8446744e19, 1.85e19, 2e19, 5.04e19, 5.1e19, 3.4028234e38], device=DEV)])
    x = torch.cat([far, -far, torch.tensor([float("inf"), float("-inf"), float("nan")], device=DEV)]).view(-1, 1)
    T = x.shape[0]
    shape = B.make_shape(T, 1, 1, 1, 1, "f32")
    ones, zeros = torch.ones(T, 1, device=DEV), torch.zeros(1, 1, device=DEV)
    ids, W = torch.zeros(T, 1, dtype=torch.int32, device=DEV), ones[:1].view(1, 1, 1)
    idx, ws = B.hexa_moe_index(shape, ids), B.alloc_workspace(shape, DEV)
    y = B.hexa_moe_fwd(shape, x, ids, ones, W, zeros, W, zeros, idx, ws)[:, 0]
    g = B.hexa_moe_bwd(shape, ones, x, ids, ones, W, W, idx, ws)["dx"][:, 0]
    n = far.numel()
    assert torch.equal(y[:n], far) and (g[:n] == 1).all()
    assert (y[n:2 * n] == 0).all() and (g[n:2 * n] == 0).all()
    assert torch.isposinf(y[-3]) and torch.isnan(y[-2:]).all() and torch.isnan(g[-3:]).all()
