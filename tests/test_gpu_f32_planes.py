"""The 64x64 and 128x64 tiles of the fp32 path, whose operands are split into three bf16 planes: sums of values of very different sizes,
values at the ends of the fp32 range, and infinities and NaN, whose tiles are multiplied on the fp32 instruction instead."""
import numpy as np
import pytest
import torch

from paper_2411_01288_amd import binding as B
from paper_2411_01288_amd.workloads import MoEWorkload, generate
from gpu_util import TOL, assert_tiles, host32, host_inputs, nrm_err, run_hip_layer

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# T, d, f of one expert and the launches on 128x64 tiles: none; fc2 and bwd_fc1; all but fc1
CLASSES = pytest.mark.parametrize("T,d,f,wide", [(5000, 560, 570, 0), (5000, 640, 704, 10), (3300, 1030, 1055, 14)])
# of three experts: fc1 and bwd_fc2 on 64x64 tiles, the others on 32x32; all but fc1 on 128x64
WORKLOADS = pytest.mark.parametrize("sizes", [(6001, 229, 517, [64, 32, 64, 32], 0), (3300, 1030, 1055, [64, 64, 64, 64], 14)])


def workload(sizes):
    T, d, f, tiles, wide = sizes
    w = MoEWorkload("planes", T, d, f, 3, 1, "f32", "topk", 77)            # rows at any dword alignment, ragged ends
    assert_tiles(w, tiles, wide)
    return w, generate(w, DEV)


@CLASSES
def test_many_decades(T, d, f, wide):
    """All launches against fp64 torch, one expert: errors of a few roundings per sum."""
    w = MoEWorkload("decades", T, d, f, 1, 1, "f32", "topk", 5)
    assert_tiles(w, [64, 64, 64, 64], wide)
    data = generate(w, DEV)
    scale = torch.logspace(-6, 6, w.d_model, device=DEV)                   # features over twelve decades
    data["x"] *= scale
    data["W1"] /= scale[None, :, None]
    # (smooth: of some three million pre-activations one or two lie within a rounding, 2^-24, of zero, where ReLU' takes the other side)
    _, y, g = run_hip_layer(w, data, activation=B.ACT_SILU)
    d = {k: v.double() for k, v in data.items() if k != "topk_idx"}
    pre = d["x"] @ d["W1"][0] + d["b1"][0]
    s = torch.sigmoid(pre)
    h = pre * s
    o = h @ d["W2"][0] + d["b2"][0]
    do = d["gate"] * d["dY"]
    dpre = (do @ d["W2"][0].t()) * s * (1 + pre * (1 - s))
    ref = {"y": d["gate"] * o, "dx": dpre @ d["W1"][0].t(), "dW1": (d["x"].t() @ dpre)[None], "dW2": (h.t() @ do)[None],
           "db1": dpre.sum(0)[None], "db2": do.sum(0)[None]}
    got = {"y": y, **g}
    for name, r in ref.items():
        if name in ("dx", "dW1"):                                          # on the scale of each feature
            s = scale.double() if name == "dx" else 1 / scale.double()[None, :, None]
            r, v = r * s, got[name].double() * s
        else:
            v = got[name].double()
        # a sum of K products is off by at most about sqrt(K) roundings of 2^-24 of its size, K <= 5000
        assert float((v - r).norm() / r.norm()) <= 70 * 2.0 ** -24, name


# the largest finite values; values whose last bit is still a multiple of 2^-133, the smallest number of the third plane
@pytest.mark.parametrize("big,weight", [(3.4e38, 1e-32), (2e-33, 1e33)])
@WORKLOADS
def test_ends_of_the_range(oracle, sizes, big, weight):
    w, data = workload(sizes)
    data["x"][:, 7] = 0.0
    data["x"][100] = 0.0
    data["x"][100, 7] = big
    data["W1"][:, 7] = torch.randn(w.E, w.d_ff, device=DEV) * weight
    _, y, _ = run_hip_layer(w, data)
    c = host_inputs(data)
    ref = oracle.fwd(c["x"], c["topk_idx"], c["gate"], c["W1"], c["b1"], c["W2"], c["b2"])
    rest = np.arange(w.T) != 100
    assert nrm_err(host32(y)[rest], ref[rest]) <= TOL["f32"]
    assert nrm_err(host32(y[100]), ref[100]) <= TOL["f32"]


def rounding(got, ref, mag):
    """Errors of sums of products as (largest, root mean square), relative to the sums of the products' sizes `mag`."""
    e = ((got.double() - ref).abs() / mag).flatten()
    return float(e.max()), float(e.square().mean().sqrt())


# bits below 2^-133 have no place in the planes
@pytest.mark.parametrize("scale", [1e-34, 1e-36, 1e-38])
@CLASSES
def test_tiny_operands(scale, T, d, f, wide):
    w = MoEWorkload("tiny", T, d, f, 1, 1, "f32", "topk", 6)
    assert_tiles(w, [64, 64, 64, 64], wide)
    data = generate(w, DEV)
    data["W1"].zero_()
    data["b1"] = data["b1"].abs() + 100.0                                  # h = b1, exactly
    data["W2"] *= 1e4                                                      # (products stay in the normal range)
    data["dY"] *= scale
    data["gate"].fill_(1.0)
    _, _, g = run_hip_layer(w, data, activation=B.ACT_RELU)
    x, dY, W2 = data["x"].double(), data["dY"].double(), data["W2"][0].double()
    h = data["b1"].double().expand(w.T, -1)
    # K roundings of 2^-24 of a sum on the way make about sqrt(K) of them, K <= 5000, so these are far from bounds for fp32 sums
    for name, got, ref, mag in (("dW2", g["dW2"][0], h.t() @ dY, h.t() @ dY.abs()),
                                ("db1", g["db1"][0], (dY @ W2.t()).sum(0), (dY.abs() @ W2.abs().t()).sum(0)),
                                ("dW1", g["dW1"][0], x.t() @ (dY @ W2.t()), x.abs().t() @ (dY.abs() @ W2.abs().t()))):
        top, rms = rounding(got, ref, mag)
        assert top <= 16 * 2.0 ** -24 and rms <= 2 * 2.0 ** -24, (name, top, rms)


def randn(gen, *shape):
    return torch.randn(shape, generator=gen, device=DEV)


def make(T, d, f, E, seed, tiles, wide=0):
    w = MoEWorkload("made", T, d, f, E, 1, "f32", "topk", seed)
    assert_tiles(w, tiles, wide)
    data = generate(w, DEV)
    data["gate"].fill_(1.0)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    return w, data, gen


# A sum of K products is off by at most K roundings of 2^-24 of the products' sizes.  A rounding is at most 2^-24 / sqrt(3) in the root mean
# square, and all K together make no more: the partial sums that are rounded grow like a square root, the sizes add up.
# 32 is the longest contraction that is not split, 64 and 65 are two steps and the first row of a third.
# (On 128x64 tiles, which take many rows per expert: three experts of `rows` rows, the others' on a fourth.)
@pytest.mark.parametrize("rows,T,size,E,wide", [(r, 64 * r, 704, 64, 0) for r in (1, 2, 3, 4, 8, 31, 32, 33, 64, 65)] + [(r, 4300, 1024, 4, 14) for r in (1, 32, 33, 64, 65)])
def test_short_token_contractions(rows, T, size, E, wide):
    w, data, _ = make(T, size, size, E, rows, [64, 64, 64, 64], wide)
    n = min(T, rows * (E if wide == 0 else E - 1)) // rows                  # experts of `rows` rows
    data["topk_idx"] = torch.where(torch.arange(T, device=DEV) < n * rows, torch.arange(T, device=DEV) % n, E - 1).to(torch.int32).view(T, 1).contiguous()
    data["W1"].zero_()
    data["b1"] = data["b1"].abs() + 0.5                                     # h = b1, exactly
    data["W2"].copy_(torch.eye(size, device=DEV))                           # dpre = dY, exactly
    _, _, g = run_hip_layer(w, data, activation=B.ACT_RELU)
    x, dY = (data[n_][:n * rows].double().view(rows, n, size) for n_ in ("x", "dY"))
    h = data["b1"][:n].double()[:, :, None]
    for name, ref, mag in (("dW1", torch.matmul(x.permute(1, 2, 0).contiguous(), dY.permute(1, 0, 2).contiguous()),
                            torch.matmul(x.abs().permute(1, 2, 0).contiguous(), dY.abs().permute(1, 0, 2).contiguous())),
                           ("dW2", h * dY.sum(0)[:, None, :], h * dY.abs().sum(0)[:, None, :])):
        top, rms = rounding(g[name][:n], ref, mag)
        assert top <= rows * 2.0 ** -24 and rms <= 0.58 * 2.0 ** -24, (name, top, rms)


@pytest.mark.parametrize("K", [1, 2, 3, 4, 8, 31, 32, 33, 64, 65])
def test_short_row_contractions(K):
    w, data, gen = make(4096, K, 1024, 1, K, [64, 32, 64, 32])
    pick = torch.randperm(1024, generator=gen, device=DEV)[:K]
    one_hot = torch.zeros(K, 1024, device=DEV)
    one_hot[torch.arange(K, device=DEV), pick] = 1.0
    # y: some columns of relu(x W1)
    data["W1"], data["W2"] = randn(gen, 1, K, 1024), one_hot.t().contiguous()[None]
    data["b1"].zero_(), data["b2"].zero_()
    _, y, _ = run_hip_layer(w, data, activation=B.ACT_RELU)
    x, W1 = data["x"].double(), data["W1"][0][:, pick].double()
    on = x @ W1 > 0
    top, rms = rounding(y[on], (x @ W1)[on], (x.abs() @ W1.abs())[on])
    assert top <= K * 2.0 ** -24 and rms <= 0.58 * 2.0 ** -24, ("fc1", top, rms)
    # dx: some columns of dY W2^T
    data["W1"], data["W2"] = one_hot[None].contiguous(), randn(gen, 1, 1024, K)
    data["b1"].fill_(100.0)
    _, _, g = run_hip_layer(w, data, activation=B.ACT_RELU)
    dY, W2 = data["dY"].double(), data["W2"][0][pick].double().t()
    top, rms = rounding(g["dx"], dY @ W2, dY.abs() @ W2.abs())
    assert top <= K * 2.0 ** -24 and rms <= 0.58 * 2.0 ** -24, ("dgrad2", top, rms)


# Few products in a long contraction: a rounding of 2^-24 for each where the large products meet the sum and one for the small ones, and as much again
# for the dropped products (2^-24 at most).  Features of 1 + 2^-7 - 2^-23 have the most in the dropped planes if these are cut off.
@pytest.mark.parametrize("count,value", [(1, None), (1, 1 + 2.0 ** -7 - 2.0 ** -23), (2, None), (4, None), (16, None)])
def test_sparse_rows(count, value):
    w, data, gen = make(4096, 512, 1024, 1, 50 + count, [64, 32, 64, 32])
    x = torch.zeros(w.T, 512, device=DEV)
    for _ in range(count):
        at = torch.randint(0, 512, (w.T,), generator=gen, device=DEV)
        x[torch.arange(w.T, device=DEV), at] = randn(gen, w.T) if value is None else torch.full((w.T,), value, device=DEV)
    data["x"] = x
    pick = torch.randperm(1024, generator=gen, device=DEV)[:512]
    data["W1"] = randn(gen, 1, 512, 1024)
    if value is not None:
        data["W1"].copy_(torch.where(data["W1"] > 0, value, 0.5 * value))
    data["W2"] = torch.zeros(1, 1024, 512, device=DEV)
    data["W2"][0, pick, torch.arange(512, device=DEV)] = 1.0
    data["b1"].zero_(), data["b2"].zero_()
    _, y, _ = run_hip_layer(w, data, activation=B.ACT_RELU)
    W1 = data["W1"][0][:, pick].double()
    ref, mag = x.double() @ W1, x.double().abs() @ W1.abs()
    on = ref > 0
    top, rms = rounding(y[on], ref[on], mag[on])
    assert top <= 2 * count * 2.0 ** -24 and rms <= 0.58 * 2.0 ** -24, (top, rms)
    if value is None:                                                      # no side is preferred
        assert abs(float((y[on].double() - ref[on]).sum() / mag[on].sum())) <= 0.05 * 2.0 ** -24


# the same on 128x64 tiles, in fc2, whose other operand fc1 passes on as it is
@pytest.mark.parametrize("count,value", [(1, None), (1, 1 + 2.0 ** -7 - 2.0 ** -23), (2, None), (4, None), (16, None)])
def test_sparse_rows_on_wide_tiles(count, value):
    w, data, gen = make(5000, 640, 640, 1, 50 + count, [64, 64, 64, 64], 10)
    x = torch.zeros(w.T, 640, device=DEV)
    for _ in range(count):
        at = torch.randint(0, 640, (w.T,), generator=gen, device=DEV)
        x[torch.arange(w.T, device=DEV), at] = randn(gen, w.T).abs() if value is None else torch.full((w.T,), value, device=DEV)
    data["x"] = x
    data["W1"].copy_(torch.eye(640, device=DEV))
    data["W2"] = randn(gen, 1, 640, 640)
    if value is not None:
        data["W2"].copy_(torch.where(data["W2"] > 0, value, -0.5 * value))
    data["b1"].zero_(), data["b2"].zero_()
    _, y, _ = run_hip_layer(w, data, activation=B.ACT_RELU)
    W2 = data["W2"][0].double()
    ref, mag = x.double() @ W2, x.double() @ W2.abs()
    top, rms = rounding(y, ref, mag)
    assert top <= 2 * count * 2.0 ** -24 and rms <= 0.58 * 2.0 ** -24, (top, rms)
    if value is None:
        assert abs(float((y.double() - ref).sum() / mag.sum())) <= 0.05 * 2.0 ** -24


@pytest.mark.parametrize("T,d,f,wide", [(5000, 560, 570, 0), (5000, 608, 704, 10), (3300, 1030, 1055, 14)])   # 18, 19, 22 and 33 steps
def test_results_do_not_depend_on_the_place_in_the_batch(T, d, f, wide):
    w, data, _ = make(T, d, f, 1, 9, [64, 64, 64, 64], wide)
    data["x"], data["dY"] = (data[n][:1].expand(w.T, -1).contiguous() for n in ("x", "dY"))
    _, y, g = run_hip_layer(w, data)
    assert torch.equal(y, y[:1].expand_as(y)) and torch.equal(g["dx"], g["dx"][:1].expand_as(g["dx"]))


@pytest.mark.parametrize("d,wide", [(512, 0), (1024, 4)])
def test_column_sums_over_many_rows(d, wide):
    """db1 as a sum over 300000 results: what is cut off to one side in each of them adds up in it."""
    w, data, _ = make(300000, d, 256, 1, 10, [64, 64, 64, 64], wide)
    data["W1"].zero_(), data["b1"].fill_(1.0)                               # dpre = dY W2^T
    _, _, g = run_hip_layer(w, data, activation=B.ACT_RELU)
    ref = sum(c.double().sum(0) for c in data["dY"].split(50000)) @ data["W2"][0].double().t()
    err = g["db1"][0].double() - ref
    # A result is off by about 2^-23 of its size at random (errors of fp32 sums of 512 or 1024 products); so is their sum, and adding up 300000 is
    # good for three times that.  The mean over 256 columns is a sixteenth of one column's, four times which is allowed.
    rms = float(ref.square().mean().sqrt())
    assert float(err.square().mean().sqrt()) <= 5 * 2.0 ** -23 * rms
    assert abs(float(err.mean())) <= 1.25 * 2.0 ** -23 * rms


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
@WORKLOADS
def test_not_finite(value, sizes):
    w, data = workload(sizes)
    _, y0, g0 = run_hip_layer(w, data, activation=B.ACT_RELU)
    x = data["x"].clone()
    x[1234, 56] = value
    _, y, g = run_hip_layer(w, {**data, "x": x}, activation=B.ACT_RELU)
    # that row of y as fp32 arithmetic gives it: relu of +-inf hidden units (or NaN -> 0), then sums of +-inf
    e = int(data["topk_idx"][1234, 0])
    pre = x[1234].cpu() @ data["W1"][e].cpu() + data["b1"][e].cpu()
    h = torch.where(pre > 0, pre, torch.zeros_like(pre))
    ref = data["gate"][1234].cpu() * (h @ data["W2"][e].cpu() + data["b2"][e].cpu())
    got = y[1234].cpu()
    assert torch.equal(torch.isnan(got), torch.isnan(ref)) and torch.equal(torch.isposinf(got), torch.isposinf(ref))
    rest = torch.arange(w.T, device=DEV) != 1234
    # the other rows: a tile's rows may have been summed the other way, a few roundings apart
    assert float((y[rest] - y0[rest]).abs().max()) <= 2e-6 * float(y0.abs().max())
    others = [i for i in range(w.E) if i != e]
    assert torch.equal(g["dW1"][others], g0["dW1"][others]) and torch.isfinite(g["dx"][rest]).all()


@pytest.mark.parametrize("name,at,value", [("x", (1234, 56), float("inf")), ("x", (-1, -1), float("nan")), ("dY", (1234, 5), float("-inf")),
                                           ("dY", (64, -1), float("nan")), ("W1", (0, 56, 17), float("inf")), ("W2", (0, -1, 5), float("-inf"))])
@CLASSES
def test_not_finite_in_every_contraction(name, at, value, T, d, f, wide):
    """All launches: what is infinite, of which sign, and what is NaN in every output, and the rest as accurate
    as ever.  Columns of one sign in W2 keep infinities of y from meeting their opposites."""
    w, data, _ = make(T, d, f, 1, 12, [64, 64, 64, 64], wide)
    data["W2"][0, :, 0].abs_(), data["W2"][0, :, 1].abs_().neg_()
    # pre-activations are odd multiples of 2^-12, so that no rounding decides which hidden units are on
    data["x"] = torch.round(data["x"] * 8) / 8
    data["W1"] = torch.round(data["W1"] * 256) / 256
    data["b1"] = torch.round(data["b1"] * 2048) / 2048 + 2.0 ** -12
    data[name][at] = value
    _, y, g = run_hip_layer(w, data, activation=B.ACT_RELU)
    x, W1, b1, W2, b2, dY = (data[n].double() if n in ("x", "dY") else data[n][0].double() for n in ("x", "W1", "b1", "W2", "b2", "dY"))
    pre = x @ W1 + b1
    on = pre > 0                                                           # (NaN: off)
    h = torch.where(on, pre, torch.zeros_like(pre))
    dpre = (dY @ W2.t()) * on
    ref = {"y": h @ W2 + b2, "dx": dpre @ W1.t(), "dW1": x.t() @ dpre, "db1": dpre.sum(0), "dW2": h.t() @ dY, "db2": dY.sum(0)}
    reached = set()
    for n, r in ref.items():
        got = (y if n == "y" else g[n]).double().view_as(r)
        for kind in (torch.isnan, torch.isposinf, torch.isneginf):
            assert torch.equal(kind(got), kind(r)), (n, kind)
        fine = torch.isfinite(r)
        if not fine.all():
            reached.add(n)
        if fine.any():
            assert nrm_err(got[fine].cpu().numpy(), r[fine].cpu().numpy()) <= TOL["f32"], n
    assert reached >= {"x": {"dW1"}, "dY": {"dx", "dW1", "db1", "dW2", "db2"}, "W1": {"y", "dx", "dW2"}, "W2": {"y", "dx", "dW1", "db1"}}[name]


# 64x64 tiles; 128x64 tiles but for fc1; rows of every tensor at any alignment, segments of 2000 and 1100 rows (no whole number of steps)
@pytest.mark.parametrize("T,d,f,wide", [(6000, 517, 523, 0), (3300, 1030, 1055, 14)])
@pytest.mark.parametrize("value", [float("inf"), float("nan"), 1e-38])
def test_values_of_a_neighbour(T, d, f, wide, value):
    """A value that no plane holds changes no bit of what other experts' tokens or other columns of weights give, also where it lies
    behind the end of one of their rows in memory."""
    w = MoEWorkload("neighbour", T, d, f, 3, 1, "f32", "topk", 13)
    assert_tiles(w, [64, 64, 64, 64], wide)
    data = generate(w, DEV)
    ids = torch.arange(T, device=DEV) % 3
    data["topk_idx"] = ids.to(torch.int32).view(T, 1).contiguous()

    def run(name, at):
        for v in (0.0, value):
            t = data[name].clone()
            t[at] = v
            _, y, g = run_hip_layer(w, {**data, name: t})
            yield {"y": y, **g}

    for token in (0, 1501):
        base, got = run("x", (token, slice(0, 3)))
        e = int(ids[token])
        for n in base:
            others = ids != e if n in ("y", "dx", "dgate") else torch.arange(3, device=DEV) != e
            assert torch.equal(base[n][others], got[n][others]), (token, n)
        if value == value and value < 1:
            assert not torch.equal(base["dW1"][e], got["dW1"][e])           # (its own tiles are summed the other way)
    base, got = run("W2", (0, 5, 1))
    if value < 1:                                                           # (y past the first tile of columns; no sum sees 1e-38)
        assert torch.equal(base["y"][:, 128:], got["y"][:, 128:])
    base, got = run("dY", (1501, 1))
    assert torch.equal(base["dW2"][:, :, 128:], got["dW2"][:, :, 128:])
