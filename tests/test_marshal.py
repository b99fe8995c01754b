"""The argument checks of a pass's calls (csrc/marshal.cpp): what was refused stays refused, with _ptr's errors, and what was
taken (tensor subclasses, an active function mode, None for an optional output) stays taken."""
import ctypes
import sysconfig

import pytest
import torch

from paper_2411_01288_amd import binding as B

T, D, F, E, K = 8, 64, 128, 4, 2


def test_host_tensors_and_other_objects_are_refused():
    shape = B.make_shape(T, D, F, E, K, "bf16")
    ids = torch.zeros(T, K, dtype=torch.int32)
    idx = {n: torch.zeros(1, dtype=torch.int32) for n in ("counts", "offsets", "perm", "inv")}
    with pytest.raises(ValueError, match="topk_idx: need a contiguous device tensor"):
        B._marshal.index(shape, ids, idx, ids, 0)
    with pytest.raises(ValueError, match="counts"):
        B._marshal.index(shape, None, idx, ids, 0)
    with pytest.raises(KeyError):
        B._marshal.index(shape, None, {}, ids, 0)
    with pytest.raises(AttributeError):
        B._marshal.index(shape, 5, idx, ids, 0)
    with pytest.raises(TypeError):
        B._marshal.index((T, D, F, E, K, 1, 0), ids, idx, ids, 0)
    with pytest.raises(TypeError):
        B._marshal.index(shape, ids, idx, ids)
    with pytest.raises(KeyError):
        B._marshal.fwd(B.make_shape(T, D, F, E, K, 7), *[None] * 7, idx, ids, None, 0)


def test_none_reaches_the_library():
    shape = B.make_shape(T, D, F, E, K, "bf16")
    none = {n: None for n in ("counts", "offsets", "perm", "inv")}
    assert B._marshal.index(shape, None, none, torch.zeros(4), 0) == 1


def test_a_module_for_another_torch_or_python_is_refused(monkeypatch):
    assert B._marshal.torch == torch.__version__
    assert B._marshal.__file__.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    monkeypatch.setattr(torch, "__version__", "1.0")
    with pytest.raises(ImportError, match="was built for torch .* build it with"):
        B._load_marshal()


def layer(dev="cuda:0"):
    gen = torch.Generator(device=dev).manual_seed(3)
    r = lambda *s, dtype=torch.bfloat16: torch.randn(s, generator=gen, device=dev).to(dtype)
    return {"x": r(T, D), "topk_idx": torch.randint(0, E, (T, K), generator=gen, device=dev, dtype=torch.int32),
            "gate": r(T, K, dtype=torch.float32), "W1": r(E, D, F), "b1": r(E, F), "W2": r(E, F, D), "b2": r(E, D)}


def fwd(a, **other):
    a = {**a, **other}
    shape = B.make_shape(T, D, F, E, K, "bf16")
    idx = B.hexa_moe_index(shape, a["topk_idx"])
    return B.hexa_moe_fwd(shape, *(a[n] for n in ("x", "topk_idx", "gate", "W1", "b1", "W2", "b2")), idx,
                          B.alloc_workspace(shape, "cuda:0"))


@pytest.mark.gpu
def test_wrong_tensors_are_refused():
    a = layer()
    for name, bad in (("x", a["x"][:, :32]), ("x", a["x"].t().contiguous().t()), ("x", a["x"].float()), ("x", a["x"].cpu()),
                      ("gate", a["gate"].reshape(K, T)), ("W1", a["W1"].reshape(E, F, D)), ("b2", a["b2"].half())):
        with pytest.raises(ValueError, match=f"^{name}: "):
            fwd(a, **{name: bad})
    with pytest.raises(B.HexaError):
        fwd(a, b1=None)


@pytest.mark.gpu
def test_subclasses_and_function_modes_are_taken():
    class Tagged(torch.Tensor):
        pass

    class Mode(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    a = layer()
    y = fwd(a)
    assert torch.isfinite(y.float()).all()
    assert torch.equal(fwd(a, W1=a["W1"].as_subclass(Tagged), b1=torch.nn.Parameter(a["b1"])), y)
    with Mode():
        assert torch.equal(fwd(a), y)


@pytest.mark.gpu
def test_equals_the_call_through_ctypes():
    a = layer()
    shape = B.make_shape(T, D, F, E, K, "bf16")
    idx = B.hexa_moe_index(shape, a["topk_idx"])
    ws, y = B.alloc_workspace(shape, "cuda:0"), torch.empty_like(a["x"])
    p = [a[n].data_ptr() for n in ("x", "topk_idx", "gate", "W1", "b1", "W2", "b2")]
    assert B.lib.hexa_moe_fwd(ctypes.byref(shape), *p, B._idx_struct(shape, idx), y.data_ptr(), ws.data_ptr(), ws.numel(),
                              B._stream()) == 0
    assert torch.equal(fwd(a), y)
