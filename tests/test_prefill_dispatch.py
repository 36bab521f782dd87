"""Which decoder layers run in the one-pass kernels and which in the tensor
operations, on the CPU: the kernels are replaced by stand-ins that compute the
same outside of autograd and of any tracing, as a call into the library does,
and the device test is the CPU's.  Everything a tensor operation would record
has to be recorded."""
import ctypes

import pytest
import torch
from torch.fx.experimental.proxy_tensor import make_fx
from torch.overrides import TorchFunctionMode
from torch.utils._python_dispatch import TorchDispatchMode

from paper_2606_09508_amd import prefill as pf

SHAPE = pf.DecoderShape(hidden=64, n_q_heads=2, n_kv_heads=1, intermediate=48, n_layers=2)
N = 6


def _opaque(fn, calls):
    """fn as a library call sees it: on raw memory, recorded by nothing."""
    def call(*args, **kw):
        calls.append(fn.__name__)
        with torch.no_grad():
            return fn(*(a.detach() if isinstance(a, torch.Tensor) else a for a in args), **kw)
    return call


def _add_rmsnorm(x, y, gain, eps):
    assert y is None or (y.shape == x.shape and y.dtype == x.dtype)
    s = x if y is None else x + y
    return s, pf._rmsnorm(s, gain, eps)


def _rope_heads(q, k, v, cos, sin):
    assert q.dtype == k.dtype == v.dtype == torch.bfloat16
    q, k, v = (t.transpose(1, 2).contiguous() for t in (q, k, v))
    return [pf._rope(q, cos, sin), pf._rope(k, cos, sin), v]


def _swiglu(g, u, out=None):
    return torch.nn.functional.silu(g) * u


def _tables(cos, sin, head_dim, theta):
    assert 0 < cos.shape[0] < 2 ** 31 and 0 < ctypes.c_float(theta).value < float("inf")
    inv = 1.0 / (theta ** (torch.arange(0, head_dim, 2, dtype=torch.float32) / head_dim))
    ang = torch.arange(cos.shape[0], dtype=torch.float32)[:, None] * inv
    cos.copy_(torch.cos(ang))
    sin.copy_(torch.sin(ang))


@pytest.fixture
def kernels(monkeypatch):
    """The stand-ins in the kernels' place; the list of the calls made."""
    calls = []
    for name, fn in (("add_rmsnorm", _add_rmsnorm), ("rope_heads", _rope_heads),
                     ("swiglu", _swiglu), ("rope_tables", _tables)):
        monkeypatch.setattr(pf.eb, name, _opaque(fn, calls))
    monkeypatch.setattr(pf, "_kernel_device", lambda dev: dev.type == "cpu")
    return calls


def _attn(q, k, v):
    """A caller's own attention, of tensor operations."""
    g = q.shape[1] // k.shape[1]
    k, v = (t.repeat_interleave(g, 1).float() for t in (k, v))
    s = torch.matmul(q.float(), k.transpose(2, 3).contiguous()) / 128 ** 0.5
    s = s.masked_fill(torch.ones(s.shape[-2:], dtype=torch.bool).triu(1), float("-inf"))
    return torch.matmul(torch.softmax(s, -1), v).to(q.dtype)


def _inputs(seed=0):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn((1, N, SHAPE.hidden), generator=g).to(torch.bfloat16)
    return x, pf.make_weights(SHAPE, 2, 3, torch.device("cpu"))


def _same(a, b):
    assert a.dtype == b.dtype and a.shape == b.shape
    # (bf16 between the operations of two layers)
    assert float((a.double() - b.double()).norm()) <= 2e-2 * float(b.double().norm())


def test_plain_layers_take_the_kernels(kernels):
    x, layers = _inputs()
    with torch.no_grad():
        pf.prefill(x, layers, SHAPE, _attn)
    assert len(kernels) == 2 * 4 + 2   # two norms, rotary, SwiGLU a layer; tables, last norm


@pytest.mark.parametrize("name", ["wo", "norm2", "w_gate", "w_up", "w_down"])
def test_gradients_cross_into_a_frozen_layer(kernels, monkeypatch, name):
    """One weight of the first layer is trained and the second layer is frozen:
    the summand that the second layer's norm adds carries the gradient."""
    x, layers = _inputs()
    grads = []
    for tensor_ops in (False, True):
        if tensor_ops:
            monkeypatch.setattr(pf, "_kernel_device", lambda dev: False)
        w = layers[0][name] = layers[0][name].detach().requires_grad_()
        last, _ = pf.prefill(x, layers, SHAPE, _attn)
        assert last.requires_grad
        last.float().square().sum().backward()
        grads.append(w.grad)
    _same(*grads)
    assert float(grads[0].float().abs().max()) > 0.0


@pytest.mark.parametrize("name", ["wo", "w_down"])
def test_summand_that_broadcasts(kernels, monkeypatch, name):
    """A projection to one column is added to every column, as x + y does."""
    x, layers = _inputs()
    layers[0][name] = layers[0][name][:, :1].contiguous()
    with torch.no_grad():
        got = pf.prefill(x, layers, SHAPE, _attn)[0]
        monkeypatch.setattr(pf, "_kernel_device", lambda dev: False)
        _same(got, pf.prefill(x, layers, SHAPE, _attn)[0])


def _run(x, layers):
    with torch.no_grad():
        return pf.prefill(x, layers, SHAPE, _attn)[0]


class _CountDispatch(TorchDispatchMode):
    seen = 0

    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        self.seen += func is torch.ops.aten.rsqrt.default
        return func(*args, **(kwargs or {}))


class _CountFunction(TorchFunctionMode):
    seen = 0

    def __torch_function__(self, func, types, args=(), kwargs=None):
        self.seen += func is torch.rsqrt
        return func(*args, **(kwargs or {}))


@pytest.mark.parametrize("tracer", ["jit", "fx"])
def test_tracers_record_every_operation(kernels, tracer):
    """A layer traced with one input computes the layer of another one."""
    x, layers = _inputs()
    if tracer == "jit":
        traced = torch.jit.trace(lambda t: _run(t, layers), x, check_trace=False)
    else:
        traced = make_fx(lambda t: _run(t, layers))(x)
    assert kernels == []
    other = _inputs(1)[0]
    _same(traced(other), _run(other, layers))


@pytest.mark.parametrize("mode", [_CountDispatch, _CountFunction])
def test_modes_see_every_operation(kernels, mode):
    x, layers = _inputs()
    with mode() as m:
        _run(x, layers)
    assert kernels == [] and m.seen == 2 * 2 + 1   # the norms


def test_default_device_keeps_the_kernels(kernels):
    x, layers = _inputs()
    with torch.device("cpu"):
        _run(x, layers)
    assert len(kernels) == 2 * 4 + 2


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_autocast(kernels, monkeypatch, dtype):
    """Under autocast the products are of its type, whatever the weights' is."""
    x, layers = _inputs()
    with torch.autocast("cpu", dtype=dtype):
        got = _run(x, layers)
        monkeypatch.setattr(pf, "_kernel_device", lambda dev: False)
        _same(got, _run(x, layers))


@pytest.mark.parametrize("device", [None, "cpu", torch.device("cpu")], ids=str)
@pytest.mark.parametrize("theta", [1e4, 500000, 1e-46, 1e39])
def test_rope_tables_arguments(monkeypatch, device, theta):
    """Every device and theta the tensor operations take."""
    ref = pf.rope_tables(3, 128, theta, torch.device("cpu"))
    monkeypatch.setattr(pf, "_kernel_device", lambda dev: dev.type == "cpu")
    monkeypatch.setattr(pf.eb, "rope_tables", _tables)
    for a, b in zip(pf.rope_tables(3, 128, theta, device), ref):
        assert torch.equal(a.nan_to_num(), b.nan_to_num()) and a.dtype == b.dtype


@pytest.mark.parametrize("N,D", [(2 ** 31, 2), (2 ** 32 + 5, 2), (1, 2 ** 31), (0, 128)])
def test_rope_tables_of_64_bit_sizes_stay_off_the_kernel(N, D):
    """(ei_rope_tables counts positions and dimensions in 32 bits.)"""
    assert not pf._tables_fit(N, D, 1e4) and pf._tables_fit(2 ** 31 - 1, 128, 1e4)
