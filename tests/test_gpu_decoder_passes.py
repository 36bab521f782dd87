"""The one-pass decoder kernels (residual sum + RMSNorm, rotary embedding to
head-major layout, SwiGLU) against the tensor operations in float64 on the CPU
over the same bf16 roundings, at the edges of their tiles."""
import pytest
import torch

from paper_2606_09508_amd import binding as eb
from paper_2606_09508_amd import prefill as pf

pytestmark = pytest.mark.gpu

# bf16 keeps 8 significant bits: rounding moves a value by at most half a step,
# 2^-8 of it.  A result rounded once from fp32 arithmetic (good to ~1e-6) is
# within 1.001 half steps of the unrounded float64 value.
HALF = 2.0 ** -8


def _rand(shape, seed, scale=1.0):
    g = torch.Generator().manual_seed(seed)
    return (torch.randn(shape, generator=g) * scale).to(torch.bfloat16)


def _close(got, ref, halves=1.001, floor=0.0):
    got, ref = got.double().cpu(), ref.double()
    assert torch.equal(got.isnan(), ref.isnan())
    err = (got - ref).abs().nan_to_num(0.0)
    assert bool((err <= halves * HALF * ref.abs().nan_to_num(0.0) + floor).all()), float(err.max())


# columns: below, at and past each of the kernel's row splits
@pytest.mark.parametrize("cols", [8, 504, 512, 520, 1024, 1032, 2048, 3584, 4096, 4104, 8200, 16384])
@pytest.mark.parametrize("rows", [1, 3, 5])
def test_add_rmsnorm(rows, cols):
    x, y, g = _rand((rows, cols), 1, 3.0), _rand((rows, cols), 2), _rand((cols,), 3)
    for add in (False, True):
        s, h = eb.add_rmsnorm(x.cuda(), y.cuda() if add else None, g.cuda(), 1e-5)
        ref_s = (x.float() + y.float()).to(torch.bfloat16) if add else x
        assert torch.equal(s.cpu(), ref_s)
        d = ref_s.double()
        _close(h, d * torch.rsqrt((d * d).mean(-1, keepdim=True) + 1e-5) * g.double())


@pytest.mark.parametrize("cols", [520, 4096, 16384])   # a wave's row, a workgroup's, the longest
@pytest.mark.parametrize("into", ["x", "y"])
def test_add_rmsnorm_in_place(cols, into):
    """The C entry writing the sum over one of its operands."""
    x, y, g = (_rand(s, i).cuda() for i, s in enumerate([(3, cols), (3, cols), (cols,)]))
    s_ref, h_ref = eb.add_rmsnorm(x, y, g, 1e-5)
    s, h = (x if into == "x" else y), torch.empty_like(x)
    assert eb.lib().ei_add_rmsnorm(x.data_ptr(), y.data_ptr(), g.data_ptr(), 3, cols, 1e-5,
                                   s.data_ptr(), h.data_ptr(), eb._stream(x)) == 0
    assert torch.equal(s, s_ref) and torch.equal(h, h_ref)


@pytest.mark.parametrize("N,D,theta", [(1, 128, 500000.0), (3, 2, 10000.0), (1000, 128, 500000),
                                       (131072, 128, 500000.0), (257, 96, 1e4)])
def test_rope_tables(N, D, theta):
    """The one-launch tables against the tensor operations on the same device:
    the same fp32 functions in the same order, so bitwise equal."""
    cos, sin = pf.rope_tables(N, D, theta, torch.device("cuda:0"))
    inv = 1.0 / (theta ** (torch.arange(0, D, 2, device="cuda", dtype=torch.float32) / D))
    ang = torch.arange(N, device="cuda", dtype=torch.float32)[:, None] * inv[None, :]
    assert torch.equal(cos, torch.cos(ang)) and torch.equal(sin, torch.sin(ang))


def _edges(n, step):
    """Slices at both ends of n rows and around every multiple of step."""
    return [slice(max(at - 500, 0), min(at + 500, n)) for at in [*range(0, n, step), n]]


def test_add_rmsnorm_of_more_rows_than_a_launch_takes():
    """A launch takes fewer than 2^32 threads, here 2^26 rows."""
    rows, cols = 2 ** 26 + 5, 8
    x, y = (_rand((4099, cols), 5 + i).cuda().repeat(rows // 4099 + 1, 1)[:rows] for i in range(2))
    g = _rand((cols,), 3).cuda()
    s, h = eb.add_rmsnorm(x, y, g, 1e-5)
    for part in _edges(rows, 2 ** 25):
        ref = eb.add_rmsnorm(x[part], y[part], g, 1e-5)
        assert torch.equal(s[part], ref[0]) and torch.equal(h[part], ref[1]), part


def test_rope_heads_of_more_sequences_than_a_launch_takes():
    B = 2 ** 24 + 3
    q, k, v = (_rand((4099, 1, 1, 128), 4 + i).cuda().repeat(B // 4099 + 1, 1, 1, 1)[:B]
               for i in range(3))
    cos, sin = pf.rope_tables(2, 128, 1e4, torch.device("cuda:0"))
    cos, sin = cos[1:], sin[1:]
    got = eb.rope_heads(q, k, v, cos, sin)
    for part in _edges(B, 2 ** 23):
        for a, b in zip(got, eb.rope_heads(q[part], k[part], v[part], cos, sin)):
            assert torch.equal(a[part], b), part
    del q, k, v, got
    torch.cuda.empty_cache()   # (26 GB)


def test_rope_tables_of_more_values_than_a_launch_takes():
    N, D, dev = 2 ** 26 + 3, 128, torch.device("cuda:0")
    cos, sin = pf.rope_tables(N, D, 1e4, dev)
    inv = 1.0 / (1e4 ** (torch.arange(0, D, 2, device=dev, dtype=torch.float32) / D))
    pos = torch.arange(N, device=dev, dtype=torch.float32)
    for part in _edges(N, 2 ** 25):
        ang = pos[part][:, None] * inv
        assert torch.equal(cos[part], torch.cos(ang)) and torch.equal(sin[part], torch.sin(ang)), part
    del cos, sin
    torch.cuda.empty_cache()   # (34 GB)


@pytest.mark.parametrize("B,N,Hq,Hkv", [(1, 1, 1, 1), (1, 33, 4, 2), (2, 31, 7, 1), (1, 64, 32, 8),
                                        (3, 100, 5, 5)])
def test_rope_heads(B, N, Hq, Hkv):
    q, k, v = (_rand((B, N, h, 128), 4 + i) for i, h in enumerate((Hq, Hkv, Hkv)))
    cos, sin = pf.rope_tables(N, 128, 500000.0, torch.device("cpu"))
    got = eb.rope_heads(*(t.cuda() for t in (q, k, v, cos, sin)))
    # the tensor operations keep the same fp32 products: bitwise equal
    for t, o in ((q, got[0]), (k, got[1])):
        assert torch.equal(o.cpu(), pf._rope(t.transpose(1, 2).contiguous(), cos, sin))
    assert torch.equal(got[2].cpu(), v.transpose(1, 2))


@pytest.mark.parametrize("n", [8, 4088, 4096, 4104, 12344])
def test_swiglu(n):
    g, u = _rand((n,), 7, 8.0), _rand((n,), 8)
    g[:8] = torch.tensor([0.0, -0.0, 87.0, -87.0, 300.0, -300.0, float("inf"), float("nan")])
    silu = (g.double() / (1.0 + torch.exp(-g.double()))).to(torch.bfloat16)
    # where the fp32 and the float64 silu straddle a rounding boundary the two
    # roundings are a step (2 half steps) apart, and so is the product, whose
    # own rounding adds a half step: (1 + 2 HALF)(1 + HALF) - 1 < 3.02 HALF
    out = eb.swiglu(g.cuda(), u.cuda())
    _close(out, silu.double() * u.double(), 3.02, floor=1e-36)
    gg = g.cuda()
    assert eb.swiglu(gg, u.cuda(), out=gg).data_ptr() == gg.data_ptr()
    assert torch.equal(gg.nan_to_num(), out.nan_to_num())


def test_swiglu_is_the_tensor_operation():
    """Every bf16 value of g: the same fp32 operations, so bitwise equal."""
    g = torch.arange(1 << 16, dtype=torch.int32).to(torch.int16).view(torch.bfloat16).cuda()
    u = _rand((1 << 16,), 3).cuda()
    ref = torch.nn.functional.silu(g) * u
    out = eb.swiglu(g, u)
    assert torch.equal(out.isnan(), ref.isnan())
    ok = ~ref.isnan()
    assert torch.equal(out[ok].view(torch.int16), ref[ok].view(torch.int16))


def test_layer_takes_tensor_operations_where_kernels_do_not_apply():
    """Autograd still reaches the hidden state, and a layer of fp32 tables in
    another layout gives the same result as the one-pass kernels."""
    dev = torch.device("cuda:0")
    shape = pf.DecoderShape(hidden=512, n_q_heads=4, n_kv_heads=2, intermediate=1024)
    w = pf.make_weights(shape, 1, 5, dev)[0]
    x = _rand((1, 256, 512), 9).cuda()
    cos, sin = pf.rope_tables(256, 128, shape.rope_theta, dev)
    attn = pf.Attention(shape, 1, 256, "dense", pf.SparseConfig(), dev)
    assert pf._one_pass(x, w, shape, cos, sin)
    fast = pf.layer_forward(x, w, shape, attn, cos, sin)
    ct, st = cos.t().contiguous().t(), sin.t().contiguous().t()
    assert not pf._one_pass(x, w, shape, ct, st)
    slow = pf.layer_forward(x, w, shape, attn, ct, st)
    # bf16 roundings a bit apart in the norms travel through the layer
    assert float((fast.float() - slow.float()).norm() / slow.float().norm()) < 4e-3
    # an attention with gradients of its own keeps them
    scale = torch.ones((), device=dev, dtype=torch.bfloat16, requires_grad=True)
    pf.layer_forward(x, w, shape, lambda q, k, v: attn(q, k, v) * scale, cos,
                     sin).float().sum().backward()
    assert scale.grad is not None
    xg = x.clone().requires_grad_()
    pf.layer_forward(xg, w, shape, attn, cos, sin).float().sum().backward()
    assert xg.grad is not None and bool(torch.isfinite(xg.grad.float()).all())


def test_gradients_cross_into_a_frozen_layer():
    """A trained MLP projection below a frozen layer: the frozen layer's norm
    adds a summand with gradients, which the tensor sum records."""
    dev = torch.device("cuda:0")
    shape = pf.DecoderShape(hidden=512, n_q_heads=4, n_kv_heads=2, intermediate=1024)
    layers = pf.make_weights(shape, 2, 5, dev)
    layers[0]["w_down"].requires_grad_()
    attn = pf.Attention(shape, 1, 256, "dense", pf.SparseConfig(), dev)
    last, _ = pf.prefill(_rand((1, 256, 512), 9).cuda(), layers, shape, attn)
    last.float().square().sum().backward()
    grad = layers[0]["w_down"].grad.float()
    assert bool(torch.isfinite(grad).all()) and float(grad.abs().max()) > 0.0
