"""Backward of the fused bias + ReLU (conv1d_relu_mask, conv1d_epilogue_bwd, conv1d_bwd_ex) against torch in float64.

The masked gradient is one product with 0 or 1 and one rounding: compared bit for bit.  The bias gradient is summed in
FP32 per wave (8 groups left to right, 3 levels within a group, 6 across the lanes) and in 64 bits after that: at most
18 roundings, 18 * 2^-24 of the sum of magnitudes.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def binding():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2104_08002_amd import binding as b

    b.load()
    return b


def _same(a, b):
    import torch

    return bool(((a == b) | (a.isnan() & b.isnan())).all()) and torch.equal(torch.signbit(a[~a.isnan()]), torch.signbit(b[~b.isnan()]))


# rows within one group of 8, shared groups at their ends, the last group of a wave's chunk (512 groups), many chunks
@pytest.mark.parametrize("N,K,Q", [(1, 1, 1), (2, 3, 5), (3, 5, 8), (2, 4, 31), (2, 15, 4089), (1, 3, 4096), (2, 2, 4097), (3, 7, 9001), (56, 16, 2000)])
@pytest.mark.parametrize("types", ["f32", "bf16", "f32_to_bf16"])
@pytest.mark.parametrize("relu", [True, False])
def test_epilogue_backward(binding, N, K, Q, types, relu):
    import torch

    gen = torch.Generator(device="cuda").manual_seed(Q)
    tin = torch.bfloat16 if types == "bf16" else torch.float32
    tout = torch.float32 if types == "f32" else torch.bfloat16
    y = torch.randn((N, K, Q), generator=gen, device="cuda").clamp(min=0).to(tin)
    for shift in (0, 1):  # an aligned gradient, and one that begins behind an element
        gy = torch.randn(N * K * Q + shift, generator=gen, device="cuda").to(tin)[shift:].view(N, K, Q)
        pos = binding.conv1d_relu_mask(y) if relu else None
        dy, db = binding.conv1d_epilogue_bwd(gy, pos, tout, True)
        m = gy * (y > 0) if relu else gy
        assert _same(dy, m.to(tout)), (shift, "dy")
        ref, mag = m.double().sum((0, 2)), m.double().abs().sum((0, 2))
        assert ((db.double() - ref).abs() <= 18 * 2.0 ** -24 * mag).all(), (shift, "db")
        assert binding.conv1d_epilogue_bwd(gy, pos, tout, False)[1] is None


def test_more_rows_than_a_launch_has_waves(binding):
    """33.6 million rows of a layer with bias and ReLU: one wave each, more than one launch takes."""
    import torch

    from paper_2104_08002_amd import autograd

    gen = torch.Generator(device="cuda").manual_seed(3)
    N, K = 2100000, 16
    x = torch.randn((N, 1, 2), generator=gen, device="cuda").requires_grad_(True)
    w = torch.randn((K, 1, 1), generator=gen, device="cuda").requires_grad_(True)
    b = torch.randn(K, generator=gen, device="cuda").requires_grad_(True)
    y = autograd.conv1d(x, w, b, 1, 0, relu=True)
    gy = torch.randn(y.shape, generator=gen, device="cuda")
    dx, dw, db = torch.autograd.grad(y, (x, w, b), gy)
    g = gy * (y > 0)
    pos = binding.conv1d_relu_mask(y.detach())
    assert torch.equal(binding.conv1d_epilogue_bwd(gy, pos, torch.float32, False)[0], g)
    rx, rw = binding.conv1d_bwd(x.detach(), g, w.detach(), 1, 0)
    assert torch.equal(dx, rx) and torch.equal(dw, rw)
    # two elements of a row are added before the sum goes on in 64 bits
    ref, mag = g.double().sum((0, 2)), g.double().abs().sum((0, 2))
    assert ((db.double() - ref).abs() <= 2 * 2.0 ** -24 * mag).all()


def test_nan_and_infinity_of_a_gradient_stay(binding):
    import torch

    nan, inf = float("nan"), float("inf")
    y = torch.tensor([1.0, 0.0, 1.0, 0.0, nan, -0.0, inf, 2.0, 3.0], device="cuda").view(1, 1, 9)
    gy = torch.tensor([nan, nan, inf, inf, 1.0, -1.0, 1.0, -inf, 0.5], device="cuda").view(1, 1, 9)
    dy, db = binding.conv1d_epilogue_bwd(gy, binding.conv1d_relu_mask(y), torch.float32, True)
    assert _same(dy, gy * (y > 0)) and db.isnan().all()


# layers whose passes over channel blocks meet in a float dx (the CPU test of the library's bounds model checks that they do,
# and that the first two below add up the weight gradient within the backward-data launch)
MEETING = [(40, 24, 901, 7, 3), (100, 100, 301, 3, 3)]


@pytest.mark.parametrize("C,K,W,S,d", [(15, 15, 6000, 5, 8), (15, 15, 60000, 51, 8), (15, 15, 3000, 51, 8), (16, 16, 1000, 51, 4), (64, 64, 2000, 5, 1),
                                       (12, 9, 777, 25, 3)] + MEETING)
def test_bf16_gradient_of_the_input_is_the_rounded_one(binding, C, K, W, S, d):
    import torch

    gen = torch.Generator(device="cuda").manual_seed(W)
    P = (S - 1) * d // 2
    x, dy = (torch.randn((3, c, W), generator=gen, device="cuda").bfloat16() for c in (C, K))
    w = torch.randn((K, C, S), generator=gen, device="cuda").bfloat16()
    dx, dw = binding.conv1d_bwd(x, dy, w, d, P)
    dx16, dw16 = binding.conv1d_bwd_ex(x, dy, w, d, P, out_bf16=True)
    assert torch.equal(dx16, dx.bfloat16()) and torch.equal(dw16, dw)
    if (C, K, W, S, d) in MEETING:
        with pytest.raises(binding.Conv1dError) as e:
            binding._bwd(x, dy, w, d, P, None, None, None, None, True)
        assert e.value.status == binding.STATUS_EUNSUPPORTED


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_layer_gradients(binding, dtype):
    """What follows the layer may change its output in place, may send an expanded gradient, and may want a graph of it."""
    import torch

    from paper_2104_08002_amd import autograd

    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn((2, 6, 500), generator=gen, device="cuda").to(t).requires_grad_(True)
    w = torch.randn((5, 6, 7), generator=gen, device="cuda").to(t).requires_grad_(True)
    b = torch.randn(5, generator=gen, device="cuda").requires_grad_(True)
    y = autograd.conv1d(x, w, b, 2, 6, relu=True, bf16_out=dtype == "bf16")
    positive = (y > 0).double()
    y.add_(1.0)
    dx, dw, db = torch.autograd.grad(y.sum(), (x, w, b))
    g = positive.to(t)
    rx, rw = binding.conv1d_bwd(x.detach(), g, w.detach(), 2, 6)
    assert torch.equal(dx, rx.to(t)) and torch.equal(dw, rw.to(t)) and torch.equal(db, positive.sum((0, 2)).float())
    y = autograd.conv1d(x, w, b, 2, 6, relu=True)
    gy = torch.randn(y.shape, generator=gen, device="cuda").requires_grad_(True)
    db, = torch.autograd.grad(y, b, gy, create_graph=True)
    back, = torch.autograd.grad(db.sum(), gy, retain_graph=True)
    assert torch.equal(back, positive.float())
    with torch.no_grad():
        assert torch.equal(autograd.conv1d(x, w, b, 2, 6, relu=True), y)
    # and forward mode over the backward: the tangent of the bias gradient is that of gy, masked and summed
    tangent = torch.randn(y.shape, generator=gen, device="cuda")
    with torch.autograd.forward_ad.dual_level():
        dual = torch.autograd.forward_ad.make_dual(gy.detach(), tangent)
        db, = torch.autograd.grad(y, b, dual)
        db, dt = torch.autograd.forward_ad.unpack_dual(db)
    assert dt is not None
    for got, of in ((db, gy.detach()), (dt, tangent)):
        ref = (of * positive).double()
        assert ((got.double() - ref.sum((0, 2))).abs() <= 1000 * 2.0 ** -24 * ref.abs().sum((0, 2))).all()  # (torch adds 1000 floats)
