"""FP32 layers on the bf16 matrix instructions (three bfloat16 parts per float), at the sizes where their tiles end.

Bound: against the 64-bit oracle every output stays within 2e-6 of sum|products|.  The parts leave 2^-25 of a product
out, partial sums of at most 128 terms are rounded 24 times at 2^-24 of their size and joined to a second sum every 128
terms: 24 * 2^-24 = 1.4e-6 if every rounding fell the same way; measured maxima are a tenth of that.
"""
import pytest

from paper_2104_08002_amd import inputs
from parity_util import check_full, gpu_passes, to_device

pytestmark = pytest.mark.gpu

TOL = 2e-6

CASES = [
    # N  C   K    W     S   d   P
    (1, 17, 1,   16,   1,  1,  0),    # one tap, one tile far from full, a channel block of one channel
    (2, 33, 17,  257,  2,  1,  1),    # one column and one filter past a tile, width not a multiple of 4
    (1, 40, 49,  320,  3,  5,  5),    # four filter blocks, the last of one filter; width = one 320-column tile
    (3, 64, 65,  511,  5,  16, 32),   # a second filter group of one filter
    (1, 24, 40,  1285, 7,  3,  30),   # padding past the halo, width one past 5 x 257
    (2, 16, 80,  384,  4,  64, 0),    # few channels, many filters; a window mostly of halo
    (1, 130, 20, 768,  9,  2,  8),    # channels two past 4 x 32, three tiles of 256 exactly
    (1, 64, 64,  1000, 52, 8,  204),  # most taps
    (1, 13, 9,   66001, 7, 2,  6),    # one channel block, wide enough for the three parts, odd width
    (1, 20, 20,  3200, 52, 20, 510),  # a halo of 1020 columns
]


@pytest.fixture(scope="module")
def binding():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2104_08002_amd import binding as b

    b.load()
    yield b
    b.conv1d_set_variant(0)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_split_layers(binding, case):
    import oracle

    oracle.build()
    N, C, K, W, S, d, P = case
    wl = inputs.scaled(inputs.TINY, name="split_" + "_".join(map(str, case)), N=N, C=C, K=K, W=W, S=S, d=d, P=P,
                       x_dist="normal", w_dist="normal_fan", dy_dist="normal", seed=inputs.BASE_SEED + 7000 + W + S)
    binding.conv1d_set_variant(0)
    for i in range(3):
        assert "mfma" in binding.conv1d_kernel_name(i, *wl.geometry(), 0)
    data = inputs.make_inputs(wl)
    errs = check_full(oracle, wl, data, gpu_passes(wl, to_device(wl, data)))
    print(case, errs, flush=True)
    assert all(e <= TOL for e in errs.values()), errs


# x = w = dy = v: every product leaves the same part out, with the same sign
ADVERSE = [1.0 + 2.0 ** -7 - 2.0 ** -16, 1.2265472412109375, 1.0 + 2.0 ** -8 - 2.0 ** -17, 2.0 - 2.0 ** -9 + 2.0 ** -18]


@pytest.mark.parametrize("v", ADVERSE)
def test_products_left_out(binding, v):
    """32 equal products per output, one step of the matrix instruction.  The parts leave at most 2^-24 of each product
    out, the instruction cuts the sum of the large parts off at 2^-23 of itself and the five smaller sums at 2^-8 of that."""
    import torch

    bound = 2.0 ** -24 + 2.0 ** -23 * (1 + 5 * 2.0 ** -8)
    x = torch.full((1, 32, 400), v, device="cuda")
    w = torch.full((32, 32, 1), v, device="cuda")
    exact = 32 * float(x[0, 0, 0]) ** 2
    for i, name in enumerate(("igemm_split_mfma_fp32", "igemm_split_mfma_fp32", "igemm_wgrad_split_mfma_fp32")):
        assert binding.conv1d_kernel_name(i, 1, 32, 32, 400 if i < 2 else 32, 1, 1, 0, 0) == name
    y = binding.conv1d_fwd(x, w, 1, 0)
    dx = binding.conv1d_bwd_data(x, w, 400, 1, 0)
    dw = binding.conv1d_bwd_weight(x[:, :, :32].contiguous(), x[:, :, :32].contiguous(), 1, 1, 0)
    for what, t in (("fwd", y), ("bwd_data", dx), ("bwd_weight", dw)):
        err = float(((t.double() - exact) / exact).abs().max())
        print(v, what, err, flush=True)
        assert err <= bound, (what, err, bound)


# channels and taps of the forward pass (K = 40), columns of the weight gradient
SHORT = [(1, 1), (2, 1), (1, 3), (4, 5), (31, 1)]


@pytest.mark.parametrize("case", SHORT, ids=lambda c: "x".join(map(str, c)))
def test_short_sums_are_rounded_as_fp32(binding, case):
    """Sums of fewer than 32 products: one rounding to nearest a product, n 2^-24 of sum|products|, as FP32 arithmetic has
    it (a single product is the correctly rounded one)."""
    import torch

    import oracle

    oracle.build()
    C, S = case
    n = C * S
    wl = inputs.scaled(inputs.TINY, name=f"short_{C}_{S}", N=2, C=C, K=40, W=3000, S=S, d=2, P=0, x_dist="normal",
                       w_dist="normal_fan", dy_dist="normal", seed=inputs.BASE_SEED + 7500 + n)
    assert binding.conv1d_kernel_name(0, *wl.geometry(), 0) == "igemm_mfma_fp32"
    data = inputs.make_inputs(wl)
    errs = check_full(oracle, wl, data, gpu_passes(wl, to_device(wl, data), passes=("fwd",)), passes=("fwd",))
    wl = inputs.scaled(wl, name=f"short_wgrad_{n}", N=1, C=40, W=n + 2 * (S - 1))
    assert wl.Q == n and binding.conv1d_kernel_name(2, *wl.geometry(), 0) == "igemm_wgrad_mfma_fp32"
    data = inputs.make_inputs(wl)
    errs.update(check_full(oracle, wl, data, gpu_passes(wl, to_device(wl, data), passes=("bwd_weight",)), passes=("bwd_weight",)))
    print(case, errs, flush=True)
    assert all(e <= n * 2.0 ** -24 * (1 + 2.0 ** -20) for e in errs.values()), errs


def test_largest_and_smallest_floats(binding):
    """One weight of 1 per filter: the output is the input, up to the largest float (no part overflows) and down to
    2^-110; below that the parts lose what lies under 2^-133."""
    import torch

    w = torch.zeros((32, 32, 1), device="cuda")
    w[torch.arange(32), torch.arange(32), 0] = 1.0
    big = torch.tensor([3.4028234663852886e38, 3.3961775292304601e38, 3.39e38, -3.4028234663852886e38, 1.0], device="cuda")
    x = big.repeat(100)[:500].expand(1, 32, 500).contiguous()
    assert binding.conv1d_kernel_name(0, 1, 32, 32, 500, 1, 1, 0, 0) == "igemm_split_mfma_fp32"
    assert torch.equal(binding.conv1d_fwd(x, w, 1, 0), x)
    gen = torch.Generator(device="cuda").manual_seed(7)
    m = 1 + torch.rand((1, 32, 500), generator=gen, device="cuda")
    x = torch.ldexp(m, torch.tensor(-110, device="cuda"))
    assert torch.equal(binding.conv1d_fwd(x, w, 1, 0), x)
    x = torch.ldexp(m, torch.tensor(-120, device="cuda"))
    assert float((binding.conv1d_fwd(x, w, 1, 0).double() - x.double()).abs().max()) < 2.0 ** -133


# layers of more than 16 channels or filters, of up to 16, of one kind on either side
BATCH = [(64, 64, 4000, 5, 2), (100, 100, 1000, 9, 1), (40, 24, 1300, 7, 3), (17, 33, 2000, 15, 4), (15, 15, 5000, 51, 8), (8, 8, 3001, 9, 2),
         (4, 12, 2500, 25, 1), (64, 16, 4000, 5, 1), (8, 40, 3000, 15, 2)]


@pytest.mark.parametrize("case", BATCH, ids=lambda c: "x".join(map(str, c)))
def test_a_sample_does_not_depend_on_its_batch(binding, case):
    """Forward and backward-data of a sample give the same bits alone and among others: tiles follow the size of the
    launch, the order of the sums must not."""
    import torch

    C, K, W, S, d = case
    P = (S - 1) * d // 2
    Q = W + 2 * P - (S - 1) * d
    gen = torch.Generator(device="cuda").manual_seed(11)
    x = torch.randn((56, C, W), generator=gen, device="cuda")
    dy = torch.randn((56, K, Q), generator=gen, device="cuda")
    w = torch.randn((K, C, S), generator=gen, device="cuda")
    y1 = torch.cat([binding.conv1d_fwd(x[i:i + 1].contiguous(), w, d, P) for i in (0, 1)])
    dx1 = torch.cat([binding.conv1d_bwd_data(dy[i:i + 1].contiguous(), w, W, d, P) for i in (0, 1)])
    for n in (2, 3, 5, 8, 13, 16, 21, 33, 40, 48, 56):
        assert torch.equal(binding.conv1d_fwd(x[:n], w, d, P)[:2], y1), n
        assert torch.equal(binding.conv1d_bwd_data(dy[:n], w, W, d, P)[:2], dx1), n
