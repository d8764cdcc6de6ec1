"""FP32 layers on the bf16 matrix instructions (three bfloat16 parts per float), one geometry per tile, at the sizes where
tiles, strips and sums end.

Bound, against the 64-bit oracle and in units of sum|products|: the parts leave at most 2^-24 of a product out; a step adds
32 products, cut off at 2^-23 of its large parts' sum and at 2^-8 of that in the five smaller ones; every step's sum is
added to a running one in FP32, 2^-24 of it; a weight gradient's running sums are then added to each other, up to eight of a
tap, and those of the strips in 32 groups.  Forward and backward-data come to a third of that and less, weight gradients,
whose products have either sign, to a thousandth.

So the whole tensor is held to a second bound, norm of the difference over norm of the result.  The roundings are
independent: T additions to a sum that grows like sqrt(t / T) make sqrt(T / 2) 2^-24 / sqrt(3) of the result, 2.5e-7 at
the 104 steps of the longest sums here, and the cut-off of the steps, always in one direction, up to as much again.  A
tensor without its third parts would be off by 2e-6.
"""
import numpy as np
import pytest

from paper_2104_08002_amd import inputs
from parity_util import REGRESSION_TOL, check_full, gpu_passes, to_device

pytestmark = pytest.mark.gpu

PASSES = ("fwd", "bwd_data", "bwd_weight")

# pass, tile, N  C  K  W  S  d  P.  tile: filter blocks of 16 and column blocks of 64 of a workgroup, planes of 8 channels of
# a step; for the weight gradient filter blocks, taps of a wave, units of the longest strip (the CPU test of the library's
# bounds model checks that these are the tiles taken, and that the kernel of one filter block, whose threads hold one to
# three slots of x, is there with each number of slots).  Widths of the output are odd and end inside a tile, filters end
# inside a block, and groups of filter blocks lack one.
TILES = [
    ("fwd",        (1, 1, 2),  (1, 14, 8, 111, 9, 16, 9)),
    ("bwd_data",   (1, 2, 4),  (11, 4, 18, 1557, 3, 5, 3)),
    ("fwd",        (1, 4, 2),  (19, 10, 4, 1731, 7, 3, 9)),
    ("bwd_data",   (1, 4, 4),  (27, 4, 34, 3591, 1, 3, 0)),
    ("fwd",        (1, 5, 1),  (37, 7, 4, 1689, 5, 2, 4)),
    ("fwd",        (1, 5, 4),  (38, 19, 4, 1851, 3, 16, 0)),
    ("fwd",        (1, 6, 2),  (27, 10, 4, 2967, 7, 8, 0)),
    ("bwd_data",   (1, 8, 2),  (53, 5, 15, 3991, 5, 16, 67)),
    ("bwd_data",   (2, 4, 2),  (57, 65, 11, 157, 3, 16, 16)),
    ("fwd",        (2, 5, 4),  (53, 19, 65, 283, 2, 8, 4)),
    ("fwd",        (2, 6, 1),  (32, 8, 129, 338, 4, 5, 0)),
    ("fwd",        (2, 8, 1),  (33, 7, 70, 2393, 5, 3, 6)),
    ("fwd",        (3, 4, 4),  (60, 32, 66, 413, 1, 1, 0)),
    ("bwd_data",   (3, 5, 2),  (37, 70, 16, 1595, 2, 5, 2)),
    ("bwd_data",   (3, 6, 1),  (34, 72, 8, 2343, 4, 3, 4)),
    ("fwd",        (4, 4, 2),  (47, 21, 101, 771, 2, 2, 5)),
    ("fwd",        (4, 5, 1),  (48, 8, 108, 1292, 4, 1, 6)),
    ("fwd",        (1, 6, 1),  (1, 16, 161, 15003, 43, 1, 21)),  # rows so long that one plane is taken for that
    ("bwd_weight", (1, 3, 1),  (1, 4, 5, 109, 1, 3, 0)),
    ("bwd_weight", (1, 3, 3),  (43, 4, 4, 3497, 1, 3, 1)),
    ("bwd_weight", (1, 5, 4),  (51, 5, 6, 3856, 4, 3, 0)),
    ("bwd_weight", (1, 7, 2),  (45, 5, 4, 1467, 7, 2, 6)),
    ("bwd_weight", (1, 5, 3),  (58, 5, 4, 2691, 9, 2, 0)),
    ("bwd_weight", (1, 9, 3),  (46, 4, 5, 3677, 33, 5, 0)),
    ("bwd_weight", (1, 13, 3), (51, 5, 4, 3302, 26, 1, 0)),
    ("bwd_weight", (1, 7, 8),  (40, 4, 4, 3501, 51, 5, 0)),
    ("bwd_weight", (1, 5, 5),  (47, 6, 4, 3117, 9, 5, 0)),
    ("bwd_weight", (1, 7, 4),  (55, 6, 6, 3521, 13, 16, 96)),
    ("bwd_weight", (1, 3, 4),  (32, 4, 135, 535, 1, 5, 3)),
    ("bwd_weight", (1, 3, 2),  (44, 4, 35, 475, 5, 16, 5)),
    ("bwd_weight", (1, 3, 2),  (51, 5, 35, 269, 9, 8, 32)),
    ("bwd_weight", (1, 7, 5),  (54, 4, 69, 487, 13, 8, 0)),
    ("bwd_weight", (1, 3, 4),  (39, 4, 66, 821, 9, 3, 27)),
    ("bwd_weight", (1, 7, 2),  (48, 5, 35, 189, 13, 16, 195)),
    ("bwd_weight", (1, 7, 3),  (46, 5, 106, 193, 13, 3, 18)),
    ("bwd_weight", (1, 3, 2),  (1, 28, 4, 511, 1, 10, 0)),
    ("bwd_weight", (1, 3, 2),  (46, 4, 5, 1503, 41, 17, 0)),
    ("bwd_weight", (1, 5, 2),  (59, 27, 34, 300, 28, 11, 0)),
    ("bwd_weight", (1, 5, 2),  (28, 33, 34, 787, 50, 16, 0)),
    ("bwd_weight", (1, 7, 2),  (29, 39, 34, 403, 41, 10, 0)),
    ("bwd_weight", (1, 9, 2),  (49, 5, 40, 465, 43, 9, 0)),
    ("bwd_weight", (1, 9, 2),  (24, 4, 6, 4699, 16, 16, 205)),
    ("bwd_weight", (1, 13, 2), (45, 6, 4, 2291, 25, 11, 130)),
    ("bwd_weight", (1, 13, 2), (55, 36, 23, 63, 49, 14, 306)),
    ("bwd_weight", (2, 2, 3),  (5, 202, 163, 21, 6, 3, 0)),
    ("bwd_weight", (2, 3, 6),  (11, 132, 269, 318, 22, 15, 0)),
    ("bwd_weight", (2, 5, 14), (27, 170, 233, 353, 33, 11, 0)),
    ("bwd_weight", (2, 7, 1),  (2, 274, 203, 140, 44, 2, 0)),
    ("bwd_weight", (2, 9, 6),  (4, 132, 282, 399, 35, 7, 0)),
    ("bwd_weight", (4, 2, 1),  (2, 204, 184, 45, 27, 1, 0)),
    ("bwd_weight", (4, 3, 1),  (2, 133, 240, 222, 52, 4, 0)),
]

# small layers at the edges of sizes
EDGES = [
    # N  C   K    W     S   d   P
    (1, 17, 1,   16,   1,  1,  0),    # a channel block of one channel; 17 products per output, 16 per weight, one per input
    (2, 33, 17,  257,  2,  1,  1),    # one column and one filter past a block, width not a multiple of 4
    (1, 40, 49,  320,  3,  5,  5),    # four filter blocks, the last of one filter
    (3, 64, 65,  511,  5,  16, 32),   # a fifth filter block of one filter
    (1, 24, 40,  1285, 7,  3,  30),   # padding past the halo
    (2, 16, 80,  384,  4,  64, 0),    # few channels, many filters; a window mostly of halo
    (1, 130, 20, 768,  9,  2,  8),    # channels two past 4 x 32
    (1, 64, 64,  1000, 52, 8,  204),  # most taps
    (1, 13, 9,   66001, 7, 2,  6),    # one channel block, odd width
    (1, 20, 20,  3200, 52, 20, 510),  # a halo of 1020 columns
]


def _bound(ps, wl, tile=None):
    """Worst case of the sums described above, in units of sum|products|."""
    if ps == 2:
        units = tile[2] if tile else 1
        steps = 16 * units + 8 + 8 + 32  # a unit is at most 512 positions; shares of a tap; strips of a group; groups
    else:
        R = wl.C if ps == 0 else wl.K
        steps = max(-(-R // (8 * pl)) * -(-wl.S * pl // 4) for pl in (1, 2, 4))
    return 2.0 ** -24 + 2.0 ** -23 * (1 + 5 * 2.0 ** -8) + steps * 2.0 ** -24


NORM_BOUND = 5e-7


def _errors(oracle, wl, data, got):
    """{pass: (largest error over sum|products|, norm of the difference over norm of the result)}"""
    errs = check_full(oracle, wl, data, got, passes=tuple(got))
    x, w, dy = (data[k].astype(np.float64) for k in ("x", "w", "dy"))
    ref = {"fwd": lambda: oracle.fwd(x, w, wl.d, wl.P), "bwd_data": lambda: oracle.bwd_data(dy, w, wl.W, wl.d, wl.P),
           "bwd_weight": lambda: oracle.bwd_weight(x, dy, wl.S, wl.d, wl.P)}
    out = {}
    for k in got:
        r = ref[k]()
        out[k] = (errs[k], float(np.linalg.norm(got[k].astype(np.float64) - r) / np.linalg.norm(r)))
    return out


def _workload(geom):
    N, C, K, W, S, d, P = geom
    return inputs.scaled(inputs.TINY, name="split_" + "_".join(map(str, geom)), N=N, C=C, K=K, W=W, S=S, d=d, P=P,
                         x_dist="normal", w_dist="normal_fan", dy_dist="normal", seed=inputs.BASE_SEED + 7000 + W + S)


@pytest.fixture(scope="module")
def binding():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2104_08002_amd import binding as b

    b.load()
    yield b
    b.conv1d_set_variant(0)


@pytest.mark.parametrize("case", TILES, ids=lambda c: "_".join([c[0]] + [str(v) for v in c[1]]))
def test_tiles(binding, oracle, case):
    what, tile, geom = case
    ps, wl = PASSES.index(what), _workload(geom)
    assert "split_mfma_fp32" in binding.conv1d_kernel_name(ps, *wl.geometry(), 0)
    data = inputs.make_inputs(wl)
    most, norm = _errors(oracle, wl, data, gpu_passes(wl, to_device(wl, data), passes=(what,)))[what]
    print(case, most, _bound(ps, wl, tile), norm, flush=True)
    assert most <= _bound(ps, wl, tile) and norm <= NORM_BOUND, (most, _bound(ps, wl, tile), norm)


@pytest.mark.parametrize("case", EDGES, ids=lambda c: "x".join(map(str, c)))
def test_edges(binding, oracle, case):
    wl = _workload(case)
    data = inputs.make_inputs(wl)
    errs = _errors(oracle, wl, data, gpu_passes(wl, to_device(wl, data)))
    print(case, errs, flush=True)
    for i, what in enumerate(PASSES):
        split = (wl.C * wl.S, wl.K * wl.S, wl.N * wl.Q)[i] >= 16
        assert ("split" in binding.conv1d_kernel_name(i, *wl.geometry(), 0)) == split, (what, split)
        bound = _bound(i, wl) if split else 16 * 2.0 ** -24
        assert errs[what][0] <= bound and errs[what][1] <= NORM_BOUND, (what, errs, bound)


# weight gradients whose dy is read by four elements: samples of four to seven outputs, rows that end one, two and three
# elements into a group, in the last of which the loads begin early, units of every number of slots per thread
QUADS = [(16, 5, 1, 4, 1, 1, 0), (8, 3, 1, 5, 1, 1, 0), (6, 2, 2, 3, 1, 1, 0), (16, 2, 7, 1, 1, 1, 0), (5, 20, 3, 7, 3, 1, 1), (3, 17, 33, 257, 2, 3, 2),
         (2, 20, 18, 225, 5, 1, 2), (1, 33, 17, 1022, 9, 16, 64), (2, 16, 40, 451, 3, 2, 2), (1, 4, 5, 2603, 51, 10, 250)]


@pytest.mark.parametrize("case", QUADS, ids=lambda c: "x".join(map(str, c)))
def test_weight_gradients_read_by_four(binding, oracle, case):
    import torch

    wl = _workload(case)
    assert "split" in binding.conv1d_kernel_name(2, *wl.geometry(), 0)
    data = inputs.make_inputs(wl)
    dev = to_device(wl, data)
    got = binding.conv1d_bwd_weight(dev["x"], dev["dy"], wl.S, wl.d, wl.P)
    # the last sample's memory ends where the tensor does, and the tensor begins behind any float
    buf = torch.full((dev["dy"].numel() + 1,), float("nan"), device="cuda")
    buf[1:] = dev["dy"].flatten()
    assert torch.equal(binding.conv1d_bwd_weight(dev["x"], buf[1:].view_as(dev["dy"]), wl.S, wl.d, wl.P), got)
    err, norm = _errors(oracle, wl, data, {"bwd_weight": got.cpu().numpy()})["bwd_weight"]
    assert err <= _bound(2, wl, (0, 0, 8)) and norm <= NORM_BOUND, (err, norm)


# weight gradients of samples of one to three outputs
FEW_OUTPUTS = [(56, 256, 1, 303, 51, 6, 0), (16, 4, 1, 9, 8, 1, 0), (16, 17, 2, 5, 5, 1, 0), (16, 17, 3, 5, 5, 1, 0), (64, 64, 1, 4, 3, 1, 0), (1024, 32, 1, 17, 17, 1, 1)]


@pytest.mark.parametrize("case", FEW_OUTPUTS, ids=lambda c: "x".join(map(str, c)))
def test_weight_gradients_of_few_outputs(binding, oracle, case):
    wl = _workload(case)
    assert wl.K * wl.Q < 4 and "split" in binding.conv1d_kernel_name(2, *wl.geometry(), 0)
    data = inputs.make_inputs(wl)
    err, norm = _errors(oracle, wl, data, gpu_passes(wl, to_device(wl, data), passes=("bwd_weight",)))["bwd_weight"]
    assert err <= _bound(2, wl, (0, 0, 8)) and norm <= NORM_BOUND, (err, norm)


# layers whose fastest tile has half the running sums, and the roundings of their sums in all strips: 2.3e-7 and 2.3e-7 so
MANY_ROUNDINGS = [((33, 160, 160, 957, 33, 12, 192), 28.6), ((2, 133, 133, 28080, 33, 10, 160), 34.6)]


@pytest.mark.parametrize("case", MANY_ROUNDINGS, ids=lambda c: "x".join(map(str, c[0])))
def test_weight_gradients_keep_their_roundings(binding, case):
    """n independent roundings of up to 2^-24 / sqrt(3) of the sum (root mean square), which is the norm of the error."""
    import torch

    (N, C, K, W, S, d, P), n = case
    gen = torch.Generator(device="cuda").manual_seed(23)
    Q = W + 2 * P - (S - 1) * d
    x = torch.rand((N, C, W), generator=gen, device="cuda") * 2 - 1
    dy = torch.rand((N, K, Q), generator=gen, device="cuda") * 2 - 1
    dw = binding.conv1d_bwd_weight(x, dy, S, d, P).double()
    xp, gt = torch.nn.functional.pad(x.double(), (P, P)), dy.double().transpose(1, 2).contiguous()
    ref = torch.stack([torch.matmul(xp[:, :, t * d:t * d + Q].contiguous(), gt).sum(0).t() for t in range(S)], 2)
    norm = float((dw - ref).norm() / ref.norm())
    print(case, norm, flush=True)
    assert norm <= 2.0 ** -24 * (n / 3) ** 0.5, norm


# layers left on the FP32 instruction, by their sums or their windows, and the kernel of each pass
LEFT = [
    # N  C   K   W     S  d     P      forward, backward-data, backward-weight
    ((2, 3,  40, 1100, 5, 3,    6),    ("igemm_mfma_fp32", "smallc_split_mfma_fp32", "igemm_wgrad_split_mfma_fp32")),
    ((1, 40, 3,  901,  5, 2,    4),    ("smallc_split_mfma_fp32", "igemm_mfma_fp32", "igemm_wgrad_split_mfma_fp32")),
    ((1, 8,  24, 3200, 4, 1100, 100),  ("igemm_mfma_fp32", "generic_fma_fp32", "generic_wgrad_fp32")),
    ((1, 92, 20, 2320, 2, 2101, 0),    ("igemm_mfma_fp32", "igemm_mfma_fp32", "generic_wgrad_fp32")),
    ((1, 50, 70, 12,   3, 1,    0),    ("igemm_split_mfma_fp32", "igemm_split_mfma_fp32", "igemm_wgrad_mfma_fp32")),
]


@pytest.mark.parametrize("case", LEFT, ids=lambda c: "x".join(map(str, c[0])))
def test_layers_left_on_the_fp32_instruction(binding, oracle, case):
    wl = _workload(case[0])
    assert tuple(binding.conv1d_kernel_name(i, *wl.geometry(), 0) for i in range(3)) == case[1]
    data = inputs.make_inputs(wl)
    errs = check_full(oracle, wl, data, gpu_passes(wl, to_device(wl, data)))
    print(case, errs, flush=True)
    assert all(e <= REGRESSION_TOL["fp32"] for e in errs.values()), errs


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
SHORT = [(1, 1), (2, 1), (1, 3), (3, 5), (15, 1)]


@pytest.mark.parametrize("case", SHORT, ids=lambda c: "x".join(map(str, c)))
def test_short_sums_are_rounded_as_fp32(binding, oracle, case):
    """Sums of fewer than 16 products: one rounding to nearest a product, n 2^-24 of sum|products|, as FP32 arithmetic has
    it (a single product is the correctly rounded one)."""
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


# columns cut into strips of one unit each, of two, of one or two, and into a single strip
CUT_OFF = [(1, 15, 15, 66000, 7, 2), (16, 15, 15, 8192, 7, 2), (3, 5, 4, 33000, 3, 1), (2, 40, 24, 3000, 5, 1), (1, 15, 15, 4000, 51, 8)]


@pytest.mark.parametrize("case", CUT_OFF, ids=lambda c: "x".join(map(str, c)))
def test_cut_off_of_weight_gradients_cancels(binding, case):
    """The matrix instruction cuts off towards minus infinity: an offset in every partial sum, with the same sign in all of
    them unless units alternate.  A coverage track (80 % zeros) has few large products, which shows it most: up to 3.6e-7 of
    the gradient against roundings of 1.4e-7; the mean of the error over the gradient holds the offset alone."""
    import torch

    N, C, K, W, S, d = case
    gen = torch.Generator(device="cuda").manual_seed(5)
    Q = W - (S - 1) * d
    x = torch.empty((N, C, W), device="cuda").exponential_(1.0, generator=gen) * (torch.rand((N, C, W), generator=gen, device="cuda") < 0.2)
    dy = torch.randn((N, K, Q), generator=gen, device="cuda")
    assert "split" in binding.conv1d_kernel_name(2, N, C, K, W, S, d, 0, 0)
    dw = binding.conv1d_bwd_weight(x, dy, S, d, 0).double()
    gt = dy.double().transpose(1, 2).contiguous()
    ref = torch.stack([torch.matmul(x[:, :, t * d:t * d + Q].double().contiguous(), gt).sum(0).t() for t in range(S)], 2)
    norm = float((dw - ref).norm() / ref.norm())
    mean = float((dw - ref).mean().abs() * ref.numel() ** 0.5 / ref.norm())
    print(case, norm, mean, flush=True)
    assert norm <= 2.2e-7 and mean <= 1e-7, (norm, mean)


# layers of 6 and 10, of 10 and 26 steps
EVEN_STEPS = [(24, 40, 7, 3), (64, 64, 5, 1), (40, 24, 7, 3), (15, 15, 51, 8)]


@pytest.mark.parametrize("case", EVEN_STEPS, ids=lambda c: "x".join(map(str, c)))
def test_cut_off_of_forward_and_backward_data_cancels(binding, case):
    """Every step's sum is cut off towards minus infinity; steps alternate in sign, so the mean error of a million outputs
    is that of a million independent roundings, 1e-7 / 1000 of their size (-1.6e-8 with all steps added)."""
    import torch

    C, K, S, d = case
    N, W, P = 6, 5000, (S - 1) * d // 2
    gen = torch.Generator(device="cuda").manual_seed(13)
    x = torch.randn((N, C, W), generator=gen, device="cuda")
    dy = torch.randn((N, K, W + 2 * P - (S - 1) * d), generator=gen, device="cuda")
    w = torch.randn((K, C, S), generator=gen, device="cuda")

    def exact(t, wt, pad):
        tp = torch.nn.functional.pad(t.double(), (pad, pad))
        n = tp.shape[2] - (S - 1) * d
        return sum(torch.matmul(wt[:, :, s].double().contiguous(), tp[:, :, s * d:s * d + n].contiguous()) for s in range(S))

    pairs = {"fwd": (binding.conv1d_fwd(x, w, d, P), exact(x, w, P)),
             "bwd_data": (binding.conv1d_bwd_data(dy, w, W, d, P), exact(dy, w.transpose(0, 1).flip(2), (S - 1) * d - P))}
    for what, (got, ref) in pairs.items():
        mean = float((got.double() - ref).mean() / ref.square().mean().sqrt())
        print(case, what, mean, flush=True)
        assert abs(mean) <= 2e-9, (what, mean)


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


# layers of more than 16 channels or filters, of up to 16, of one kind on either side, on the FP32 instruction
BATCH = [(64, 64, 4000, 5, 2), (100, 100, 1000, 9, 1), (40, 24, 1300, 7, 3), (17, 33, 2000, 15, 4), (15, 15, 5000, 51, 8), (8, 8, 3001, 9, 2),
         (4, 12, 2500, 25, 1), (64, 16, 4000, 5, 1), (8, 40, 3000, 15, 2), (16, 161, 15001, 43, 2), (3, 40, 3000, 5, 3), (3, 2, 5000, 5, 8)]


@pytest.mark.parametrize("case", BATCH, ids=lambda c: "x".join(map(str, c)))
def test_a_sample_does_not_depend_on_its_batch(binding, case):
    """Forward and backward-data of a sample give the same bits alone and among others: tiles follow the size of the
    launch, the order of the sums must not."""
    import torch

    C, K, W, S, d = case  # (the last two: forward sums of 15 products)
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
