"""Host-side bounds model: every kernel of the library, compiled as CPU code (tests/hostmodel), is run thread by
thread on seeded geometries with each tensor of the call surrounded by inaccessible address space; any global-memory
address outside its tensor (a wrong sample index, an unclamped halo, a tail that is not masked) stops the run and is
reported with the workgroup and thread that formed it.  No GPU is involved: this is how an off-by-one in the
producers' request arithmetic is found without a memory fault on the device.
"""
import ctypes
import os
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.join(HERE, "hostmodel"))

PASS_NAMES = ("fwd", "bwd_data", "bwd_weight", "bwd", "fwd_ex", "bwd_data_ex", "bwd_ex")


def _load(path):
    lib = ctypes.CDLL(path)
    lib.hostmodel_run.argtypes = [ctypes.c_int] * 11 + [ctypes.c_char_p, ctypes.c_int]
    lib.hostmodel_run.restype = ctypes.c_int
    return lib


@pytest.fixture(scope="module")
def model():
    import build as hostmodel_build

    return _load(hostmodel_build.build())


def _run(lib, ps, geom, dtype, variant=0, placement=0):
    msg = ctypes.create_string_buffer(512)
    rc = lib.hostmodel_run(ps, *geom, dtype, variant, placement, msg, 512)
    return rc, msg.value.decode()


def _check(lib, geom, dtype, passes=range(7), placements=(0, 1), variant=0):
    ran = 0
    for ps in passes:
        for pl in placements:
            rc, msg = _run(lib, ps, geom, dtype, variant, pl)
            if rc == 102:        # CONV1D_EUNSUPPORTED: a forced family that cannot run this geometry
                continue
            assert rc == 0, f"{PASS_NAMES[ps]} {geom} dtype {dtype} placement {pl} variant {variant}: rc {rc} {msg}"
            ran += 1
    return ran


def _curated():
    sys.path.insert(0, HERE)
    import test_gpu_parity as t

    cases = [c[1:] for c in t.SMALL] + [c[1:] for c in t.UNALIGNED]
    cases += [(2, 4, 4, 256, 5, 2, 0), (3, 15, 15, 5000, 51, 8, 200), (2, 15, 15, 4096 + 37, 51, 8, 200),
              (2, 64, 64, 3007, 51, 8, 200), (2, 64, 64, 3007, 5, 1, 2), (2, 256, 256, 1000, 9, 4, 16)]
    return cases


@pytest.mark.parametrize("dtype", [0, 1], ids=["fp32", "bf16"])
def test_curated_geometries_stay_inside_their_tensors(model, dtype):
    """The geometries of the GPU parity suite (every kernel family, odd sizes, halos wider than the row, the shape of
    the one memory fault this library ever had), every entry point, tensors flush against the guard on either side."""
    n = 0
    for geom in _curated():
        if max(geom[1], geom[2]) > 600:      # the streamed-weight shapes: forward and backward-data only (seconds each)
            n += _check(model, geom, dtype, passes=(0, 1), placements=(0, 1))
        else:
            n += _check(model, geom, dtype)
    assert n > 300


def test_element_aligned_tensors(model):
    """Every tensor shifted by one element inside its allocation: the kernels' unaligned paths."""
    for geom in [(2, 15, 15, 3000, 51, 8, 200), (1, 64, 64, 1536, 51, 8, 200), (2, 64, 64, 1200, 9, 2, 8),
                 (2, 40, 24, 2000, 33, 4, 64), (2, 9, 13, 1777, 25, 3, 36), (1, 256, 256, 600, 9, 4, 16)]:
        for dtype in (0, 1):
            _check(model, geom, dtype, placements=(2,))


def test_forced_kernel_families(model):
    for variant in (1, 2, 3):
        for geom in [(2, 4, 4, 256, 5, 2, 0), (2, 15, 13, 2500, 25, 3, 36), (2, 17, 33, 1200, 9, 2, 8), (1, 64, 64, 2500, 33, 16, 256)]:
            for dtype in (0, 1):
                _check(model, geom, dtype, passes=(0, 1, 2), placements=(0,), variant=variant)


def _random_geometry(rng):
    d = int(rng.choice([1, 1, 2, 2, 3, 4, 4, 5, 7, 8, 8, 8, 16, 16]))
    S = int(rng.choice([1, 2, 3, 4, 5, 7, 9, 12, 15, 17, 20, 21, 25, 31, 33, 49, 51, 52, 53, 70]))
    kind = rng.integers(0, 10)
    if kind < 4:
        C, K = int(rng.integers(1, 17)), int(rng.integers(1, 17))
    elif kind < 8:
        C, K = int(rng.integers(17, 97)), int(rng.integers(17, 97))
    else:
        C, K = int(rng.integers(100, 300)), int(rng.integers(100, 300))
    if S > 52:  # the plain-FMA kernels start one workgroup per weight-gradient element: keep that count small
        C, K = min(C, 24), min(K, 24)
    span = (S - 1) * d
    W = int(rng.choice([rng.integers(1, 64), rng.integers(64, 700), rng.integers(700, 2600), 8 * rng.integers(8, 300)]))
    P = int(rng.choice([0, span // 2, rng.integers(0, span + 1), span + int(rng.integers(0, 9)), 8 * (span // 16)]))
    N = int(rng.integers(1, 4))
    if W + 2 * P - span < 1:
        W = span - 2 * P + int(rng.integers(1, 40))
    # the model runs every thread of every workgroup on one core: bound the work of a geometry
    while N * C * K * S * (W + 2 * P - span) > 3e7 and W - (W + 2 * P - span) // 2 >= 1:
        W -= (W + 2 * P - span) // 2
    return (N, C, K, W, S, d, P)


def test_seeded_random_geometries(model):
    rng = np.random.default_rng(20210408)
    ran = 0
    for i in range(800):
        geom = _random_geometry(rng)
        dtype = i & 1
        # forward, backward-data and backward-weight always; the combined and fused entry points on every fourth one
        passes = range(7) if i % 4 == 0 else (0, 1, 2)
        ran += _check(model, geom, dtype, passes=passes, placements=(i // 2 % 2,))
    assert ran >= 2400


def test_seeded_random_few_tap_small_dilation(model):
    """The corner of the register-shift backward-weight kernel and the light prologue paths of the resident-weight
    kernel: bfloat16, 2-17 taps at dilations 1, 2, 4, any padding up to a little beyond the span."""
    rng = np.random.default_rng(20210409)
    ran = 0
    for i in range(150):
        N, C, K, W, S, d, P = _random_geometry(rng)
        d = int(rng.choice([1, 2, 4]))
        S = int(rng.integers(2, 18))
        if (S - 1) * d > 32:
            S = 32 // d + 1
        P = int(rng.integers(0, (S - 1) * d + 9))
        if W + 2 * P - (S - 1) * d < 1:
            W = (S - 1) * d + 5
        ran += _check(model, (N, C, K, W, S, d, P), 1, passes=(0, 1, 2), placements=(i % 2,))
    assert ran >= 450


def _split_tile(lib, ps, geom):
    """(filter blocks, column blocks or taps per wave, planes or units per strip, workgroups, slots of x a thread holds)
    of the FP32 kernels in three bfloat16 parts; None where they do not take the pass.  The slots tell the two
    weight-gradient kernels apart (none: the one of several filter blocks)."""
    t = (ctypes.c_long * 5)()
    return tuple(t) if lib.hostmodel_split_tile(ps, *geom, t) else None


def test_three_part_tiles_of_the_parity_cases(model):
    """The geometries of the GPU parity suite land on the tiles it says, every tile the library has is among them, and no
    access of these launches leaves its tensor."""
    sys.path.insert(0, HERE)
    import test_gpu_split_f32 as t

    seen = set()
    for i, (what, tile, geom) in enumerate(t.TILES):
        ps = t.PASSES.index(what)
        taken = _split_tile(model, ps, geom)
        assert taken[:3] == tile, (what, tile, geom)
        assert ps < 2 or (tile[0] == 1) == (taken[4] > 0), (tile, geom)
        seen.add((ps == 2,) + tile[:2] + taken[4:])
        _check(model, geom, 0, passes=(ps,), placements=(i % 3,))
    for geom in t.FEW_OUTPUTS:
        assert _split_tile(model, 2, geom) is not None, geom
    for geom in t.EDGES + t.QUADS + t.FEW_OUTPUTS[1:]:
        _check(model, geom, 0, passes=(0, 1, 2), placements=(0,))
    rng = np.random.default_rng(3)
    for _ in range(6000):
        geom = tuple(int(v) for v in (rng.integers(1, 65), np.exp(rng.uniform(0, 5.7)), np.exp(rng.uniform(0, 5.7)),
                                      np.exp(rng.uniform(3, 11)), rng.integers(1, 53), rng.integers(1, 17), 0))
        if geom[3] > (geom[4] - 1) * geom[5]:
            for ps in range(3):
                tile = _split_tile(model, ps, geom)
                assert tile is None or (ps == 2,) + tile[:2] + tile[4:] in seen, (ps, geom, tile)
    # layers whose fastest tile among those of several filter blocks has one block
    for geom in [(18, 199, 210, 5253, 50, 1, 24), (47, 295, 202, 17163, 35, 20, 340), (34, 209, 239, 740, 41, 20, 400),
                 (48, 210, 208, 8788, 39, 16, 304), (5, 170, 360, 2597, 6, 24, 60)]:
        tile = _split_tile(model, 2, geom)
        assert tile[0] == 1 and tile[4] > 0 and (True,) + tile[:2] + tile[4:] in seen, (geom, tile)


def _roundings(lib, geom):
    r = (ctypes.c_double * 2)()
    lib.hostmodel_wgrad_roundings(*geom, r)
    return r[0], r[1]


def test_fp32_weight_gradients_round_no_more_often_than_in_all_strips(model):
    """The tiles of the kernel with waves for staging and multiplying may be shorter of sums than those of the kernel of
    several filter blocks (all strips, eight shares of most taps), never with more roundings, but for a handful."""
    for geom, most in [((33, 160, 160, 957, 33, 12, 192), 27), ((2, 133, 133, 28080, 33, 10, 160), 33), ((16, 15, 15, 60000, 51, 8, 200), 32)]:
        assert 0 < _roundings(model, geom)[0] <= most, (geom, _roundings(model, geom))
    rng = np.random.default_rng(17)
    seen = 0
    for _ in range(4000):
        geom = tuple(int(v) for v in (np.exp(rng.uniform(0, 4.1)), np.exp(rng.uniform(0, 5.7)), np.exp(rng.uniform(0, 5.7)),
                                      np.exp(rng.uniform(5, 11)), rng.integers(1, 53), rng.integers(1, 17), 0))
        if geom[3] > (geom[4] - 1) * geom[5]:
            taken, other = _roundings(model, geom)
            assert taken <= max(other, 8) + 1e-6, (geom, taken, other)
            seen += taken > 8
    assert seen > 300


def test_launches_of_fp32_layers_off_the_three_part_kernels(model):
    """What the three-part kernels leave still runs as before: one launch while the weights of all channel blocks and the
    window fit in LDS, else one per channel block, with bias and ReLU in a launch of their own at the end."""
    for geom, fwd, fwd_ex in [((2, 3, 40, 1100, 5, 3, 6), 1, 1), ((1, 8, 24, 3200, 4, 1100, 100), 1, 1), ((1, 92, 20, 2320, 2, 2101, 0), 6, 7)]:
        assert _split_tile(model, 0, geom) is None
        for ps, n in ((0, fwd), (4, fwd_ex)):
            for placement in (0, 1, 2):
                assert _run(model, ps, geom, 0, 0, placement) == (0, "")
                assert model.hostmodel_launches() == n, (geom, ps)
    assert _split_tile(model, 0, (2, 64, 64, 3007, 33, 4, 64)) is not None
    assert _run(model, 0, (2, 64, 64, 3007, 33, 4, 64), 0) == (0, "") and model.hostmodel_launches() == 1


def test_small_launches_of_the_three_part_kernels_take_small_tiles(model):
    """A launch that leaves CUs idle takes narrow tiles (a workgroup alone on its CU takes as long as its chain of steps),
    one that fills the chip several times takes wide ones."""
    for C, K, S, d in [(64, 64, 33, 4), (64, 64, 5, 1), (128, 128, 3, 2), (24, 40, 7, 3)]:
        small = _split_tile(model, 0, (1, C, K, 1000, S, d, (S - 1) * d // 2))
        large = _split_tile(model, 0, (16, C, K, 30000, S, d, (S - 1) * d // 2))
        assert small[:2] == (1, 1) and large[0] * large[1] >= 8, (C, K, S, d, small, large)


def test_long_rows_of_many_taps_are_not_padded_for_one_plane(model):
    """Long rows take steps of one plane and four taps, but where that would multiply more taps than two planes do."""
    for S in range(40, 53):
        for C, K, W in [(64, 64, 60000), (128, 128, 60000), (16, 161, 15001)]:
            planes = _split_tile(model, 0, (1, C, K, W, S, 1, S // 2))[2]
            assert planes == (2 if S % 4 in (1, 2) else 1), (S, C, K, W, planes)


def test_windows_that_just_fit_are_taken(model):
    """Planes are rounded up to start in the same bank where LDS has the room, no layer is refused for it."""
    for ps, geom in [(0, (2, 11, 39, 1392, 2, 1385, 0)), (1, (2, 11, 39, 1392, 2, 1385, 0)), (1, (2, 1, 115, 1380, 2, 1379, 0)), (1, (2, 4, 11, 1383, 2, 1381, 0))]:
        assert _split_tile(model, ps, geom) is not None, geom
        for placement in (0, 1, 2):
            assert _run(model, ps, geom, 0, 0, placement) == (0, "")


def test_rounded_planes_do_not_cost_a_turn_of_the_chip(model):
    """Nor are planes rounded up where a CU then holds a workgroup less and the launch is longer for it: these layers keep
    the tiles whose planes leave LDS for two workgroups only as they are, where a smaller one took their place."""
    for ps, geom, tile in [(0, (19, 172, 172, 1624, 5, 10, 20), (4, 4)), (1, (19, 172, 172, 1624, 5, 10, 20), (4, 4)),
                           (0, (42, 29, 29, 3840, 7, 7, 21), (2, 5)), (0, (8, 64, 144, 39864, 9, 1, 4), (3, 5)),
                           (1, (21, 4, 44, 46819, 21, 13, 130), (1, 8)), (0, (2, 63, 63, 21736, 9, 1, 1), (1, 6))]:
        assert _split_tile(model, ps, geom)[:2] == tile, (ps, geom)
    # planes as they are and rounded up for fewer workgroups per CU
    for geom in [(3, 33, 20, 1624, 5, 10, 20), (43, 28, 28, 600, 17, 2, 0)]:
        _check(model, geom, 0, passes=(0, 1), placements=(0, 1))


def test_weights_of_the_three_part_kernels_stay_within_32_bits(model):
    """Weights are read at 32-bit byte offsets: a layer of 2^30 weights and more is left to the other kernels."""
    for C, K, S, taken in [(8192, 8192, 15, True), (8192, 8192, 16, False), (4096, 8191, 32, True), (4096, 8192, 32, False)]:
        for ps in (0, 1):
            assert (_split_tile(model, ps, (1, C, K, 500, S, 1, 0)) is not None) == taken, (C, K, S, ps)


def test_columns_of_the_three_part_kernels_stay_within_32_bits(model):
    """An output row may be up to 2^31 - 1 columns wide: no tile may end behind the last number a 32-bit column can take
    (its last columns would come out negative and pass for columns of the row)."""
    for short in (0, 1, 63, 130, 200, 300, 700):
        Q = 2 ** 31 - 1 - short
        for C, K, S, d in [(32, 17, 1, 1), (32, 64, 2, 1), (16, 40, 3, 5), (40, 50, 5, 2)]:
            W = 2000 + (1 - (Q + (S - 1) * d) % 2)
            P = (Q - W + (S - 1) * d) // 2
            if W + 2 * P - (S - 1) * d != Q:
                W += 1
                P = (Q - W + (S - 1) * d) // 2
            assert W + 2 * P - (S - 1) * d == Q
            t = _split_tile(model, 0, (1, C, K, W, S, d, P))
            if t:
                width = 64 * t[1]
                assert (Q + width - 1) // width * width <= 2 ** 31, (Q, C, K, S, d, t)


def test_the_model_finds_a_planted_off_by_one():
    """The one GPU memory fault in this library's history: the streamed-weight kernel asked for a stage behind its
    counters and took its sample index one past the batch.  With that repair removed from the model's copy of the
    source, the geometry that faulted must be reported (and the unchanged source must pass it)."""
    import build as hostmodel_build

    repair = """            while (cc < 0) {
                cc += a.ncc;
                if (tc-- == 0) {
                    tc = a.tiles_per_row - 1;
                    --n;
                }
            }
"""
    lib = _load(hostmodel_build.build(mutate={"conv1d_igemm_stream_bf16.hip": lambda t: t.replace(repair, "")},
                                      tag="planted_stream"))
    geom = (4, 232, 1056, 200, 17, 2, 16)
    rc, msg = _run(lib, 0, geom, 1)
    assert rc == 1 and "outside x" in msg, (rc, msg)
    assert _run(_load(hostmodel_build.build()), 0, geom, 1)[0] == 0


def test_backward_of_the_epilogue_stays_inside_its_tensors(model):
    """conv1d_relu_mask and conv1d_epilogue_bwd: rows of every remainder of 8 and around a wave's 512 groups, every remainder
    of the whole, both types, each output with and without the others, a workspace of the bytes the query names."""
    msg = ctypes.create_string_buffer(512)
    model.hostmodel_run_epilogue.argtypes = [ctypes.c_int] * 9 + [ctypes.c_char_p, ctypes.c_int]
    sizes = [(n, k, q) for q in range(1, 18) for n, k in ((1, 1), (1, 3), (2, 5), (3, 8))]
    sizes += [(2, 3, q) for q in list(range(4079, 4106)) + [8185, 8191, 8192, 9001]]
    for i, (N, K, Q) in enumerate(sizes):
        for in16, out16 in ((0, 0), (1, 1), (0, 1)):
            for placement in (0, 1, 2):
                for relu, dy, bias in ((1, 1, 1),) if (i + placement) % 4 else ((1, 1, 1), (0, 1, 1), (1, 1, 0), (0, 0, 1), (1, 0, 1)):
                    rc = model.hostmodel_run_epilogue(N, K, Q, in16, out16, relu, dy, bias, placement, msg, 512)
                    assert rc == 0, (N, K, Q, in16, out16, relu, dy, bias, placement, rc, msg.value.decode())


def test_launches_of_a_backward_with_bfloat16_dx(model):
    """Small-channel layers whose backward-data launch is wide enough add up the weight gradient's partial tiles in it, with
    a bfloat16 dx as with floats: two launches, three with a second stage of its own.  Where passes over channel blocks meet
    in the output, a bfloat16 one is refused before anything is launched."""
    for geom, launches in [((2, 15, 15, 6000, 5, 8, 16), 2), ((2, 15, 15, 60000, 51, 8, 200), 2), ((3, 15, 15, 3000, 51, 8, 200), 3)]:
        for ps in (3, 6):
            assert _run(model, ps, geom, 1) == (0, "") and model.hostmodel_launches() == launches, (geom, ps, model.hostmodel_launches())
    import test_gpu_epilogue_bwd as t

    for C, K, W, S, d in t.MEETING:
        geom = (3, C, K, W, S, d, (S - 1) * d // 2)
        assert _run(model, 6, geom, 1)[0] == 102 and model.hostmodel_launches() == 0, geom


def test_backward_of_the_epilogue_in_pieces():
    """More workgroups than one launch takes are launched in pieces.  In a model that takes three per launch: the mask and
    the masked gradient (every thread's own elements, so the model has their values) are those of the definition."""
    import build as hostmodel_build

    lib = _load(hostmodel_build.build(mutate={"conv1d_epilogue_bwd.hip": lambda t: t.replace("0x7fffffffL / kThreads", "3")},
                                      tag="pieces"))
    vp, sz = ctypes.c_void_p, ctypes.c_size_t
    lib.conv1d_relu_mask.argtypes = [vp, vp, sz, ctypes.c_int, vp]
    lib.conv1d_epilogue_bwd.argtypes = [vp] * 5 + [sz] + [ctypes.c_int] * 5 + [vp]
    rng = np.random.default_rng(4)
    for N, K, Q, mask_launches, launches in [(5, 7, 3, 1, 4), (3, 5, 5001, 4, 4), (2, 13, 8192, 9, 8), (1, 12, 17, 1, 2), (1, 13, 17, 1, 3)]:
        y = np.maximum(rng.standard_normal((N, K, Q)), 0).astype(np.float32)
        gy = rng.standard_normal((N, K, Q)).astype(np.float32)
        dy, db = np.full_like(gy, np.nan), np.zeros(K, np.float32)
        bits, ws = np.full((y.size + 7) // 8, 255, np.uint8), np.empty(1 << 20, np.uint8)
        lib.hostmodel_reset_launches()
        assert lib.conv1d_relu_mask(y.ctypes.data, bits.ctypes.data, y.size, 0, None) == 0
        assert lib.hostmodel_launches() == mask_launches
        assert (np.unpackbits(bits, bitorder="little")[:y.size].reshape(y.shape) == (y > 0)).all()
        lib.hostmodel_reset_launches()
        assert lib.conv1d_epilogue_bwd(gy.ctypes.data, bits.ctypes.data, dy.ctypes.data, db.ctypes.data, ws.ctypes.data, ws.size,
                                       N, K, Q, 0, 0, None) == 0
        assert lib.hostmodel_launches() == launches
        assert (dy == gy * (y > 0)).all(), (N, K, Q)


def test_multiply_high_division_is_exact(model):
    """The kernels divide small indices by launch constants with one multiply-high; the host accepts a divisor only with
    the largest dividend it was checked for.  Every accepted (divisor, bound) pair is compared with the plain quotient
    over its whole range; pairs the host refuses are counted, not trusted."""
    import ctypes as ct

    model.hostmodel_fastdiv_mismatch.argtypes = [ct.c_long, ct.c_long]
    model.hostmodel_fastdiv_mismatch.restype = ct.c_long
    rng = np.random.default_rng(7)
    divisors = list(range(1, 70)) + [95, 117, 118, 188, 255, 256, 257, 626, 641, 1000, 1023, 4097, 65535, 65537] + \
        [int(v) for v in rng.integers(2, 200000, 40)]
    accepted = refused = 0
    for d in divisors:
        for nmax in (d - 1, 5 * d + 3, 70000, 1 << 20):
            r = model.hostmodel_fastdiv_mismatch(d, nmax)
            assert r in (-1, -2), f"fast_div({r}, {d}) differs from {r} // {d} although the bound {nmax} was accepted"
            accepted += r == -1
            refused += r == -2
    assert accepted > 300 and refused < accepted
