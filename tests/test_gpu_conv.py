"""GPU parity: the three convolutions through the C ABI against the fp64 oracle."""
import numpy as np
import pytest

import oracle
from paper_1901_09290_amd import workloads as wl
from paper_1901_09290_amd.workloads import ConvSpec

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _spec(N, H, W, C, K, R, st, pad):
    return ConvSpec("t", N, H, W, C, K, R, R, st, pad, None, None)


def _check_full(spec, seed, xp=None, yp=None, wp=None, pad_zero=False):
    from gpu_util import CONV_TOL, rel_err, run_conv_all, strict_rel_err
    rng = np.random.Generator(np.random.PCG64(seed))
    t = wl.conv_tensors(spec, rng)
    y, dx, dw = run_conv_all(spec, t["x"], t["w"], t["dy"], xp, yp, wp, pad_zero)
    s = oracle.shape_of(spec)
    refs = (oracle.conv_fwd(s, t["x"], t["w"]), oracle.conv_bwd_data(s, t["dy"], t["w"]),
            oracle.conv_bwd_weight(s, t["x"], t["dy"]))
    errs = tuple(rel_err(g, r) for g, r in zip((y, dx, dw), refs))
    assert max(errs) <= CONV_TOL, (spec, errs)
    # the plain element-wise relative error away from cancellation zeros obeys the same bound (bf16 rounding of an
    # output is 2^-9 relative; fp32 accumulation adds far less on elements of this size)
    strict = tuple(strict_rel_err(g, r) for g, r in zip((y, dx, dw), refs))
    assert max(strict) <= CONV_TOL, (spec, strict)
    return errs + strict


def test_cfg1_single_layer():
    from gpu_util import CONV_TOL, rel_err, run_conv_all
    c = wl.cfg1(0)
    spec = c["spec"]
    y, dx, dw = run_conv_all(spec, c["x"], c["w"], c["dy"])
    s = oracle.shape_of(spec)
    ry, rdx, rdw = (oracle.conv_fwd(s, c["x"], c["w"]), oracle.conv_bwd_data(s, c["dy"], c["w"]),
                    oracle.conv_bwd_weight(s, c["x"], c["dy"]))
    assert rel_err(y, ry) <= CONV_TOL and rel_err(dx, rdx) <= CONV_TOL and rel_err(dw, rdw) <= CONV_TOL
    # zeroed groups give exact zeros: outputs of zero filters, input gradients of zero input channels
    assert np.all(y[..., c["zero_out"]] == 0.0)
    assert np.all(dx[..., c["zero_in"]] == 0.0)


SMALL = [
    # N  H   W   C    K   R st pad    several tiles + ragged tails in every GEMM dimension
    (2, 12, 12, 64, 64, 3, 1, 1),
    (3, 9, 11, 24, 40, 3, 1, 1),
    (2, 14, 14, 128, 96, 1, 1, 0),
    (2, 15, 15, 40, 136, 3, 2, 1),
    (2, 16, 16, 64, 128, 1, 2, 0),
    (1, 37, 37, 8, 16, 7, 2, 3),
    (5, 7, 7, 264, 72, 3, 1, 1),
    (1, 20, 20, 16, 200, 1, 1, 0),
    (1, 1, 1, 8, 8, 1, 1, 0),          # a single pixel
    (2, 5, 5, 8, 8, 5, 1, 0),          # filter as large as the image
    (1, 8, 8, 8, 8, 3, 3, 1),          # stride 3: parity classes with uneven tap counts
]


@pytest.mark.parametrize("case", SMALL)
def test_small_layers_full_tensor(case):
    _check_full(_spec(*case), seed=100 + sum(case))


RAGGED = [
    # logical C, K not multiples of 8; pitches padded to 8 (vector path with masked tails)
    ((2, 10, 10, 37, 51, 3, 1, 1), True),
    ((2, 12, 12, 203, 77, 1, 1, 0), True),
    ((1, 9, 9, 19, 131, 3, 2, 1), True),
    ((2, 18, 18, 3, 16, 7, 2, 3), True),   # image-like 3-channel input, pitch 8: filter rows folded into one run
    ((2, 30, 30, 3, 28, 7, 2, 3), True),
    ((3, 13, 13, 5, 24, 3, 1, 1), True),
    ((2, 11, 11, 12, 40, 5, 1, 2), True),  # pitch 16 with 12 real channels: a masked chunk inside every tap
    ((2, 9, 9, 32, 48, 2, 1, 0), True),    # folded run of exactly 64 elements
    ((2, 20, 20, 45, 38, 3, 1, 1), True),  # folded runs of 48 with 45 real channels: a tail in every 64-block
    ((2, 20, 20, 63, 40, 3, 1, 1), True),  # one 64-block per tap, tail in its last chunk
    ((2, 14, 14, 209, 45, 1, 1, 0), True),  # tail only in the last of four blocks
    # same shapes stored dense: pitches are odd, element-wise path
    ((2, 10, 10, 37, 51, 3, 1, 1), False),
    ((1, 9, 9, 19, 131, 3, 2, 1), False),
    ((2, 18, 18, 3, 16, 7, 2, 3), False),  # image-like 3-channel input
]


@pytest.mark.parametrize("case,padded", RAGGED)
def test_ragged_channel_counts(case, padded):
    from gpu_util import pitch8
    spec = _spec(*case)
    if padded:
        _check_full(spec, 200 + sum(case), pitch8(spec.C), pitch8(spec.K), pitch8(spec.C))
    else:
        _check_full(spec, 300 + sum(case))


@pytest.mark.parametrize("case", [c for c, padded in RAGGED if padded] + [(2, 20, 20, 45, 38, 3, 1, 1),
                                                                          (2, 20, 20, 63, 40, 3, 1, 1),
                                                                          (2, 14, 14, 209, 45, 1, 1, 0)])
def test_ragged_channel_counts_with_zero_padding_vouched(case):
    """PT_CONV_PAD_ZERO: the inputs' padding channels are zero and the kernels skip clearing them."""
    from gpu_util import pitch8
    spec = _spec(*case)
    _check_full(spec, 400 + sum(case), pitch8(spec.C), pitch8(spec.K), pitch8(spec.C), pad_zero=True)


@pytest.mark.parametrize("R,S,pad", [(1, 33, 16), (1, 40, 20), (1, 64, 31), (2, 32, 16), (40, 1, 20), (1, 9, 4), (1, 65, 32)])
@pytest.mark.parametrize("C,K", [(64, 40), (12, 24), (56, 16)])
def test_long_filters(R, S, pad, C, K):
    """Filter rows past the 32 taps of a 32-bit mask, runs of folded taps past the eight blocks of the table of tails (NaN in
    the channel padding), and more taps than the direct kernel has bits for."""
    from gpu_util import pitch8
    _check_full(wl.ConvSpec("t", 1, 45, 47, C, K, R, S, 1, pad, None, None), 700 + R + S + C, pitch8(C), pitch8(K), pitch8(C))


MANY_TILES = [
    # launches with more tiles than the chip holds workgroups at once (650 - 770 pixel tiles, all whole), in both
    # pipeline depths of the direct kernel and with one, two, four and nine reduction steps per tile
    ((5, 128, 130, 64, 64, 1, 1, 0), False),    # one step per tile, three stages; input gradient alike
    ((5, 128, 130, 64, 128, 1, 1, 0), False),   # one step per tile, two stages; input gradient: two steps
    ((5, 128, 130, 128, 128, 1, 1, 0), False),  # two steps per tile, two stages, both directions
    ((7, 128, 100, 24, 64, 1, 1, 0), False),    # partial 64-channel block
    ((5, 128, 130, 64, 64, 3, 1, 1), False),    # nine steps per tile, image borders
    ((17, 128, 160, 64, 64, 2, 2, 0), False),   # strided: four input-gradient classes, scattered destination pixels
    ((6, 256, 256, 3, 64, 7, 2, 3), True),      # image-like input, filter rows folded, zero padding vouched for
    # 1 x 1 layers with several resident rounds of tiles: ragged channel counts on either side, an odd pixel count (the
    # last tile is partial and the last pixel has no partner in the paired stores)
    ((17, 55, 55, 40, 209, 1, 1, 0), True),     # forward: 402 x 2 tiles of 128 x 128, one partial reduction step
    ((24, 55, 55, 209, 33, 1, 1, 0), True),     # forward: 568 narrow tiles, four steps; input gradient: 568 x 2 tiles
    ((9, 128, 128, 72, 136, 1, 1, 0), False),   # channel counts multiples of 8 but not of 64, padding not vouched for
]


@pytest.mark.parametrize("case,pad_zero", MANY_TILES, ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else str(c))
def test_many_whole_tiles(case, pad_zero):
    from gpu_util import pitch8
    spec = _spec(*case)
    _check_full(spec, 600 + sum(case), pitch8(spec.C), pitch8(spec.K), pitch8(spec.C), pad_zero=pad_zero)


FEW_TILES = [
    # problems of few tiles with long reductions: the waves of a workgroup divide the reduction of one small tile
    ((1, 31, 1, 520, 33, 1, 1, 0), False),      # one pixel and one channel off a 32 x 32 tile, a partial 64-channel step
    ((3, 11, 1, 1032, 31, 1, 1, 0), False),     # seventeen steps in stages of four
    ((2, 16, 16, 256, 96, 3, 1, 1), False),     # whole 32 x 32 tiles both ways, image borders
    ((10, 28, 28, 192, 65, 3, 1, 1), False),    # 64 x 64 tiles, one channel past the tile
    ((8, 28, 28, 130, 120, 3, 1, 1), True),     # undefined lanes of a 64-block masked, zero padding vouched for
    ((4, 28, 28, 133, 264, 3, 1, 1), True),     # ragged output tail in the gradient
    ((6, 28, 28, 136, 264, 3, 2, 1), False),    # strided: four classes under one choice, scattered destination pixels
    ((8, 14, 13, 512, 512, 3, 2, 1), False),    # the same, odd grid
    ((8, 15, 14, 256, 512, 1, 2, 0), False),    # strided 1 x 1: zeros for the untouched pixels, cells cut by the border
    ((8, 15, 15, 253, 512, 1, 3, 0), True),     # the same at stride 3, ragged channels
    ((4, 32, 32, 5, 16, 5, 1, 2), True),        # filter rows folded
    ((4, 24, 23, 297, 5, 4, 3, 2), True),       # nine classes, four to a launch, 64 x 64 tiles,
    ((15, 6, 7, 13, 128, 5, 3, 2), True),       # ... 32 x 32 tiles
    ((2, 7, 7, 2048, 520, 1, 1, 0), False),     # weights the larger operand: neighbouring tiles share weights
    # input gradients of 45, 40 and 39 steps in 135 tiles of 128 x 64
    ((2, 17, 18, 1697, 290, 3, 1, 1), True), ((2, 17, 18, 1696, 2560, 1, 1, 0), False), ((2, 17, 18, 1696, 2496, 1, 1, 0), False),
]


@pytest.mark.parametrize("case,pad_zero", FEW_TILES, ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else str(c))
def test_few_tiles_with_long_reductions(case, pad_zero):
    from gpu_util import pitch8
    spec = _spec(*case)
    _check_full(spec, 700 + sum(case), pitch8(spec.C), pitch8(spec.K), pitch8(spec.C), pad_zero=pad_zero)


DEEP = [
    # forward in 128 x 128 tiles: 1 x 1 and 3 x 3, ragged on every side (256 tiles, 5 and 18 steps), a stride, 4 steps
    ((5, 20, 20, 300, 1990, 1, 1, 0), True), ((5, 20, 20, 70, 1990, 3, 1, 1), True), ((8, 31, 31, 256, 1921, 1, 2, 0), True),
    # ... in 256 x 128 tiles (294 tiles of 128 x 128, 154 of these), whole and ragged
    ((7, 19, 20, 72, 1697, 3, 1, 1), True), ((7, 19, 20, 1024, 1696, 1, 1, 0), False),
    # whole channel blocks with padding in both; 1 x 1, ragged, in 256 x 128 tiles
    ((5, 20, 21, 64, 1024, 3, 1, 1), False), ((8, 17, 18, 128, 1690, 3, 1, 1), False), ((7, 19, 20, 1020, 1696, 1, 1, 0), True),
]


@pytest.mark.parametrize("case,pad_zero", DEEP, ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else str(c))
def test_fragments_a_step_ahead(case, pad_zero):
    from gpu_util import pitch8
    spec = _spec(*case)
    _check_full(spec, 700 + sum(case), pitch8(spec.C), pitch8(spec.K), pitch8(spec.C), pad_zero=pad_zero)


@pytest.mark.parametrize("C", [60, 64, 128, 200, 256, 320, 512, 590])
@pytest.mark.parametrize("R", [1, 3])
def test_small_tiles_around_their_number_of_stages(C, R):
    """Reductions of one step to past two rounds of the stages of 32 x 32 tiles, with one block of channels a tap and several (1 x
    1: of up to three steps in 128 x 64 tiles)."""
    from gpu_util import pitch8
    spec = _spec(2, 7, 8, C, 70 if R == 3 else 40, R, 1, R // 2)
    _check_full(spec, 800 + C + R, pitch8(spec.C), pitch8(spec.K), pitch8(spec.C), pad_zero=True)


# Calls in 64 x 64 tiles (four stages of a step): gradients of two to five steps that also clear pixels, forward calls of six to
# nine, and gradients of four classes, of one to four and of two to eight.
TILES_64 = ([("bwd_data", (16, 14, 14, 330, 64 * n - 4, 1, 2, 0)) for n in range(2, 6)] +
            [("fwd", (16, 14, 14, 64 * n - 4, 130, 1, 1, 0)) for n in range(6, 10)] +
            [("bwd_data", (2, 28, 28, 130, K, 3, 2, 1)) for K in (60, 120)])


@pytest.mark.parametrize("call,case", TILES_64, ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else c)
def test_tiles_of_64_by_64_around_their_number_of_stages(call, case):
    from gpu_util import pitch8
    spec = _spec(*case)
    _check_full(spec, 850 + sum(case), pitch8(spec.C), pitch8(spec.K), pitch8(spec.C), pad_zero=True)


FIRST_LAYER = [
    # image-like inputs (at most 4 channels at a pitch of 8, zero padding vouched for): the first-layer forward kernel
    (2, 33, 35, 1, 20, 3, 1, 1),      # one channel, 3 x 3 at stride 1 (one step per filter row)
    (3, 40, 70, 2, 70, 5, 1, 2),      # two channels, 5 x 5, two output-channel tiles with a ragged second one
    (2, 41, 150, 4, 64, 7, 1, 3),     # four channels, 7 x 7 at stride 1, rows of three tiles (the last partial)
    (2, 37, 37, 3, 40, 3, 2, 1),      # 3 x 3 at stride 2
    (2, 50, 50, 3, 100, 5, 2, 2),     # 5 x 5 at stride 2 (filter rows past the fifth multiply zeros)
    (2, 24, 24, 4, 24, 8, 2, 3),      # the largest filter the kernel takes
    (2, 10, 10, 4, 16, 1, 1, 0),      # a single tap
    (3, 21, 21, 3, 12, 2, 2, 0),      # 2 x 2 at stride 2, no padding
    (41, 200, 120, 3, 45, 7, 2, 3),   # 1025 tiles: runs of three tiles per workgroup, the last run of two
    (11, 200, 200, 3, 64, 7, 2, 3),   # 550 tiles: runs of two, alternating between the columns of a tile row
]


@pytest.mark.parametrize("case", FIRST_LAYER, ids=lambda c: "x".join(map(str, c)))
def test_image_like_first_layer(case):
    from gpu_util import pitch8
    spec = _spec(*case)
    _check_full(spec, 800 + sum(case), pitch8(spec.C), pitch8(spec.K), pitch8(spec.C), pad_zero=True)


@pytest.mark.parametrize("case", [(8, 256, 256, 8, 16, 1, 1, 0), (2, 515, 511, 5, 24, 3, 1, 1), (3, 420, 420, 16, 64, 1, 1, 0)],
                         ids=lambda c: "x".join(map(str, c)))
def test_narrow_outputs_over_very_many_pixels(case):
    """More than half a million output pixels with at most 64 output channels: the forward launch takes 256-pixel tiles
    (whole and ragged pixel counts, plain / folded / partial-block reductions)."""
    from gpu_util import pitch8
    spec = _spec(*case)
    _check_full(spec, 700 + sum(case), pitch8(spec.C), pitch8(spec.K), pitch8(spec.C), pad_zero=True)


EARLY_3X3 = [
    # 3 x 3, stride 1, padding 1, at most 64 channels on either side: the kernel that keeps the filter bank in LDS
    # (forward and input gradient); tiles are 4 rows x up to 56 columns
    ((2, 56, 56, 64, 64, 3, 1, 1), False),     # the shape it is for: one tile column of seven 8-pixel blocks
    ((3, 30, 70, 64, 64, 3, 1, 1), False),     # two tile columns (the second partial), a partial last tile row
    ((2, 13, 21, 40, 24, 3, 1, 1), False),     # three column blocks, 24 outputs: one accumulator block, 40 inputs: 2.5 steps
    ((2, 9, 5, 8, 8, 3, 1, 1), False),         # narrower than one block, a single 8-channel chunk
    ((2, 17, 33, 45, 38, 3, 1, 1), True),      # ragged counts, zero padding vouched for
    ((2, 20, 20, 26, 40, 3, 1, 1), True),
    ((2, 6, 60, 33, 56, 3, 1, 1), True),
    ((20, 56, 56, 32, 64, 3, 1, 1), False),    # 280 tiles: runs of two tiles per workgroup, the last run of one
    ((37, 28, 28, 16, 48, 3, 1, 1), False),    # 259 tiles of four blocks
    ((2, 20, 20, 48, 64, 3, 1, 1), False),     # input gradient: four 16-channel steps per tap and two accumulator blocks
    ((40, 32, 32, 16, 16, 3, 1, 1), False),    # several row blocks a tile: two of four column blocks,
    ((60, 23, 25, 45, 38, 3, 1, 1), True),     # ... the last tile row with one block outside the image,
    ((150, 16, 16, 32, 24, 3, 1, 1), False),   # ... four of two,
    ((130, 9, 8, 24, 40, 3, 1, 1), False),     # ... three of one
]


@pytest.mark.parametrize("case,pad_zero", EARLY_3X3, ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else str(c))
def test_early_3x3_layers_with_resident_weights(case, pad_zero):
    from gpu_util import pitch8
    spec = _spec(*case)
    _check_full(spec, 950 + sum(case), pitch8(spec.C), pitch8(spec.K), pitch8(spec.C), pad_zero=pad_zero)


LAYOUTS = dict(C=[9, 16, 17, 32, 33, 48, 49, 64], K=[7, 32, 33, 50, 64], images=[(3, 10, 12), (110, 11, 55)])  # (330 tiles: runs of two)


@pytest.mark.parametrize("C", LAYOUTS["C"])
@pytest.mark.parametrize("K", LAYOUTS["K"])
@pytest.mark.parametrize("N,H,W", LAYOUTS["images"], ids=["one_tile", "runs"])
def test_early_3x3_layers_around_the_layouts_of_bank_and_patch(C, K, N, H, W):
    """One to four 16-channel steps a tap, one and two output blocks, loads of bank and patch left out; one patch buffer and two."""
    from gpu_util import pitch8
    spec = _spec(N, H, W, C, K, 3, 1, 1)
    _check_full(spec, 1700 + C + K, pitch8(C), pitch8(K), pitch8(C), pad_zero=True)


BATCHED_FWD = [
    # independent forward convolutions in one call: pairs that share a launch of the direct kernel (same tile shape and
    # variant: a block's first convolution and its strided shortcut), pairs that do not, and the other kernels mixed in
    [(4, 28, 28, 128, 64, 1, 1, 0), (4, 28, 28, 128, 256, 1, 2, 0)],          # 1x1 and strided 1x1 shortcut, same input shape
    [(6, 56, 56, 256, 128, 1, 1, 0), (6, 56, 56, 256, 512, 1, 2, 0)],         # both 128 x 128 tiles: one launch, two problems
    [(6, 56, 56, 209, 87, 1, 1, 0), (6, 56, 56, 209, 371, 1, 2, 0)],          # ragged widths
    [(2, 14, 14, 64, 64, 3, 1, 1), (2, 14, 14, 64, 256, 1, 1, 0), (2, 14, 14, 64, 64, 1, 1, 0)],   # three problems, mixed shapes
    [(2, 18, 18, 3, 16, 7, 2, 3), (2, 12, 12, 24, 40, 3, 1, 1)],               # an image-like first layer beside a 3 x 3 layer
    [(2, 9, 9, 16, 24, 1, 1, 0)] * 5,                                          # more problems than one launch holds
    # 128 x 128 tiles of different instantiations that share a launch of the more general one: with and without taps outside
    # the image, then with folded filter rows as well, and one folded problem beside one without any test
    [(4, 56, 56, 72, 384, 3, 1, 1), (4, 56, 56, 72, 384, 1, 1, 0)],
    [(4, 56, 56, 72, 384, 1, 1, 0), (4, 56, 56, 24, 384, 3, 1, 1), (4, 56, 56, 72, 384, 3, 1, 1)],
    [(4, 56, 56, 24, 384, 3, 1, 1), (4, 56, 56, 72, 384, 1, 2, 0), (4, 56, 56, 72, 1536, 1, 2, 0)],
]


@pytest.mark.parametrize("cases", BATCHED_FWD, ids=lambda cs: "+".join("x".join(map(str, c)) for c in cs)[:60])
def test_batched_forward_against_oracle_and_single_calls(cases):
    """pt_conv_fwd_batched: every problem's output against the oracle and bit for bit against pt_conv_fwd alone."""
    from gpu_util import CONV_TOL, DEV, dev_bf16, host_bf16, pitch8, rel_err
    from paper_1901_09290_amd import binding as B
    specs = [_spec(*c) for c in cases]
    rng = np.random.Generator(np.random.PCG64(900 + sum(map(sum, cases))))
    descs, xs, ws, ys, singles, refs = [], [], [], [], [], []
    for spec in specs:
        t = wl.conv_tensors(spec, rng, want=("x", "w"))
        xp, yp, wp = pitch8(spec.C), pitch8(spec.K), pitch8(spec.C)
        d = B.desc_of(spec, xp, yp, wp, B.CONV_PAD_ZERO)
        x, w = dev_bf16(t["x"], xp, pad=0), dev_bf16(t["w"], wp, pad=0)   # zero padding, as vouched for
        y = torch.full((spec.N, spec.P, spec.Q, yp), -1, dtype=torch.int16, device=DEV)
        y1 = torch.full_like(y, -1)
        B.conv_fwd(d, x, w, y1)
        descs.append(d); xs.append(x); ws.append(w); ys.append(y); singles.append(y1)
        refs.append(oracle.conv_fwd(oracle.shape_of(spec), t["x"], t["w"]))
    B.conv_fwd_batched(B.conv_fwd_jobs(descs, xs, ws, ys))
    torch.cuda.synchronize()
    for spec, y, y1, ref in zip(specs, ys, singles, refs):
        assert torch.equal(y, y1), spec
        assert rel_err(host_bf16(y, spec.K), ref) <= CONV_TOL, spec


FUSED_LASSO = [
    # N  H   W   C    K   R st pad   flags  path    reductions split over many workgroups, and single-slab ones
    ((2, 12, 12, 64, 64, 3, 1, 1), 3, None),
    ((3, 9, 11, 24, 40, 3, 1, 1), 3, None),
    ((2, 14, 14, 128, 96, 1, 1, 0), 1, None),
    ((2, 15, 15, 40, 136, 3, 2, 1), 2, None),
    ((2, 18, 18, 3, 16, 7, 2, 3), 1, None),          # a first layer: input groups exempt
    ((2, 10, 10, 37, 51, 3, 1, 1), 3, None),         # ragged counts
    ((1, 7, 7, 520, 520, 3, 1, 1), 3, "none"),       # more tiles than the split target: one slab, no split
    ((5, 128, 130, 64, 64, 1, 1, 0), 3, "deep"),     # very many pixels: many slices over few outputs
    # few slices over many outputs (the late layers of a deep network): the wide reduction adds the regulariser
    ((8, 14, 14, 256, 256, 3, 1, 1), 3, "wide"),
    ((8, 14, 14, 203, 171, 3, 1, 1), 3, "wide"),     # the same with ragged counts
    ((8, 14, 14, 203, 171, 3, 1, 1), 1, "wide"),
    ((8, 14, 14, 203, 171, 3, 1, 1), 2, "wide"),
    ((16, 14, 14, 520, 264, 1, 1, 0), 3, "wide"),
]


@pytest.mark.parametrize("case,flags,path", FUSED_LASSO,
                         ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else str(c))
@pytest.mark.parametrize("padded", [True, False])
def test_weight_gradient_with_regulariser_folded_in(case, flags, path, padded):
    """pt_conv_bwd_weight_lasso against the oracle's weight gradient plus the oracle's lasso gradient (convolution
    tolerance on the sum, 1e-5 on the added term itself), and against the two separate GPU calls.  Where a case is
    meant for one of the reduction passes, the library's own plan must say that it takes it."""
    from gpu_util import CONV_TOL, DEV, F32_TOL, dev_bf16, dev_f32, pitch8, rel_err, workspace
    from paper_1901_09290_amd import binding as B
    spec = _spec(*case)
    if path is not None and padded:
        info = B.conv_bwd_weight_plan(B.desc_of(spec, pitch8(spec.C), pitch8(spec.K), pitch8(spec.C)), True)
        kinds = {"none": B.WGRAD_REDUCE_NONE, "deep": B.WGRAD_REDUCE_DEEP, "wide": B.WGRAD_REDUCE_WIDE}
        assert info.reduce_kind == kinds[path], (case, info.splits, info.tiles, info.reduce_kind)
        assert (info.splits == 1) == (path == "none")
    rng = np.random.Generator(np.random.PCG64(800 + sum(case) + flags))
    t = wl.conv_tensors(spec, rng, want=("x", "dy"))
    w = (rng.standard_normal((spec.K, spec.R, spec.S, spec.C)) * 0.05).astype(np.float32)
    w[0] = 0.0                    # a zero output group and a zero input group: their terms are exactly 0
    w[..., spec.C - 1] = 0.0
    lam = 0.5                     # large, so that the added term is visible beside the data gradient
    xp, yp, wp = (pitch8(spec.C), pitch8(spec.K), pitch8(spec.C)) if padded else (spec.C, spec.K, spec.C)
    d = B.desc_of(spec, xp, yp, wp)
    xd, dyd, wd = dev_bf16(t["x"], xp), dev_bf16(t["dy"], yp), dev_f32(w, wp)
    ron, rin = oracle.group_norms(w)
    on = torch.from_numpy(ron.astype(np.float32)).to(DEV)
    inn = torch.from_numpy(rin.astype(np.float32)).to(DEV)
    RS = spec.R * spec.S
    ws = workspace(max(B.conv_bwd_weight_lasso_workspace_bytes(d), B.conv_bwd_weight_workspace_bytes(d)))
    dw_f = torch.full((spec.K, spec.R, spec.S, wp), float("nan"), dtype=torch.float32, device=DEV)
    dw_s = torch.full((spec.K, spec.R, spec.S, wp), float("nan"), dtype=torch.float32, device=DEV)
    B.conv_bwd_weight_lasso(d, xd, dyd, wd, on, inn, lam, flags, dw_f, ws)
    B.conv_bwd_weight(d, xd, dyd, dw_s, ws)
    torch.cuda.synchronize()
    plain = dw_s.cpu().numpy()[..., : spec.C].copy()
    B.group_lasso_grad(wd, on, inn, lam, flags, dw_s, spec.K, RS, spec.C, wp)
    torch.cuda.synchronize()
    fused, separate = dw_f.cpu().numpy()[..., : spec.C], dw_s.cpu().numpy()[..., : spec.C]
    if wp != spec.C:
        assert bool(torch.isnan(dw_f[..., spec.C:]).all())              # padding untouched
    rdw = oracle.conv_bwd_weight(oracle.shape_of(spec), t["x"], t["dy"])
    ref = oracle.group_lasso_grad(w, on.cpu().numpy(), inn.cpu().numpy(), lam, flags, rdw)
    assert rel_err(fused, ref) <= CONV_TOL
    # the added term alone: what the fused call wrote minus the plain weight gradient of the same kernels
    term_ref = oracle.group_lasso_grad(w, on.cpu().numpy(), inn.cpu().numpy(), lam, flags, np.zeros_like(rdw))
    # (one fp32 rounding of the sum, a few ulps of the larger operand, plus 1e-5 of the term)
    big = np.maximum(np.abs(plain), np.abs(fused)).astype(np.float32)
    slack = 4 * np.spacing(big).astype(np.float64) + 1e-5 * (np.abs(term_ref) + np.sqrt(np.mean(term_ref ** 2)))
    assert np.all(np.abs(fused.astype(np.float64) - plain - term_ref) <= slack)
    assert rel_err(fused, separate) <= F32_TOL
    if flags == 1:
        assert np.array_equal(fused[0], plain[0])                       # zero output group: nothing added


def test_results_are_run_to_run_identical():
    from gpu_util import run_conv_all
    spec = _spec(4, 14, 14, 72, 104, 3, 1, 1)
    t = wl.conv_tensors(spec, np.random.Generator(np.random.PCG64(7)))
    a = run_conv_all(spec, t["x"], t["w"], t["dy"])
    b = run_conv_all(spec, t["x"], t["w"], t["dy"])
    for u, v in zip(a, b):
        assert np.array_equal(u, v)


def test_cfg2_resnet32_distinct_layers_full_tensor():
    """Every distinct layer shape of the ResNet-32-shaped stack at batch 128, whole tensors."""
    layers, _ = wl.resnet32_layers(N=128)
    rng_seed = 1
    for i, (spec, _) in enumerate(wl.distinct_shapes(layers)):
        errs = _check_full(spec, rng_seed * 1000 + i)
        print(spec.name, spec.shape_key(), "metric", ["%.2e" % e for e in errs[:3]], "element-wise", ["%.2e" % e for e in errs[3:]],
              flush=True)


@pytest.mark.parametrize("K,RS,C,pitch,shift_in,shift_out", [
    (1, 1, 1, 8, 0, 0), (8, 9, 8, 8, 0, 0), (63, 2, 65, 72, 0, 0), (64, 3, 64, 64, 0, 0), (65, 1, 63, 64, 0, 0), (200, 1, 136, 136, 0, 0),
    (71, 2, 37, 40, 0, 0), (130, 9, 70, 70, 0, 0), (66, 1, 129, 131, 0, 0), (64, 1, 72, 72, 1, 0), (64, 2, 72, 72, 0, 1), (9, 4, 77, 80, 3, 5)])
def test_transposed_weight_copy(K, RS, C, pitch, shift_in, shift_out):
    """Edges of the 64 x 64 tiles, rows that are no multiple of 16 bytes and buffers that do not start on one (`shift`, in
    elements), as the middle one of three jobs: exact, padding of k zero, nothing else written."""
    import torch
    from gpu_util import DEV
    from paper_1901_09290_amd import binding as B
    kp = (K + 7) // 8 * 8
    src = torch.randint(-32768, 32767, (K * RS * pitch + shift_in,), dtype=torch.int16, device=DEV)
    dst = torch.full((3, C * RS * kp + shift_out + 8), 7, dtype=torch.int16, device=DEV)
    w = src[shift_in:]
    job = lambda i: B.layer_crsk(w.view(torch.bfloat16), dst[i, shift_out:].view(torch.bfloat16), K, RS, C, pitch)
    B.weights_to_crsk_batched([job(0), job(1), job(2)])
    torch.cuda.synchronize()
    want = torch.zeros((C, RS, kp), dtype=torch.int16, device=DEV)
    want[..., :K] = w.view(K, RS, pitch)[..., :C].permute(2, 1, 0)
    for i in range(3):
        got = dst[i, shift_out:]
        assert torch.equal(got[: want.numel()].view(want.shape), want)
        assert (got[want.numel():] == 7).all() and (dst[i, :shift_out] == 7).all()


@pytest.mark.parametrize("case", [(2, 15, 15, 40, 136, 3, 2, 1), (2, 10, 10, 37, 51, 3, 1, 1), (2, 16, 16, 64, 128, 1, 2, 0)])
def test_bwd_data_from_pretransposed_weights(case):
    """pt_weights_to_crsk_batched + pt_conv_bwd_data_crsk: the transposed copy is an exact permutation
    (k padding zero) and the input gradient is bit-identical to pt_conv_bwd_data's."""
    import torch
    from gpu_util import DEV, dev_bf16, empty_bf16, pitch8, workspace
    from paper_1901_09290_amd import binding as B
    spec = _spec(*case)
    t = wl.conv_tensors(spec, np.random.Generator(np.random.PCG64(900 + sum(case))))
    xp, yp, wp = pitch8(spec.C), pitch8(spec.K), pitch8(spec.C)
    d = B.desc_of(spec, xp, yp, wp)
    wd, dyd = dev_bf16(t["w"], wp), dev_bf16(t["dy"], yp)
    RS = spec.R * spec.S
    wt = torch.full((spec.C, RS, yp), float("nan"), dtype=torch.bfloat16, device=DEV)
    other = torch.full((7, 1, 8), float("nan"), dtype=torch.bfloat16, device=DEV)   # a second job in the same launch
    w2 = dev_bf16(np.arange(5 * 7, dtype=np.float32).reshape(5, 1, 7), 8)
    B.weights_to_crsk_batched([B.layer_crsk(wd, wt, spec.K, RS, spec.C, wp), B.layer_crsk(w2, other, 5, 1, 7, 8)])
    dx_a = empty_bf16((spec.N, spec.H, spec.W, xp), fill=0x7FC0)
    dx_b = empty_bf16((spec.N, spec.H, spec.W, xp), fill=0x7FC0)
    B.conv_bwd_data_crsk(d, dyd, wt, dx_a)
    B.conv_bwd_data(d, dyd, wd, dx_b, workspace(B.conv_bwd_data_workspace_bytes(d)))
    torch.cuda.synchronize()
    want = np.zeros((spec.C, RS, yp), dtype=np.float32)
    want[..., : spec.K] = t["w"].reshape(spec.K, RS, spec.C).transpose(2, 1, 0)
    assert np.array_equal(wt.float().cpu().numpy(), want)
    o = other.float().cpu().numpy()
    assert np.array_equal(o[:, 0, :5], np.arange(35, dtype=np.float32).reshape(5, 7).T) and not o[:, 0, 5:].any()
    assert torch.equal(dx_a.view(torch.int16), dx_b.view(torch.int16))


def _random_specs(n, seed):
    """Seeded random small layers: arbitrary (pruned-looking) channel counts, filter sizes 1/3/5/7, strides 1-3."""
    rng = np.random.Generator(np.random.PCG64(seed))
    out = []
    while len(out) < n:
        R = int(rng.choice([1, 1, 3, 3, 5, 7]))
        stride = int(rng.choice([1, 1, 2, 3]))
        pad = int(rng.integers(0, R // 2 + 1))
        H, W = int(rng.integers(max(R, 4), 24)), int(rng.integers(max(R, 4), 24))
        C = int(rng.choice([rng.integers(1, 16), rng.integers(16, 80), rng.integers(80, 300)]))
        K = int(rng.choice([rng.integers(1, 16), rng.integers(16, 80), rng.integers(80, 300)]))
        N = int(rng.integers(1, 5))
        if H + 2 * pad < R or W + 2 * pad < R:
            continue
        out.append((N, H, W, C, K, R, stride, pad))
    return out


@pytest.mark.parametrize("case", _random_specs(36, 20260101), ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("pad_zero", [False, True])
def test_random_ragged_layers(case, pad_zero):
    """Arbitrary widths on 8-padded pitches, padding NaN (kernels clear the tails) or vouched zero."""
    from gpu_util import pitch8
    N, H, W, C, K, R, stride, pad = case
    spec = _spec(N, H, W, C, K, R, stride, pad)
    _check_full(spec, 500 + sum(case), pitch8(C), pitch8(K), pitch8(C), pad_zero=pad_zero)


BATCHED_WGRAD = [
    # N  H   W   C    K   R st pad: every tile configuration and address mode, ragged counts, a first layer, one pixel, and
    # more layers than a launch holds
    (2, 12, 12, 128, 128, 3, 1, 1), (2, 12, 13, 64, 128, 3, 1, 1), (2, 12, 12, 128, 64, 1, 1, 0), (3, 9, 11, 24, 40, 3, 1, 1),
    (2, 15, 15, 40, 136, 3, 2, 1), (2, 15, 15, 130, 51, 1, 2, 0), (2, 18, 18, 3, 16, 7, 2, 3), (1, 1, 1, 8, 8, 1, 1, 0),
    (2, 10, 10, 37, 51, 3, 1, 1), (16, 28, 28, 33, 20, 1, 1, 0), (2, 7, 7, 260, 136, 1, 1, 0), (1, 5, 5, 16, 16, 3, 1, 1),
]


@pytest.mark.parametrize("n,workgroups", [(1, 0), (1, 16), (5, 0), (12, 0), (12, 40), (45, 0)])
def test_batched_weight_gradients_match_the_oracle(n, workgroups):
    """pt_conv_bwd_weight_batched: layers of every kind in one call, with and without the regulariser, against the oracle;
    padding untouched; the same call twice gives the same bits."""
    from gpu_util import CONV_TOL, DEV, dev_bf16, dev_f32, pitch8, rel_err, workspace
    from paper_1901_09290_amd import binding as B
    rng = np.random.Generator(np.random.PCG64(900 + n))
    jobs, checks, keep = [], [], []
    for i in range(n):
        spec = _spec(*BATCHED_WGRAD[i % len(BATCHED_WGRAD)])
        t = wl.conv_tensors(spec, rng, want=("x", "dy"))
        xp, yp = pitch8(spec.C), pitch8(spec.K)
        d = B.desc_of(spec, xp, yp, xp)
        xd, dyd = dev_bf16(t["x"], xp), dev_bf16(t["dy"], yp)
        dw = torch.full((spec.K, spec.R, spec.S, xp), float("nan"), dtype=torch.float32, device=DEV)
        ref = oracle.conv_bwd_weight(oracle.shape_of(spec), t["x"], t["dy"])
        reg = ()
        if i % 3 != 2:
            w = (rng.standard_normal((spec.K, spec.R, spec.S, spec.C)) * 0.05).astype(np.float32)
            ron, rin = oracle.group_norms(w)
            flags = 1 + i % 3 * 2
            reg = (dev_f32(w, xp), torch.from_numpy(ron.astype(np.float32)).to(DEV),
                   torch.from_numpy(rin.astype(np.float32)).to(DEV), flags)
            ref = oracle.group_lasso_grad(w, ron, rin, 0.5, flags, ref)
        jobs.append(B.layer_wgrad(d, xd, dyd, dw, *reg))
        keep.append((xd, dyd, reg))
        checks.append((spec, dw, ref))
    ws = workspace(B.conv_bwd_weight_batched_workspace_bytes(jobs, workgroups))
    B.conv_bwd_weight_batched(jobs, 0.5, ws, workgroups)
    torch.cuda.synchronize()
    first = [dw.clone() for _, dw, _ in checks]
    for spec, dw, ref in checks:
        assert rel_err(dw.cpu().numpy()[..., : spec.C], ref) <= CONV_TOL, spec
        assert bool(torch.isnan(dw[..., spec.C:]).all()), spec
        dw.fill_(float("nan"))
    B.conv_bwd_weight_batched(jobs, 0.5, ws, workgroups)
    torch.cuda.synchronize()
    for a, (_, dw, _) in zip(first, checks):
        assert torch.equal(a.view(torch.int32), dw.view(torch.int32))


def test_batched_input_gradients_match_single_calls():
    """Strided and unstrided problems, some sharing launches, some with a kernel of their own: bit for bit the single calls."""
    from gpu_util import DEV, dev_bf16, pitch8
    from paper_1901_09290_amd import binding as B
    rng = np.random.Generator(np.random.PCG64(31))
    specs = [_spec(*c) for c in [(2, 14, 14, 64, 256, 1, 2, 0), (2, 7, 7, 128, 256, 1, 1, 0), (2, 15, 13, 40, 72, 3, 2, 1),
                                 (2, 12, 12, 32, 48, 3, 1, 1), (2, 9, 9, 37, 51, 1, 1, 0)]]
    descs, dys, wts, dxs, singles = [], [], [], [], []
    for s in specs:
        t = wl.conv_tensors(s, rng, want=("w", "dy"))
        xp, yp = pitch8(s.C), pitch8(s.K)
        d = B.desc_of(s, xp, yp, xp)
        w, wt = dev_bf16(t["w"], xp), torch.zeros((s.C, s.R, s.S, yp), dtype=torch.bfloat16, device=DEV)
        B.weights_to_crsk_batched([B.layer_crsk(w, wt, s.K, s.R * s.S, s.C, xp)])
        dy = dev_bf16(t["dy"], yp)
        dx, dx1 = (torch.full((s.N, s.H, s.W, xp), -1, dtype=torch.int16, device=DEV) for _ in range(2))
        B.conv_bwd_data_crsk(d, dy, wt, dx1)
        descs.append(d); dys.append(dy); wts.append(wt); dxs.append(dx); singles.append(dx1)
    B.conv_bwd_data_crsk_batched(B.conv_fwd_jobs(descs, dys, wts, dxs))
    torch.cuda.synchronize()
    for s, a, b in zip(specs, dxs, singles):
        assert torch.equal(a, b), s


@pytest.mark.parametrize("case", [(3, 5, 1, 19, 13, 1, 1, 0), (3, 1, 6, 19, 13, 1, 1, 0), (7, 1, 1, 21, 35, 1, 1, 0),
                                  (5, 3, 2, 9, 17, 3, 2, 1), (2, 33, 31, 11, 7, 3, 1, 1)])
def test_odd_pitches_and_images_one_pixel_wide_or_high(case):
    """The register-staged kernels' pixel divisions: by one, by two and by what is no power of two."""
    _check_full(_spec(*case), 700 + sum(case))


TILES_32 = [(2, 4, 4, 205, 56, 1, 1, 0), (3, 9, 9, 400, 70, 1, 1, 0), (2, 5, 6, 455, 15, 1, 1, 0),
            (18, 21, 22, 210, 14, 5, 1, 2),    # forward: 260 tiles of 50 stages
            # the four classes of an input gradient: of one stage and two, of one to four, 512 tiles of up to 14
            (3, 6, 6, 25, 20, 3, 2, 1), (1, 8, 9, 68, 78, 3, 2, 1), (5, 14, 14, 500, 407, 3, 2, 1)]


@pytest.mark.parametrize("case", TILES_32)
def test_small_tiles_of_32_by_32(case):
    """Reductions of up to the four stages (of two steps each), and long ones where there are more tiles than CUs."""
    from gpu_util import pitch8
    spec = _spec(*case)
    _check_full(spec, 600 + sum(case), pitch8(spec.C), pitch8(spec.K), pitch8(spec.C), pad_zero=True)


WGRAD_TILES = [
    # N   H   W   C    K   R st pad   tile      splits: one call alone, ragged in both channel counts, every tile form
    ((21, 6, 6, 89, 66, 3, 2, 1), (64, 64), (1, 1)),        # unsplit: the epilogue writes dw (and the regulariser)
    ((9, 9, 9, 577, 319, 3, 2, 1), (128, 64), (1, 1)),
    ((18, 6, 8, 434, 485, 3, 2, 1), (64, 128), (1, 1)),
    ((5, 8, 10, 693, 341, 3, 2, 1), (128, 128), (1, 1)),
    ((23, 10, 11, 109, 69, 1, 2, 0), (64, 64), (2, 4)),     # partial sums: one wavefront per 256 outputs, ...
    ((3, 26, 26, 298, 69, 3, 1, 1), (64, 128), (2, 4)),
    ((2, 33, 34, 681, 11, 3, 1, 1), (128, 64), (2, 4)),
    ((7, 22, 23, 649, 218, 1, 1, 0), (64, 64), (5, 8)),     # ... two, ...
    ((4, 34, 35, 353, 26, 3, 1, 1), (128, 64), (9, 16)),    # ... four
    ((13, 22, 24, 113, 596, 1, 1, 0), (64, 64), (9, 16)),
]


@pytest.mark.parametrize("case,tile,splits", WGRAD_TILES, ids=lambda c: "x".join(map(str, c)))
def test_weight_gradient_tile_forms(case, tile, splits):
    """Every tile form of a weight gradient called alone, written directly and through one, two and four groups of splits,
    without and with the regulariser folded in."""
    from gpu_util import CONV_TOL, dev_bf16, dev_f32, DEV, pitch8, rel_err, workspace
    from paper_1901_09290_amd import binding as B
    spec = _spec(*case)
    xp, yp = pitch8(spec.C), pitch8(spec.K)
    d = B.desc_of(spec, xp, yp, xp)
    info = B.conv_bwd_weight_plan(d, True)
    assert (info.tile_m, info.tile_n) == tile and splits[0] <= info.splits <= splits[1], (info.tile_m, info.tile_n, info.splits)
    rng = np.random.Generator(np.random.PCG64(1000 + sum(case)))
    t = wl.conv_tensors(spec, rng, want=("x", "dy"))
    w = (rng.standard_normal((spec.K, spec.R, spec.S, spec.C)) * 0.05).astype(np.float32)
    w[0] = 0.0
    xd, dyd, wd = dev_bf16(t["x"], xp), dev_bf16(t["dy"], yp), dev_f32(w, xp)
    on, inn = (torch.from_numpy(n.astype(np.float32)).to(DEV) for n in oracle.group_norms(w))
    ws = workspace(max(B.conv_bwd_weight_lasso_workspace_bytes(d), B.conv_bwd_weight_workspace_bytes(d)))
    ref = oracle.conv_bwd_weight(oracle.shape_of(spec), t["x"], t["dy"])
    dw = torch.full((spec.K, spec.R, spec.S, xp), float("nan"), dtype=torch.float32, device=DEV)
    B.conv_bwd_weight(d, xd, dyd, dw, ws)
    assert rel_err(dw.cpu().numpy()[..., : spec.C], ref) <= CONV_TOL
    B.conv_bwd_weight_lasso(d, xd, dyd, wd, on, inn, 0.5, 3, dw, ws)
    ref = oracle.group_lasso_grad(w, on.cpu().numpy(), inn.cpu().numpy(), 0.5, 3, ref)
    assert rel_err(dw.cpu().numpy()[..., : spec.C], ref) <= CONV_TOL
    if xp != spec.C:
        assert bool(torch.isnan(dw[..., spec.C:]).all())


def test_weight_gradient_rows_past_the_direct_kernels_addressing():
    """A dw row of more than 2^22 elements (a wide pitch): the register-staged kernel takes the layer."""
    spec = _spec(2, 9, 9, 24, 3, 1, 1, 0)
    _check_full(spec, 1100, 24, 8, (1 << 22) + 8)


@pytest.mark.parametrize("C,K,pad_zero", [(8, 8, False), (64, 48, False), (16, 64, False), (48, 64, False), (40, 24, False),
                                          (9, 17, True), (33, 56, True), (63, 45, True), (1, 64, True), (64, 3, True)])
@pytest.mark.parametrize("extra", [0, 8])
def test_early_3x3_input_gradient_transposes_the_filter_bank_itself(C, K, pad_zero, extra):
    """pt_conv_bwd_data, where the kernel reads the filter bank as it is, against the same kernel on the k-innermost copy: bit
    for bit; NaN in the filters' channel padding reaches nothing, the workspace is not needed for the result."""
    from gpu_util import DEV, dev_bf16, host_bf16, pitch8, workspace
    from paper_1901_09290_amd import binding as B
    spec = _spec(3, 14, 19, C, K, 3, 1, 1)
    t = wl.conv_tensors(spec, np.random.Generator(np.random.PCG64(C * 64 + K)), want=("dy", "w"))
    xp, yp, wp = pitch8(C), pitch8(K), pitch8(C) + extra
    d = B.desc_of(spec, xp, yp, wp, B.CONV_PAD_ZERO if pad_zero else 0)
    dy, w = dev_bf16(t["dy"], yp, pad=0) if pad_zero else dev_bf16(t["dy"], yp), dev_bf16(t["w"], wp)
    wt = torch.zeros((C, 9, yp), dtype=torch.bfloat16, device=DEV)
    B.weights_to_crsk_batched([B.layer_crsk(w, wt, K, 9, C, wp)])
    dx = [torch.zeros((3, 14, 19, xp), dtype=torch.bfloat16, device=DEV) for _ in range(2)]
    B.conv_bwd_data(d, dy, w, dx[0], workspace(B.conv_bwd_data_workspace_bytes(d)))
    B.conv_bwd_data_crsk(d, dy, wt, dx[1])
    torch.cuda.synchronize()
    a, b = (host_bf16(v, C) for v in dx)
    assert np.isfinite(a).all() and np.array_equal(a, b)



@pytest.mark.parametrize("C,K,own", [(8, 64, True), (64, 8, True), (48, 16, True), (16, 64, True), (24, 32, True), (31, 23, True),
                                     (17, 33, False), (32, 32, False), (33, 17, False), (33, 56, False), (63, 45, False)])
def test_early_3x3_input_gradient_by_the_size_of_the_filter_bank(C, K, own):
    """pt_conv_bwd_data transposes banks of up to 768 weights a tap (channel counts in eights), of up to 16 input channels all,
    inside the kernel, leaving the workspace as it was, and the others, faster so, through a k-innermost copy in the workspace.  Two tiles a
    workgroup; against the gradient in fp32 and, bit for bit, the call on a k-innermost copy."""
    from gpu_util import CONV_TOL, DEV, dev_bf16, host_bf16, pitch8, rel_err, workspace
    from paper_1901_09290_amd import binding as B
    N, H = 80, 30
    spec = _spec(N, H, H, C, K, 3, 1, 1)
    t = wl.conv_tensors(spec, np.random.Generator(np.random.PCG64(C * 65 + K)), want=("dy", "w"))
    xp, yp = pitch8(C), pitch8(K)
    d = B.desc_of(spec, xp, yp, xp, B.CONV_PAD_ZERO)
    dy, w = dev_bf16(t["dy"], yp, pad=0), dev_bf16(t["w"], xp)
    ws = workspace(B.conv_bwd_data_workspace_bytes(d)).fill_(0x5A)
    wt = torch.zeros((C, 9, yp), dtype=torch.bfloat16, device=DEV)
    B.weights_to_crsk_batched([B.layer_crsk(w, wt, K, 9, C, xp)])
    dx = [torch.zeros((N, H, H, xp), dtype=torch.bfloat16, device=DEV) for _ in range(2)]
    B.conv_bwd_data(d, dy, w, dx[0], ws)
    B.conv_bwd_data_crsk(d, dy, wt, dx[1])
    torch.cuda.synchronize()
    assert bool((ws == 0x5A).all()) == own
    a, b = (host_bf16(v, C) for v in dx)
    assert np.array_equal(a, b)
    ref = torch.nn.functional.conv_transpose2d(torch.from_numpy(t["dy"]).permute(0, 3, 1, 2),
                                               torch.from_numpy(t["w"]).permute(0, 3, 1, 2), padding=1)
    assert rel_err(a, ref.permute(0, 2, 3, 1).numpy()) <= CONV_TOL


@pytest.mark.parametrize("R", [3, 5, 7])
@pytest.mark.parametrize("N,H,W", [(3, 1, 1), (5, 1, 3), (4, 3, 1), (3, 2, 5), (2, 7, 33), (70, 4, 4), (1, 64, 32), (2, 65, 31)])
def test_weight_gradient_taps_outside_small_images(R, N, H, W):
    """'Same'-padded filters on images smaller than the filter, of one column or row, and around a reduction step's pixels:
    which places of an image a tap may use is counted cyclically along the rows and along the images."""
    _check_full(_spec(N, H, W, 72, 40, R, 1, R // 2), 1200 + N + H + W + R)


ROW3 = [
    # N   H   W   C    K  pad_zero: 3 x 3 layers whose three taps of a filter row share a tile (3000 pixels on)
    (26, 14, 14, 64, 64, True),       # whole tiles
    (105, 7, 7, 129, 190, True),      # image rows of eight places, one channel in the last tile
    (1250, 1, 4, 64, 64, False), (400, 4, 4, 64, 63, False),   # one filter row that ever falls inside; small images
    (40, 2, 63, 45, 130, True), (14, 6, 62, 64, 64, False),     # a row is a step of places, or one less
    (3, 41, 43, 203, 171, False),     # slices that end inside a row
    (7, 30, 25, 64, 320, True), (64, 14, 14, 256, 256, True),
]

# ... and layers that take that form called by themselves, some of them of fewer pixels: unsplit and split
ROW3_ALONE = [(64, 14, 14, 256, 256, True), (45, 7, 8, 311, 755, True), (1, 27, 29, 888, 279, False), (400, 4, 4, 300, 800, True), (700, 3, 5, 250, 300, False)]


@pytest.mark.parametrize("N,H,W,C,K,pad_zero", ROW3)
@pytest.mark.parametrize("workgroups", [0, 1, 24, 160])
def test_weight_gradient_three_taps_from_one_tile(N, H, W, C, K, pad_zero, workgroups):
    """The form that multiplies a filter row's taps from one tile of x, unsplit and split, written directly and through the
    reduction, with the regulariser: against the oracle, and the same bits on a second run.  (0: another form for most.)"""
    _check_three_taps(N, H, W, C, K, pad_zero, workgroups)


@pytest.mark.parametrize("N,H,W,C,K,pad_zero", ROW3_ALONE)
def test_weight_gradient_three_taps_from_one_tile_alone(N, H, W, C, K, pad_zero):
    _check_three_taps(N, H, W, C, K, pad_zero, 0)


def _check_three_taps(N, H, W, C, K, pad_zero, workgroups):
    from gpu_util import CONV_TOL, DEV, dev_bf16, dev_f32, pitch8, rel_err, workspace
    from paper_1901_09290_amd import binding as B
    spec = _spec(N, H, W, C, K, 3, 1, 1)
    xp, yp = pitch8(C), pitch8(K)
    rng = np.random.Generator(np.random.PCG64(1300 + N + H + W + C + K))
    t = wl.conv_tensors(spec, rng, want=("x", "dy"))
    w = (rng.standard_normal((K, 3, 3, C)) * 0.05).astype(np.float32)
    pad = 0 if pad_zero else 0x7FC0
    d = B.desc_of(spec, xp, yp, xp, B.CONV_PAD_ZERO if pad_zero else 0)
    xd, dyd, wd = dev_bf16(t["x"], xp, pad), dev_bf16(t["dy"], yp, pad), dev_f32(w, xp)
    on, inn = (torch.from_numpy(n.astype(np.float32)).to(DEV) for n in oracle.group_norms(w))
    ref = oracle.conv_bwd_weight(oracle.shape_of(spec), t["x"], t["dy"])
    ref_l = oracle.group_lasso_grad(w, on.cpu().numpy(), inn.cpu().numpy(), 0.5, 3, ref)
    got = []
    for weights, want in ((None, ref), (wd, ref_l), (wd, ref_l)):
        dw = torch.full((K, 3, 3, xp), float("nan"), dtype=torch.float32, device=DEV)
        jobs = [B.layer_wgrad(d, xd, dyd, dw, *((weights, on, inn, 3) if weights is not None else ()))]
        ws = workspace(B.conv_bwd_weight_batched_workspace_bytes(jobs, workgroups))
        B.conv_bwd_weight_batched(jobs, 0.5, ws, workgroups)
        assert rel_err(dw.cpu().numpy()[..., :C], want) <= CONV_TOL
        if xp != C:
            assert bool(torch.isnan(dw[..., C:]).all())
        got.append(dw)
    assert torch.equal(got[1][..., :C], got[2][..., :C])


@pytest.mark.parametrize("N,H,W,C,K,workgroups", [(26, 14, 14, 64, 64, 24), (64, 14, 14, 200, 136, 96), (400, 4, 4, 120, 70, 24), (3, 41, 43, 203, 171, 0),
                                                  (3, 40, 50, 64, 64, 1), (26, 14, 14, 64, 64, 0)])
def test_weight_gradient_of_infinities_at_the_borders(N, H, W, C, K, workgroups):
    """Infinities and a NaN in border pixels of x: only the taps that read them may show it, whatever form the layer takes."""
    from gpu_util import CONV_TOL, DEV, dev_bf16, pitch8, rel_err, workspace
    from paper_1901_09290_amd import binding as B
    spec = _spec(N, H, W, C, K, 3, 1, 1)
    xp, yp = pitch8(C), pitch8(K)
    t = wl.conv_tensors(spec, np.random.Generator(np.random.PCG64(1380 + N + H)), want=("x", "dy"))
    x = t["x"]
    for c, (n, h, w, v) in enumerate([(0, 0, 0, np.inf), (0, H - 1, W - 1, np.inf), (N - 1, 1, W - 1, -np.inf), (N - 1, H - 1, 0, np.inf), (1, 2, 0, np.nan),
                                      (1, 0, W - 1, np.inf), (N - 1, H - 1, W - 1, np.nan), (2, 1, 1, np.inf)]):
        x[n, h, w, c * 7 % C] = v
    d = B.desc_of(spec, xp, yp, xp, 0)
    xd, dyd = dev_bf16(x, xp, 0x7FC0), dev_bf16(t["dy"], yp, 0x7FC0)
    dw = torch.zeros((K, 3, 3, xp), dtype=torch.float32, device=DEV)
    jobs = [B.layer_wgrad(d, xd, dyd, dw)]
    B.conv_bwd_weight_batched(jobs, 0.0, workspace(B.conv_bwd_weight_batched_workspace_bytes(jobs, workgroups)), workgroups)
    got, want = dw.cpu().numpy()[..., :C], oracle.conv_bwd_weight(oracle.shape_of(spec), x, t["dy"])
    finite = np.isfinite(want)
    assert 0 < np.sum(~finite) < finite.size // 8
    assert np.array_equal(np.isfinite(got), finite)
    assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)])
    assert rel_err(got[finite], want[finite]) <= CONV_TOL


@pytest.mark.parametrize("N", [2891, 2892])
def test_weight_gradient_three_taps_at_the_limit_of_their_offsets(N):
    """The last image of tensors of just under and just over 2^30 bytes, read as one slice (520 channels, 17 x 21): everything else is
    zero, so dw is the last image's.  The larger one is past the row form's offsets."""
    from gpu_util import CONV_TOL, DEV, dev_bf16, rel_err, workspace
    from paper_1901_09290_amd import binding as B
    H, W, C = 17, 21, 520
    spec, one = _spec(N, H, W, C, C, 3, 1, 1), _spec(1, H, W, C, C, 3, 1, 1)
    d = B.desc_of(spec, C, C, C, B.CONV_PAD_ZERO)
    plan = B.conv_bwd_weight_plan(d)
    assert ((plan.tile_m, plan.splits) == (192, 1)) == (N == 2891)
    t = wl.conv_tensors(one, np.random.Generator(np.random.PCG64(1350)), want=("x", "dy"))
    x, dy = (torch.zeros((N, H, W, C), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    x[-1:], dy[-1:] = dev_bf16(t["x"], C, 0), dev_bf16(t["dy"], C, 0)
    dw = torch.empty((C, 3, 3, C), dtype=torch.float32, device=DEV)
    B.conv_bwd_weight(d, x, dy, dw, workspace(B.conv_bwd_weight_workspace_bytes(d)))
    got, want = dw.cpu().numpy(), oracle.conv_bwd_weight(oracle.shape_of(one), t["x"], t["dy"])
    assert rel_err(got, want) <= CONV_TOL
    assert rel_err(got[:, :, :, -40:], want[:, :, :, -40:]) <= CONV_TOL   # (the channels past the limit)


@pytest.mark.parametrize("case", [(4, 16, 16, 16, 16, 3, 1, 1), (2, 15, 15, 40, 136, 3, 2, 1), (64, 14, 14, 64, 64, 3, 1, 1), (2, 18, 18, 3, 16, 7, 2, 3),
                                  (1, 7, 7, 520, 520, 3, 1, 1)], ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("small_workspace", [False, True])
def test_layer_step_is_its_calls(case, small_workspace):
    """A layer's step in one call against its calls one by one: outputs, input gradient and norms bit for bit, the weight gradient
    with the regulariser in either place to F32_TOL."""
    from gpu_util import F32_TOL, rel_err
    from paper_1901_09290_amd import binding as B
    from paper_1901_09290_amd import harness as hz
    gen = torch.Generator(device=hz.DEV)
    gen.manual_seed(7)
    l = hz.ConvLayer(_spec(*case), gen=gen)
    d = l.desc
    ws = hz.make_workspace([l])
    if small_workspace:  # without the slab that the fused weight gradient asks for
        ws = ws[:max(256, B.conv_bwd_data_workspace_bytes(d), B.conv_bwd_weight_workspace_bytes(d),
                     B.group_norms_workspace_bytes(l.spec.K, l.RS, l.spec.C))]
    l.norms(ws); l.fwd(ws); l.bwd_data(ws); l.bwd_weight(ws); l.lasso(0.5)
    want = {n: getattr(l, n).clone() for n in ("y", "dx", "dw", "out_norm", "in_norm", "w_bf16") if getattr(l, n) is not None}
    for n in want:
        getattr(l, n).zero_()
    l.train_step(ws, 0.5)
    for n, v in want.items():
        if n == "dw":
            assert rel_err(l.dw.cpu().numpy(), v.cpu().numpy()) <= F32_TOL
        else:
            assert torch.equal(getattr(l, n), v), n


@pytest.mark.parametrize("case,pad_zero", [((N, H, W, K, C, *r), z) for (N, H, W, C, K, *r), z in DEEP if r[1] == 1],
                         ids=lambda c: "x".join(map(str, c)) if isinstance(c, tuple) else str(c))
def test_fragments_a_step_ahead_in_gradients(case, pad_zero):
    """The sizes of DEEP the other way round: an input gradient by itself against the oracle, and bit for bit the batched call's,
    which takes the forms that share a CU."""
    from gpu_util import CONV_TOL, DEV, dev_bf16, host_bf16, pitch8, rel_err
    from paper_1901_09290_amd import binding as B
    spec = _spec(*case)
    xp, yp = pitch8(spec.C), pitch8(spec.K)
    t = wl.conv_tensors(spec, np.random.Generator(np.random.PCG64(750 + sum(case))), want=("w", "dy"))
    pad = 0 if pad_zero else 0x7FC0
    d = B.desc_of(spec, xp, yp, xp, B.CONV_PAD_ZERO if pad_zero else 0)
    dy = dev_bf16(t["dy"], yp, pad)
    wt = dev_bf16(np.ascontiguousarray(t["w"].transpose(3, 1, 2, 0)), yp, 0)
    dx = [torch.zeros((spec.N, spec.H, spec.W, xp), dtype=torch.bfloat16, device=DEV) for _ in range(2)]
    B.conv_bwd_data_crsk(d, dy, wt, dx[0])
    B.conv_bwd_data_crsk_batched(B.conv_fwd_jobs([d], [dy], [wt], [dx[1]]))
    torch.cuda.synchronize()
    assert torch.equal(dx[0], dx[1])
    assert rel_err(host_bf16(dx[0], spec.C), oracle.conv_bwd_data(oracle.shape_of(spec), t["dy"], t["w"])) <= CONV_TOL


@pytest.mark.parametrize("N,H,W,C,K,pad_zero", [(3, 14, 19, 64, 64, False), (49, 16, 56, 64, 56, False), (50, 15, 55, 59, 61, True), (2, 1, 1, 64, 64, False),
                                                  (36, 31, 32, 64, 64, False), (100, 27, 25, 61, 60, True), (20, 48, 60, 64, 64, False)])
def test_early_3x3_input_gradient_with_a_large_bank(N, H, W, C, K, pad_zero):
    """Resident weights in a gradient by itself: against the oracle and, bit for bit, the batched call, which takes other tiles (and where
    those add in another order, so does the call by itself)."""
    from gpu_util import CONV_TOL, DEV, dev_bf16, host_bf16, pitch8, rel_err
    from paper_1901_09290_amd import binding as B
    spec = _spec(N, H, W, C, K, 3, 1, 1)
    xp, yp = pitch8(C), pitch8(K)
    t = wl.conv_tensors(spec, np.random.Generator(np.random.PCG64(N + H + W)), want=("w", "dy"))
    d = B.desc_of(spec, xp, yp, xp, B.CONV_PAD_ZERO if pad_zero else 0)
    dy, wt = dev_bf16(t["dy"], yp, 0 if pad_zero else 0x7FC0), dev_bf16(np.ascontiguousarray(t["w"].transpose(3, 1, 2, 0)), yp, 0)
    dx = [torch.zeros((N, H, W, xp), dtype=torch.bfloat16, device=DEV) for _ in range(2)]
    B.conv_bwd_data_crsk(d, dy, wt, dx[0])
    B.conv_bwd_data_crsk_batched(B.conv_fwd_jobs([d], [dy], [wt], [dx[1]]))
    ref = oracle.conv_bwd_data(oracle.shape_of(spec), t["dy"], t["w"])
    for v in dx:
        assert rel_err(host_bf16(v, C), ref) <= CONV_TOL
    assert torch.equal(dx[0], dx[1])
