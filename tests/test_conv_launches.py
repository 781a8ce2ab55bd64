"""CPU: which kernel a convolution call takes, by the library's own host code (see launches.py)."""
import os
import shutil
import subprocess

import pytest

from launches import HERE, ROOT, of_calls
from paper_1901_09290_amd import binding as B


@pytest.fixture(scope="module")
def launches():
    if shutil.which("gcc") is None:
        pytest.skip("no gcc")
    if not os.path.exists(B._SO):
        from paper_1901_09290_amd import build as hip_build
        hip_build.build()
    build = os.path.join(ROOT, "_build", "launches")
    os.makedirs(build, exist_ok=True)
    so = os.path.join(build, "recorder.so")
    subprocess.run(["gcc", "-std=c11", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "launch_recorder.c")], check=True)
    return lambda calls: of_calls(calls, so)


# Calls of few tiles: (call, N, H, W, C, K, R, stride), us in 128 x 64, 64 x 64 and 32 x 32 tiles (mean of operands in the caches and
# from memory).
FEW_TILES = [
    # reductions of one to four steps
    (("fwd", 1, 11, 13, 96, 32, 1, 2), (2.88, 3.44, 3.38)), (("fwd", 2, 49, 50, 66, 28, 1, 1), (3.36, 3.81, 3.70)),
    (("fwd", 97, 5, 6, 127, 68, 1, 1), (3.56, 4.14, 4.46)), (("fwd", 2, 28, 28, 128, 512, 1, 1), (3.74, 4.19, 7.29)),
    (("fwd", 7, 24, 24, 192, 32, 1, 1), (3.63, 4.15, 4.05)), (("fwd", 46, 14, 14, 69, 133, 1, 2), (3.60, 3.94, 4.63)),
    (("fwd", 1, 18, 19, 128, 1440, 1, 1), (3.79, 4.19, 4.97)), (("bwd_data", 2, 5, 7, 32, 96, 1, 1), (2.91, 3.52, 3.42)),
    (("bwd_data", 24, 20, 22, 32, 96, 1, 1), (3.68, 4.15, 4.81)), (("bwd_data", 1, 6, 7, 63, 72, 1, 1), (3.11, 3.51, 3.39)),
    (("fwd", 31, 10, 12, 320, 96, 1, 1), (4.46, 4.65, 5.28)), (("bwd_data", 11, 5, 6, 1392, 316, 1, 1), (4.65, 4.75, 5.47)),
    # the four classes of a strided gradient, two to eight steps
    (("bwd_data", 25, 15, 17, 352, 96, 3, 2), (6.53, 8.71, 16.26)),
    # a filter smaller than its stride: a tile clears the other pixels of its cells
    (("bwd_data", 41, 6, 8, 64, 96, 1, 2), (4.86, 3.98, 3.85)), (("bwd_data", 2, 46, 48, 608, 177, 1, 2), (6.38, 5.23, 8.17)),
    (("bwd_data", 102, 9, 11, 185, 205, 1, 2), (6.15, 5.18, 7.79)), (("bwd_data", 2, 43, 44, 832, 96, 1, 2), (6.11, 5.13, 8.75)),
    # ... few of them where it is hardly filled
    (("bwd_data", 4, 9, 10, 35, 57, 1, 2), (3.36, 3.88, 3.94)), (("bwd_data", 1, 6, 7, 33, 98, 1, 2), (3.49, 3.77, 3.69)),
    # six steps and more: small tiles, larger ones where there are many
    (("bwd_data", 6, 11, 13, 64, 352, 1, 1), (4.72, 4.65, 4.08)), (("bwd_data", 2, 14, 14, 118, 655, 1, 1), (6.38, 5.83, 4.67)),
    (("fwd", 40, 14, 14, 187, 17, 3, 1), (8.96, 9.01, 6.34)), (("fwd", 12, 9, 9, 224, 480, 3, 2), (12.74, 10.32, 6.86)),
    (("fwd", 32, 7, 7, 820, 324, 1, 1), (7.41, 6.64, 8.88)), (("bwd_data", 37, 9, 11, 154, 80, 3, 1), (8.31, 7.48, 9.69)),
    (("bwd_data", 3, 46, 46, 192, 704, 1, 2), (7.53, 6.25, 6.79)), (("fwd", 14, 8, 9, 441, 1161, 1, 1), (5.52, 6.65, 10.65)),
]


def test_few_tiles_take_the_faster_form(launches):
    forms = [["k_igemm_dl", 128, 64], ["k_igemm_small", 64, 64], ["k_igemm_small", 32, 32]]
    for (c, us), got in zip(FEW_TILES, launches([[*c, c[6] // 2, True] for c, _ in FEW_TILES])):
        assert got[0]["kernel"][:3] == forms[us.index(min(us))], (c, us, got)


def test_near_ties_of_short_reductions_are_one_launch(launches):
    """Four and five steps: with statistics in one launch, and a block's first convolution and its shortcut (as their gradients) in
    the same form, so that a call of both is one launch."""
    for case in [(27, 22, 22, 224, 32, 1, 1, 0), (90, 11, 13, 257, 22, 1, 1, 0), (2, 49, 49, 256, 64, 1, 1, 0), (7, 20, 20, 296, 655, 1, 2, 0)]:
        (got,) = launches([["fwd_stats", *case, True]])
        assert [g["kernel"][:3] for g in got] == [["k_igemm_dl", 128, 64]], (case, got)
    pairs = [("fwd", (4, 56, 56, 256, 64, 1, 1, 0), (4, 56, 56, 256, 512, 1, 2, 0)), ("fwd", (10, 32, 32, 256, 64, 1, 1, 0), (10, 32, 32, 256, 512, 1, 2, 0)),
             ("bwd_data", (8, 28, 28, 82, 293, 1, 1, 0), (8, 56, 56, 195, 293, 1, 2, 0))]
    for call, one, other in pairs:
        a, b = launches([[call, *one, True], [call, *other, True]])
        assert a[0]["kernel"][:3] == b[0]["kernel"][:3], (call, one, other, a, b)


@pytest.mark.parametrize("case", [(24, 24, 24, 297, 5, 4, 3, 2), (62, 16, 16, 289, 4, 5, 3, 2), (18, 27, 27, 328, 51, 5, 3, 2),
                                  (15, 6, 7, 13, 128, 5, 3, 2)])
def test_classes_of_a_gradient_share_launches_whatever_their_number(launches, case):
    """The nine classes of a gradient at stride 3, four to a launch: each four choose one form."""
    (got,) = launches([["bwd_data", *case, True]])
    assert [g["grid"][1] for g in got] == [4, 4, 1], got


def _forms(launches, calls):
    return [[g["kernel"] for g in got] for got in launches([list(c) for c in calls])]


def test_cases_of_the_gpu_tests_reach_the_forms_they_are_for(launches):
    """The lists of test_gpu_conv.py whose cases were chosen for one kernel."""
    from test_gpu_conv import DEEP, TILES_32, TILES_64
    for (call, case), got in zip(TILES_64, _forms(launches, [(call, *case, True) for call, case in TILES_64])):
        assert [k[:3] for k in got] == [["k_igemm_small", 64, 64]], (call, case, got)
    for case, got in zip(TILES_32, _forms(launches, [("fwd", *case, True) for case in TILES_32])):
        assert [k[:3] for k in got] == [["k_igemm_small", 32, 32]], (case, got)
    for case, got in zip(TILES_32[4:], _forms(launches, [("bwd_data", *case, True) for case in TILES_32[4:]])):
        assert [k[:3] for k in got] == [["k_igemm_small", 32, 32]], (case, got)
    deep = _forms(launches, [("fwd", *case, zero) for case, zero in DEEP])
    for (case, _), got in zip(DEEP, deep):
        assert [k[0] for k in got] == ["k_igemm_dl"] and got[0][-1] == 1, (case, got)
    # (tile, ragged, no tap outside the image)
    assert {(k[1], k[2], k[6], k[9]) for (k,) in deep} == {(m, 128, r, a) for m in (128, 256) for r in (0, 1) for a in (0, 1)}


def test_runs_of_tiles_have_two_patch_buffers(launches):
    """The larger images of the early 3 x 3 layers: more LDS than the same rows in one tile a workgroup take, for every layout."""
    from test_gpu_conv import LAYOUTS
    _, (N, H, W) = LAYOUTS["images"]
    shapes = [(C, K) for C in LAYOUTS["C"] for K in LAYOUTS["K"]]
    one, two = ([g[0] for g in launches([["fwd", n, H, W, C, K, 3, 1, 1, True] for C, K in shapes])] for n in (N // 2, N))
    for shape, a, b in zip(shapes, one, two):
        assert a["kernel"] == b["kernel"] and b["kernel"][0] == "k_conv3x3_res" and b["lds"] > a["lds"], (shape, a, b)


def test_stride_1_gradients_by_themselves_take_the_deep_forms(launches):
    """An input gradient at stride 1 takes what a forward call of the same sizes takes; a strided one's classes do without."""
    cases = [(64, 14, 14, 256, 256, 3, 1, 1), (88, 12, 12, 152, 156, 3, 1, 1), (12, 30, 30, 377, 739, 1, 1, 0), (64, 28, 28, 128, 128, 3, 1, 1)]
    got = _forms(launches, [("bwd_data", *c, True) for c in cases])
    assert [k[0][-1] for k in got] == [1, 1, 1, 1], got
    mirrored = _forms(launches, [("fwd", N, H, W, K, C, *r, True) for N, H, W, C, K, *r in cases])
    assert [[k[:6] for k in g] for g in got] == [[k[:6] for k in g] for g in mirrored]
    (strided,) = _forms(launches, [("bwd_data", 64, 28, 28, 256, 256, 3, 2, 1, True)])
    assert [k[-1] for k in strided] == [0], strided


def test_early_3x3_gradients_by_themselves_keep_their_weights_in_lds(launches):
    """Banks of more than 3072 weights a tap: where the tiles fill the eight waves."""
    resident = [(100, 32, 32, 64, 64), (128, 14, 14, 64, 64), (64, 56, 56, 64, 64), (14, 56, 56, 63, 57)]
    others = [(10, 14, 14, 64, 64), (10, 56, 56, 64, 64), (24, 48, 48, 64, 64), (6, 33, 33, 64, 64), (2, 112, 112, 64, 64)]
    got = _forms(launches, [("bwd_data", *c, 3, 1, 1, True) for c in resident + others])
    assert [k[0][0] == "k_conv3x3_res" for k in got] == [True] * 4 + [False] * 5, got
    # ... and forward calls, which take it for smaller banks whatever the image
    wide = [(24, 48, 48, 64, 64), (16, 64, 64, 64, 64), (2, 96, 96, 64, 60), (10, 56, 56, 64, 64)]
    got = _forms(launches, [("fwd", *c, 3, 1, 1, True) for c in resident + [(24, 112, 112, 64, 64), (24, 48, 48, 48, 64)] + wide])
    assert [k[0][0] == "k_conv3x3_res" for k in got] == [True] * 6 + [False] * 4, got


# Sizes around the limits of the row form's offsets: (N, H, W, C, K), and whether it may take them.  Its x is addressed from one pixel
# ahead, so all channels of the last pixel have to lie inside 2^30 bytes counted from there.
ROW3_LIMITS = [((2891, 17, 21, 520, 520), True), ((2892, 17, 21, 520, 520), False), ((12, 91, 240, 2040, 2040), True),
               ((12, 91, 241, 2040, 2040), False), ((2048, 16, 16, 1024, 64), False), ((2047, 16, 16, 64, 1024), True),
               ((2048, 16, 16, 64, 1024), False), ((233016, 8, 8, 32, 32), True), ((233017, 8, 8, 32, 32), False)]


def test_limits_of_three_taps_from_one_tile(launches):
    """With operands beyond its 30 bits, or places beyond 24, a weight gradient takes another form, called alone and in a batched call."""
    for (N, H, W, C, K), ok in ROW3_LIMITS:
        pixels, last = N * H * W, 2 * ((N * H * W + 1) * C)  # (C a multiple of 8: the pitch)
        assert ok == (last <= 1 << 30 and 2 * pixels * K < 1 << 30 and pixels + N * H < 1 << 24)
        got = launches([["bwd_weight", N, H, W, C, K, 3, 1, 1, True], *(["bwd_weight_batched", N, H, W, C, K, 3, 1, 1, True, w] for w in (0, 96))])
        took = ["k_wgrad_row3" in [g["kernel"][0] for g in call] for call in got]
        assert took == [ok, ok, ok and C > 32], (N, H, W, C, K, took)  # (32 channels beside others: estimated to be slower)


@pytest.mark.parametrize("case", [(4, 64, 64, 128, 128, 3, 1, 1), (64, 14, 14, 64, 64, 3, 1, 1), (2, 15, 15, 40, 136, 3, 2, 1), (1, 7, 7, 520, 520, 1, 1, 0),
                                  (2, 18, 18, 3, 16, 7, 2, 3)], ids=lambda c: "x".join(map(str, c)))
def test_a_layer_step_refuses_before_it_launches(launches, case):
    """A workspace that is enough for some of the calls of a layer's step and not for others: refused with nothing launched."""
    N, H, W, Ch, K, R, stride, pad = case
    d = B.conv_desc(N, H, W, Ch, K, R, R, stride, pad, (Ch + 7) // 8 * 8, (K + 7) // 8 * 8, (Ch + 7) // 8 * 8, B.CONV_PAD_ZERO)
    steps = [B.group_norms_workspace_bytes(K, R * R, Ch), B.conv_bwd_data_workspace_bytes(d), B.conv_bwd_weight_workspace_bytes(d),
             B.conv_bwd_weight_lasso_workspace_bytes(d)]
    sizes = sorted({max(0, n + e) for n in steps for e in (-256, 0)} | {0, 9216, 294912})
    got = launches([["layer_step", *case, True, n] for n in sizes])
    for n, g in zip(sizes, got):
        if n < max(steps[:2]):
            assert g == [-3, 0], (n, g)
        elif n >= max(steps[:3]):
            assert len(g) >= 4 and all("kernel" in launch for launch in g), (n, g)
        else:  # (the weight gradient's query covers unaligned tensors too)
            assert g == [-3, 0] or len(g) >= 4, (n, g)


def test_early_3x3_layers_with_statistics_are_one_launch(launches):
    """Large banks on images whose columns do not fill the resident kernel's waves: the same tiles with statistics and without, alone and
    in a batched call, and statistics in the same launch."""
    for case in [(4, 56, 56, 64, 64), (2, 44, 44, 64, 56), (8, 36, 36, 60, 64), (1, 80, 80, 64, 64), (10, 40, 40, 57, 63), (24, 48, 48, 64, 64)]:
        got = _forms(launches, [(call, *case, 3, 1, 1, True) for call in ("fwd", "fwd_stats", "fwd_batched")])
        assert all(len(g) == 1 and g[0][:3] == ["k_igemm_dl", 128, 64] for g in got), (case, got)


# 64 -> 64 channels, 3 x 3: (N, H, W) and whether the resident kernel's rounds are fewer than those of 128 x 64 tiles
ROUNDS = [((31, 32, 32), True), ((30, 33, 33), False), ((10, 56, 56), False), ((11, 56, 56), True), ((18, 56, 56), True), ((20, 56, 56), False),
          ((64, 32, 32), True), ((64, 28, 28), True), ((80, 28, 28), False), ((100, 24, 24), False), ((3, 112, 112), True), ((3, 128, 128), False),
          ((40, 40, 40), False), ((48, 40, 40), True), ((64, 48, 48), True), ((24, 80, 80), True), ((40, 70, 70), False), ((128, 33, 33), False),
          ((64, 56, 56), True)]


def test_early_3x3_layers_with_large_banks_by_rounds(launches):
    """Forward calls and input gradients by themselves alike; a batched gradient leaves the resident kernel to smaller banks."""
    calls = [[(call, *size, 64, 64, 3, 1, 1, True) for size, _ in ROUNDS] for call in ("fwd", "bwd_data", "bwd_data_batched")]
    fwd, alone, batched = (_forms(launches, c) for c in calls)
    for (size, resident), f, a, b in zip(ROUNDS, fwd, alone, batched):
        want = ["k_conv3x3_res"] if resident else ["k_igemm_dl"]
        assert [k[0] for k in f] == want and [k[0] for k in a] == want and [k[0] for k in b] == ["k_igemm_dl"], (size, f, a, b)


def test_cases_of_three_taps_from_one_tile_reach_it(launches):
    """The lists of test_gpu_conv.py for that form: batched calls of one layer planned for few workgroups, and calls by themselves."""
    from test_gpu_conv import ROW3, ROW3_ALONE
    calls = [["bwd_weight_batched", *case[:5], 3, 1, 1, case[5], w] for case in ROW3 for w in (1, 24, 160)]
    calls += [["bwd_weight", *case[:5], 3, 1, 1, case[5]] for case in ROW3_ALONE]
    split = set()
    for call, got in zip(calls, launches(calls)):
        assert got[0]["kernel"] == ["k_wgrad_row3"], (call, got)
        split.add((call[0], len(got)))
    assert split == {("bwd_weight_batched", 1), ("bwd_weight_batched", 2), ("bwd_weight", 1), ("bwd_weight", 2)}


def test_three_taps_from_one_tile_whatever_the_number_of_pixels(launches):
    """By estimated time alone when a call has the chip to itself; beside other kernels from 3000 pixels on."""
    for case, alone, beside in [((60, 7, 7, 512, 512), True, False), ((64, 7, 7, 512, 512), True, False), ((4, 22, 22, 145, 1412), True, False),
                                ((5, 13, 13, 72, 40), False, False), ((15, 14, 14, 256, 256), False, False), ((16, 14, 14, 256, 256), False, True)]:
        a, b = launches([["bwd_weight", *case, 3, 1, 1, True], ["bwd_weight_batched", *case, 3, 1, 1, True, 96]])
        assert [g[0]["kernel"][0] == "k_wgrad_row3" for g in (a, b)] == [alone, beside], (case, a, b)
