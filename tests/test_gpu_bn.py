"""GPU parity: feature normalisation forward / backward through the C ABI against the fp64 oracle.

Tolerances: per-channel statistics and parameter gradients (fp32 partial sums combined in fp64) 1e-5 in the
metric of gpu_util.rel_err; the bf16 tensors y and dx must land on the bf16 value nearest the oracle's fp64
result for nearly every element (fp32 evaluation may cross a rounding boundary now and then), and never be
further than one bf16 step away: |g - r| <= 2^-7 |r| + 1e-6 rms.
"""
import numpy as np
import pytest

import oracle
from paper_1901_09290_amd import binding as B
from paper_1901_09290_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

STAT_TOL = 1e-5
EPS = 1e-5


def _inputs(pixels, C, seed):
    """Activations like a convolution's output: per-channel scale and offset vary; channel 0 is constant
    (variance 0), channel 1 sits far from zero against its spread (cancellation case)."""
    rng = np.random.Generator(np.random.PCG64(seed))
    scale = np.exp(rng.uniform(-2.0, 1.0, size=C))
    shift = rng.standard_normal(C) * scale
    x = rng.standard_normal((pixels, C)) * scale + shift
    x[:, 0] = 0.75
    if C > 1:
        x[:, 1] = 8.0 + 0.5 * rng.standard_normal(pixels)
    x = wl.to_bf16_grid(x.astype(np.float32))
    dy = wl.to_bf16_grid((rng.standard_normal((pixels, C)) * 0.1).astype(np.float32))
    gamma = (1.0 + 0.2 * rng.standard_normal(C)).astype(np.float32)
    beta = (0.1 * rng.standard_normal(C)).astype(np.float32)
    return x, dy, gamma, beta


def _bf16_close(got, ref, C):
    ref = np.asarray(ref, dtype=np.float64).reshape(-1, C)
    got = np.asarray(got, dtype=np.float64).reshape(-1, C)
    rms = float(np.sqrt(np.mean(ref * ref)))
    bound = 2.0 ** -7 * np.abs(ref) + 1e-6 * rms + 1e-30
    assert np.all(np.abs(got - ref) <= bound), float(np.max(np.abs(got - ref) / bound))
    nearest = wl.to_bf16_grid(ref.astype(np.float32)).astype(np.float64)
    return float(np.mean(got == nearest))


def _run(pixels, C, xp, yp, dyp, dxp, seed):
    from gpu_util import DEV, dev_bf16, empty_bf16, host_bf16, rel_err, workspace
    x, dy, gamma, beta = _inputs(pixels, C, seed)
    xd, dyd = dev_bf16(x, xp), dev_bf16(dy, dyp)
    gd, bd = torch.from_numpy(gamma).to(DEV), torch.from_numpy(beta).to(DEV)
    y, dx = empty_bf16((pixels, yp), fill=0x7FC0), empty_bf16((pixels, dxp), fill=0x7FC0)
    mean, invstd, dgamma, dbeta = (torch.full((C,), float("nan"), device=DEV) for _ in range(4))
    ws = workspace(B.bn_workspace_bytes(pixels, C))
    ws.fill_(0xFF)
    B.bn_fwd(xd, pixels, C, xp, gd, bd, EPS, y, yp, mean, invstd, ws)
    B.bn_bwd(xd, dyd, pixels, C, xp, dyp, gd, mean, invstd, dx, dxp, dgamma, dbeta, ws)
    torch.cuda.synchronize()

    ry, rmean, rinv = oracle.bn_fwd(x.astype(np.float64), gamma, beta, EPS)
    rdx, rdg, rdb = oracle.bn_bwd(x.astype(np.float64), dy.astype(np.float64), gamma, rmean, rinv)
    assert rel_err(mean.cpu().numpy(), rmean) <= STAT_TOL
    assert rel_err(invstd.cpu().numpy(), rinv) <= STAT_TOL
    assert rel_err(dbeta.cpu().numpy(), rdb) <= STAT_TOL
    assert rel_err(dgamma.cpu().numpy(), rdg) <= STAT_TOL
    # the constant channel: variance exactly 0, so invstd = 1/sqrt(eps), y = beta, dx follows the formula
    assert abs(invstd[0].item() - 1.0 / np.sqrt(EPS)) <= 1e-4 / np.sqrt(EPS)
    hit_y = _bf16_close(host_bf16(y, C), ry, C)
    hit_dx = _bf16_close(host_bf16(dx, C), rdx, C)
    assert hit_y >= 0.98 and hit_dx >= 0.98, (hit_y, hit_dx)
    c8 = (C + 7) // 8 * 8
    for t, p in ((y, yp), (dx, dxp)):
        raw = t.view(torch.int16)
        assert bool((raw[:, C:c8] == 0).all())              # padding inside the last vector: written as zero
        assert bool((raw[:, c8:] == 0x7FC0).all())          # further padding: untouched
    return x, dy, gamma, beta, xd, dyd, gd, bd, ws


# (pixels, C, x pitch, y pitch, dy pitch, dx pitch)
CASES = [
    (37, 5, 8, 8, 8, 8),
    (1, 8, 8, 8, 8, 8),                       # one pixel: every variance is 0
    (2, 1, 8, 16, 8, 24),
    (1000, 64, 64, 64, 64, 64),
    (3137, 203, 208, 216, 208, 224),          # ragged channel count, unequal pitches
    (50000, 16, 24, 16, 16, 24),              # many pixel ranges, few channels
    (64 * 14 * 14, 1024, 1024, 1024, 1024, 1024),
    (200, 2048, 2048, 2048, 2048, 2048),      # the channel limit
    (7, 2041, 2048, 2048, 2048, 2048),
    (9001, 811, 816, 816, 816, 816),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[:2])))
def test_bn_forward_backward_match_oracle(case):
    _run(*case, seed=sum(case))


@pytest.mark.parametrize("pixels,C", [
    (1, 17), (7, 371), (256 * 8 * 6 - 1, 320), (256 * 8 * 5 + 3, 371), (512 * 16 * 5 + 9, 376), (2049, 2041), (517, 1032),
])
def test_bn_edges_of_row_batches_and_workgroup_ranges(pixels, C):
    """Rows left over after the batches of eight and four, widths whose vectors do not divide a workgroup, one row a block."""
    p = (C + 7) // 8 * 8
    _run(pixels, C, p, p, p, p, seed=pixels + C)


def test_bn_is_run_to_run_identical_and_full_size():
    """A ResNet-50 stage-1 activation (batch 64, 56x56, 64 channels) compared element by element, twice."""
    from gpu_util import DEV, empty_bf16
    pixels, C = 64 * 56 * 56, 64
    x, dy, gamma, beta, xd, dyd, gd, bd, ws = _run(pixels, C, C, C, C, C, seed=77)
    outs = []
    for _ in range(2):
        y, dx = empty_bf16((pixels, C)), empty_bf16((pixels, C))
        mean, invstd, dgamma, dbeta = (torch.empty((C,), device=DEV) for _ in range(4))
        B.bn_fwd(xd, pixels, C, C, gd, bd, EPS, y, C, mean, invstd, ws)
        B.bn_bwd(xd, dyd, pixels, C, C, C, gd, mean, invstd, dx, C, dgamma, dbeta, ws)
        torch.cuda.synchronize()
        outs.append([t.clone() for t in (y.view(torch.int16), dx.view(torch.int16), mean, invstd, dgamma, dbeta)])
    for a, b in zip(*outs):
        assert torch.equal(a, b)


def test_bn_sums_have_short_chains():
    """The first row that a thread meets is 1, the 97 behind it 2^-25 each, less than half a unit in the last place of 1: one
    sum that takes them all loses them all (2.9e-6).  The plain sum's chain is 3 + 1 additions for a batch of eight rows, 12
    for the batches, 1 for the rows left over; that of the products 25 in each of four sums, 2 for the four, 1 for the rows
    left over; then 4 for the row groups of a workgroup, fp64 and one rounding.  For positive terms the relative error is at
    most that many half units."""
    from gpu_util import DEV, workspace
    pixels, C, ranges, groups = 64 * 56 * 56, 256, 256, 8
    dy = torch.full((pixels, C), 2.0 ** -25, dtype=torch.bfloat16, device=DEV)
    dy.view(ranges, pixels // ranges, C)[:, :groups] = 1.0
    x = torch.zeros_like(dy)
    ones, out = torch.ones(C, device=DEV), [torch.zeros(C, device=DEV) for _ in range(2)]
    ws = workspace(B.bn_workspace_bytes(pixels, C))
    B.bn_bwd(x, dy, pixels, C, C, C, ones, ones, ones, torch.empty_like(x), C, out[0], out[1], ws)
    torch.cuda.synchronize()
    exact = ranges * groups + (pixels - ranges * groups) * 2.0 ** -25
    err = float((out[1].double() - exact).abs().max()) / exact
    assert err <= (3 + 1 + 12 + 1 + 4 + 1) * 2.0 ** -24, err
    assert float((out[0].double() + exact).abs().max()) / exact <= (25 + 2 + 1 + 4 + 1) * 2.0 ** -24   # xhat = -1


FUSED = [
    # N  H   W   C    K   R st pad
    (2, 12, 12, 64, 64, 3, 1, 1),
    (3, 9, 11, 24, 40, 3, 1, 1),
    (2, 14, 14, 128, 96, 1, 1, 0),
    (2, 15, 15, 40, 136, 3, 2, 1),
    (2, 30, 30, 3, 28, 7, 2, 3),       # image-like input, zero padding vouched for
    (2, 13, 13, 45, 38, 3, 1, 1),      # ragged both ways
    (4, 28, 28, 128, 128, 3, 1, 1),    # several pixel tiles, two wave rows per tile
    (1, 1, 1, 8, 8, 1, 1, 0),
    (2, 40, 44, 64, 60, 3, 1, 1),      # early 3 x 3 layers whose columns do not fill the resident kernel's tiles
    (1, 50, 50, 57, 63, 3, 1, 1),
]


def test_statistics_of_small_tiles_have_short_chains():
    """Sums of a small layer's output, taken tile by tile of 128 pixels: every 32nd pixel 1, the others 2^-25 (the weights are
    the unit matrix in the middle of a 3 x 3 filter, so y = x, and the layer is one that takes small tiles).  The 32 partial sums of a channel added one by one lose all but the first (9e-7); added as
    trees the chain is 2 + 5 additions, and a term of its own may be added to each of the four rows' sums."""
    from gpu_util import DEV, dev_bf16, empty_bf16, workspace
    N, H, C = 2, 16, 128
    spec = wl.ConvSpec("t", N, H, H, C, C, 3, 3, 1, 1, None, None)
    w = np.zeros((C, 3, 3, C), dtype=np.float32)
    w[:, 1, 1] = np.eye(C)
    x = np.full((N * H * H, C), 2.0 ** -25, dtype=np.float32)
    x[::32] = 1.0
    d = B.desc_of(spec, C, C, C, B.CONV_PAD_ZERO)
    nbytes, n_partial = B.conv_fwd_stats_workspace(d)
    sums, y = workspace(nbytes), empty_bf16((N * H * H, C), fill=0)
    xd, wd = dev_bf16(x), dev_bf16(w)
    B.conv_fwd_stats(d, xd, wd, y, sums)
    torch.cuda.synchronize()
    assert n_partial == 4 and torch.equal(y, xd)
    got = sums.view(torch.float32)[: 2 * n_partial * C].view(2, n_partial, C).double()
    for which, tiny in enumerate((2.0 ** -25, 2.0 ** -50)):
        exact = 4 + 124 * tiny
        assert float((got[which] - exact).abs().max()) <= (3 + 5) * 2.0 ** -24 * exact


@pytest.mark.parametrize("case", FUSED, ids=lambda c: "x".join(map(str, c)))
def test_conv_with_statistics_epilogue_feeds_the_normalisation(case):
    """pt_conv_fwd_stats + pt_bn_fwd_from_sums against the oracle's convolution, rounded to bf16 as stored, followed
    by the oracle's normalisation; and against the unfused GPU path (same y bit for bit, statistics to 1e-5)."""
    from gpu_util import CONV_TOL, DEV, dev_bf16, empty_bf16, host_bf16, pitch8, rel_err, workspace
    N, H, W, C, K, R, st, pad = case
    spec = wl.ConvSpec("t", N, H, W, C, K, R, R, st, pad, None, None)
    t = wl.conv_tensors(spec, np.random.Generator(np.random.PCG64(900 + sum(case))), want=("x", "w"))
    xp, yp = pitch8(C), pitch8(K)
    d = B.desc_of(spec, xp, yp, xp, B.CONV_PAD_ZERO)
    xd, wd = dev_bf16(t["x"], xp, 0), dev_bf16(t["w"], xp, 0)
    pixels = N * spec.P * spec.Q
    rng = np.random.Generator(np.random.PCG64(7))
    gamma = (1.0 + 0.2 * rng.standard_normal(K)).astype(np.float32)
    beta = (0.1 * rng.standard_normal(K)).astype(np.float32)
    gd, bd = torch.from_numpy(gamma).to(DEV), torch.from_numpy(beta).to(DEV)

    nbytes, n_partial = B.conv_fwd_stats_workspace(d)
    assert n_partial == (pixels + 127) // 128
    sums = workspace(nbytes)
    sums.fill_(0xFF)
    y = empty_bf16((N, spec.P, spec.Q, yp), fill=0)
    z = empty_bf16((pixels, yp), fill=0x7FC0)
    mean, invstd = (torch.full((K,), float("nan"), device=DEV) for _ in range(2))
    B.conv_fwd_stats(d, xd, wd, y, sums)
    B.bn_fwd_from_sums(y, pixels, K, yp, sums, n_partial, gd, bd, EPS, z, yp, mean, invstd)
    # unfused path on the same inputs
    y2 = empty_bf16((N, spec.P, spec.Q, yp), fill=0)
    z2 = empty_bf16((pixels, yp), fill=0x7FC0)
    mean2, invstd2 = (torch.full((K,), float("nan"), device=DEV) for _ in range(2))
    B.conv_fwd(d, xd, wd, y2)
    ws = workspace(B.bn_workspace_bytes(pixels, K))
    B.bn_fwd(y2, pixels, K, yp, gd, bd, EPS, z2, yp, mean2, invstd2, ws)
    torch.cuda.synchronize()
    assert torch.equal(y.view(torch.int16), y2.view(torch.int16))
    assert rel_err(mean.cpu().numpy(), mean2.cpu().numpy()) <= 1e-5
    assert rel_err(invstd.cpu().numpy(), invstd2.cpu().numpy()) <= 1e-5

    ry = oracle.conv_fwd(oracle.shape_of(spec), t["x"], t["w"])
    assert rel_err(host_bf16(y, K), ry) <= CONV_TOL
    ry_stored = wl.to_bf16_grid(ry.astype(np.float32)).astype(np.float64).reshape(pixels, K)
    rz, rmean, rinv = oracle.bn_fwd(ry_stored, gamma, beta, EPS)
    # the two sides round a few outputs to neighbouring bf16 values: the statistics agree to that (derived: one bf16
    # step on a fraction of elements moves a mean by << 1e-3 of the channel's spread)
    assert rel_err(mean.cpu().numpy(), rmean) <= 1e-3
    assert rel_err(invstd.cpu().numpy(), rinv) <= 1e-3
    assert rel_err(host_bf16(z, K), rz) <= CONV_TOL
