"""GPU parity: group norms, lasso gradient, zero-group detection, reconciliation, plan and the
compaction gathers through the C ABI against the fp64 oracle (masks/indices/gathers bit-exact)."""
import numpy as np
import pytest

import oracle
from paper_1901_09290_amd import binding as B
from paper_1901_09290_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _norms_gpu(w, pitch=None, shadow=False):
    from gpu_util import DEV, dev_f32, workspace
    K, C = w.shape[0], w.shape[-1]
    RS = w.size // (K * C)
    pitch = pitch or C
    wd = dev_f32(w, pitch)
    on = torch.full((K,), float("nan"), device=DEV)
    inn = torch.full((C,), float("nan"), device=DEV)
    sh = None
    if shadow:
        sh = torch.empty((K, RS, pitch), dtype=torch.bfloat16, device=DEV)
        sh.view(torch.int16).fill_(0x7FC0)
    ws = workspace(B.group_norms_workspace_bytes(K, RS, C))
    B.group_norms(wd, K, RS, C, pitch, on, inn, sh, ws)
    torch.cuda.synchronize()
    return wd, on, inn, sh


NORM_SHAPES = [(16, 3, 3, 16), (64, 1, 1, 64), (256, 1, 1, 64), (64, 7, 7, 3), (128, 3, 3, 128), (37, 3, 3, 51),
               (203, 1, 1, 811), (512, 1, 1, 2048), (5, 1, 1, 1), (1, 1, 1, 9), (700, 3, 3, 24),
               # one, two, four and eight 16-byte columns per thread, rows that do not fill the last batch of a chunk
               (207, 1, 1, 655), (45, 3, 3, 209), (300, 1, 1, 1000), (2100, 1, 1, 260), (3, 1, 1, 2048), (20, 1, 1, 516),
               (4099, 1, 1, 4), (131, 3, 3, 12), (17, 5, 5, 2047)]


@pytest.mark.parametrize("shape", NORM_SHAPES)
@pytest.mark.parametrize("padded", [False, True])
def test_group_norms_and_shadow(shape, padded):
    from gpu_util import F32_TOL, host_bf16, pitch8, rel_err
    rng = np.random.Generator(np.random.PCG64(sum(shape)))
    w = rng.standard_normal(shape, dtype=np.float32) * np.float32(0.05)
    w[0] = 0.0
    w[..., shape[-1] - 1] = 0.0
    pitch = pitch8(shape[-1]) if padded else shape[-1]
    _, on, inn, sh = _norms_gpu(w, pitch, shadow=True)
    ron, rin = oracle.group_norms(w)
    assert rel_err(on.cpu().numpy(), ron) <= F32_TOL
    assert rel_err(inn.cpu().numpy(), rin) <= F32_TOL
    assert on[0].item() == 0.0 and inn[-1].item() == 0.0          # exact zeros stay exact
    # shadow = round-to-nearest-even bf16 of the master weights, bit for bit
    got = sh.view(torch.int16).cpu().numpy().view(np.uint16).reshape(shape[0], -1, pitch)
    want = wl.bf16_bits(wl.to_bf16_grid(w)).reshape(shape[0], -1, shape[-1])
    assert np.array_equal(got[..., : shape[-1]], want)
    if pitch != shape[-1]:
        assert np.all(got[..., shape[-1]:] == 0x7FC0)


@pytest.mark.parametrize("shape", NORM_SHAPES)
@pytest.mark.parametrize("flags", [3, 1, 2])
def test_group_lasso_grad(shape, flags):
    from gpu_util import F32_TOL, dev_f32, pitch8, rel_err
    rng = np.random.Generator(np.random.PCG64(sum(shape) + flags))
    w = rng.standard_normal(shape, dtype=np.float32) * np.float32(0.05)
    w[0] = 0.0
    w[..., 0] = 0.0
    dw0 = rng.standard_normal(shape, dtype=np.float32)
    lam = 1e-3
    K, C = shape[0], shape[-1]
    RS = w.size // (K * C)
    for pitch in (C, pitch8(C)):
        wd, on, inn, _ = _norms_gpu(w, pitch)
        dwd = dev_f32(dw0, pitch)
        B.group_lasso_grad(wd, on, inn, lam, flags, dwd, K, RS, C, pitch)
        torch.cuda.synchronize()
        got = dwd.cpu().numpy()[..., :C]
        ron, rin = oracle.group_norms(w)
        ref = oracle.group_lasso_grad(w, ron, rin, lam, flags, dw0)
        assert rel_err(got, ref) <= F32_TOL
        if flags == 1:
            assert np.array_equal(got[0], dw0[0])                            # zero out-group: dw untouched
    # pure gradient (dw = 0): 1e-5 on the gradient itself
    wd, on, inn, _ = _norms_gpu(w, C)
    dwd = torch.zeros(shape, dtype=torch.float32, device="cuda:0")
    B.group_lasso_grad(wd, on, inn, lam, flags, dwd, K, RS, C, C)
    torch.cuda.synchronize()
    ref = oracle.group_lasso_grad(w, ron, rin, lam, flags, np.zeros(shape))
    assert rel_err(dwd.cpu().numpy(), ref) <= F32_TOL
    g = dwd.cpu().numpy()
    if flags & 1:
        assert np.all(g[0] == 0.0)
    if flags == 2:
        assert np.all(g[..., 0] == 0.0)


def test_batched_norms_and_lasso_match_oracle_per_layer():
    """All layers of a ResNet-32-shaped stack (plus two ragged ones and an unaligned one) through the
    multi-layer calls: more layers than one launch holds, both loader kinds in one call."""
    from gpu_util import DEV, F32_TOL, dev_f32, host_bf16, pitch8, rel_err
    specs, _ = wl.resnet32_layers(N=1)
    shapes = [(s.K, s.R, s.S, s.C) for s in specs] * 2 + [(203, 1, 1, 811), (37, 3, 3, 51), (64, 3, 3, 37)]
    rng = np.random.Generator(np.random.PCG64(21))
    lam = 2e-3
    ws_h, jobs_n, jobs_l, devs = [], [], [], []
    for i, sh in enumerate(shapes):
        w = rng.standard_normal(sh, dtype=np.float32) * np.float32(0.05)
        w[0] = 0.0
        dw0 = rng.standard_normal(sh, dtype=np.float32)
        K, C = sh[0], sh[-1]
        RS = sh[1] * sh[2]
        pitch = C if i == len(shapes) - 1 else pitch8(C)          # the last layer is stored unaligned
        wd, dwd = dev_f32(w, pitch), dev_f32(dw0, pitch)
        on = torch.full((K,), float("nan"), device=DEV)
        inn = torch.full((C,), float("nan"), device=DEV)
        sh_t = torch.zeros((K, RS, pitch), dtype=torch.bfloat16, device=DEV)
        flags = 1 if i == 0 else 3
        jobs_n.append(B.layer_weights(wd, K, RS, C, pitch, on, inn, sh_t))
        jobs_l.append(B.layer_lasso(wd, on, inn, dwd, K, RS, C, pitch, flags))
        ws_h.append((w, dw0, flags))
        devs.append((wd, dwd, on, inn, sh_t))
    assert len(shapes) > 64
    ws = torch.empty(B.group_norms_batched_workspace_bytes(jobs_n), dtype=torch.uint8, device=DEV)
    B.group_norms_batched(jobs_n, ws)
    B.group_lasso_grad_batched(jobs_l, lam)
    torch.cuda.synchronize()
    for (w, dw0, flags), (wd, dwd, on, inn, sh_t), sh in zip(ws_h, devs, shapes):
        ron, rin = oracle.group_norms(w)
        assert rel_err(on.cpu().numpy(), ron) <= F32_TOL and rel_err(inn.cpu().numpy(), rin) <= F32_TOL
        ref = oracle.group_lasso_grad(w, ron, rin, lam, flags, dw0)
        assert rel_err(dwd.cpu().numpy()[..., : sh[-1]], ref) <= F32_TOL
        got = host_bf16(sh_t, sh[-1]).reshape(sh)
        assert np.array_equal(got, wl.to_bf16_grid(w))
    # running the same call again gives bit-identical norms (fixed reduction order)
    before = [d[2].clone() for d in devs]
    B.group_norms_batched(jobs_n, ws)
    torch.cuda.synchronize()
    assert all(torch.equal(a, d[2]) for a, d in zip(before, devs))


def test_zero_groups_bit_exact_and_threshold_edges():
    from gpu_util import DEV
    rng = np.random.Generator(np.random.PCG64(5))
    n = 5000
    norms = np.abs(rng.standard_normal(n)).astype(np.float32) * np.float32(0.1) + np.float32(1e-2)
    norms[rng.choice(n, 1500, replace=False)] = 0.0
    nd = torch.from_numpy(norms).to(DEV)
    for thr in (1e-6, 1e-4, 0.0, -1.0, 0.05):
        z = torch.full((n,), 7, dtype=torch.uint8, device=DEV)
        B.zero_groups(nd, n, thr, z)
        torch.cuda.synchronize()
        ref = oracle.zero_groups(norms.astype(np.float64), float(np.float32(thr)))
        assert np.array_equal(z.cpu().numpy(), ref)
    # exactly at the threshold: strict comparison
    v = np.array([1e-4, np.nextafter(np.float32(1e-4), np.float32(0)), np.nextafter(np.float32(1e-4), np.float32(1))],
                 dtype=np.float32)
    z = torch.zeros(3, dtype=torch.uint8, device=DEV)
    B.zero_groups(torch.from_numpy(v).to(DEV), 3, float(np.float32(1e-4)), z)
    torch.cuda.synchronize()
    assert z.cpu().numpy().tolist() == [0, 1, 0]
    B.zero_groups(nd, 0, 1.0, z)  # empty input is a no-op


def test_norms_to_masks_match_oracle_near_threshold():
    """fp32 GPU norms vs fp64 oracle norms decide the same mask except inside a relative 1e-5 guard
    band around the threshold (the only place where both answers are acceptable)."""
    from gpu_util import DEV
    rng = np.random.Generator(np.random.PCG64(6))
    K, RS, C = 300, 9, 40
    scale = (10.0 ** rng.uniform(-6, -2, size=(K, 1, 1))).astype(np.float32)
    w = (rng.standard_normal((K, RS, C), dtype=np.float32) * scale).astype(np.float32)
    thr = 1e-4
    _, on, inn, _ = _norms_gpu(w.reshape(K, 3, 3, C))
    z = torch.zeros(K, dtype=torch.uint8, device=DEV)
    B.zero_groups(on, K, thr, z)
    torch.cuda.synchronize()
    ron, _ = oracle.group_norms(w)
    ref = oracle.zero_groups(ron, thr)
    safe = np.abs(ron - thr) > 1e-5 * thr
    assert safe.sum() > K - 5 and ref.sum() > 10 and ref.sum() < K - 10
    assert np.array_equal(z.cpu().numpy()[safe], ref[safe])


@pytest.mark.parametrize("n,n_prod,n_cons", [(64, 1, 1), (2048, 4, 5), (37, 7, 0), (1000, 0, 3), (1, 2, 2)])
def test_reconcile_and_plan_bit_exact(n, n_prod, n_cons):
    from gpu_util import DEV
    rng = np.random.Generator(np.random.PCG64(n + n_prod))
    masks = [(rng.random(n) < 0.7).astype(np.uint8) for _ in range(n_prod + n_cons)]
    md = [torch.from_numpy(m).to(DEV) for m in masks]
    keep = torch.full((n,), 9, dtype=torch.uint8, device=DEV)
    B.reconcile_edge(md[:n_prod], md[n_prod:], n, keep)
    idx = torch.full((n,), -1, dtype=torch.int32, device=DEV)
    cnt = torch.full((1,), -1, dtype=torch.int32, device=DEV)
    B.compact_plan(keep, n, idx, cnt)
    torch.cuda.synchronize()
    rkeep = oracle.reconcile_edge(masks[:n_prod], masks[n_prod:])
    ridx = oracle.compact_plan(rkeep)
    assert np.array_equal(keep.cpu().numpy(), rkeep)
    assert cnt.item() == ridx.size
    assert np.array_equal(idx.cpu().numpy()[: ridx.size], ridx)
    assert np.all(idx.cpu().numpy()[ridx.size:] == -1)


@pytest.mark.parametrize("n", [0, 1, 63, 64, 1023, 1024, 1025, 5000])
@pytest.mark.parametrize("mode", ["all", "none", "random"])
def test_plan_edge_cases(n, mode):
    from gpu_util import DEV
    rng = np.random.Generator(np.random.PCG64(n))
    keep = {"all": np.ones(n, np.uint8), "none": np.zeros(n, np.uint8),
            "random": (rng.random(n) < 0.5).astype(np.uint8) * 3}[mode]       # any non-zero byte keeps
    kd = torch.from_numpy(keep).to(DEV) if n else torch.empty(1, dtype=torch.uint8, device=DEV)
    idx = torch.full((max(n, 1),), -1, dtype=torch.int32, device=DEV)
    cnt = torch.full((1,), -1, dtype=torch.int32, device=DEV)
    B.compact_plan(kd, n, idx, cnt)
    torch.cuda.synchronize()
    ridx = oracle.compact_plan(keep)
    assert cnt.item() == ridx.size
    assert np.array_equal(idx.cpu().numpy()[: ridx.size], ridx)


@pytest.mark.parametrize("shape,pad_out", [((16, 3, 3, 16), False), ((203, 1, 1, 811), True), ((64, 7, 7, 3), False),
                                           ((130, 3, 3, 37), True)])
def test_compact_weights_bit_exact(shape, pad_out):
    from gpu_util import DEV, dev_f32, pitch8
    rng = np.random.Generator(np.random.PCG64(sum(shape)))
    K, C = shape[0], shape[-1]
    RS = shape[1] * shape[2]
    w = rng.standard_normal(shape, dtype=np.float32)
    ik = np.sort(rng.choice(K, max(1, K * 2 // 3), replace=False)).astype(np.int32)
    ic = np.sort(rng.choice(C, max(1, C * 3 // 5), replace=False)).astype(np.int32)
    wd = dev_f32(w)
    for use_k, use_c in ((True, True), (True, False), (False, True)):
        Kp, Cp = (ik.size if use_k else K), (ic.size if use_c else C)
        op = pitch8(Cp) if pad_out else Cp
        out = torch.full((Kp, RS, op), float("nan"), dtype=torch.float32, device=DEV)
        B.compact_weights(wd, K, RS, C, C, torch.from_numpy(ik).to(DEV) if use_k else None, Kp,
                          torch.from_numpy(ic).to(DEV) if use_c else None, Cp, out, op)
        torch.cuda.synchronize()
        ref = oracle.compact_weights(w, ik if use_k else None, ic if use_c else None).astype(np.float32)
        got = out.cpu().numpy()
        assert np.array_equal(got[..., :Cp].reshape(ref.shape), ref)
        assert np.all(np.isnan(got[..., Cp:]))


def test_compact_vector_bit_exact():
    from gpu_util import DEV
    rng = np.random.Generator(np.random.PCG64(11))
    n = 2048
    idx = np.sort(rng.choice(n, 1301, replace=False)).astype(np.int32)
    idd = torch.from_numpy(idx).to(DEV)
    for dt in (np.uint8, np.int16, np.float32, np.float64):
        v = (rng.standard_normal(n) * 100).astype(dt)
        out = torch.zeros(idx.size, dtype=getattr(torch, np.dtype(dt).name), device=DEV)
        B.compact_vector(torch.from_numpy(v).to(DEV), np.dtype(dt).itemsize, idd, idx.size, out)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), oracle.compact_vector(v, idx))
    B.compact_vector(idd, 4, idd, 0, idd)  # empty gather is a no-op


@pytest.mark.parametrize("pixels,C,pad", [(4 * 16 * 16, 16, 0), (3 * 7 * 7, 203, 8), (1000, 64, 8),
                                          (129, 811, 8), (50, 5, 0), (1, 8, 0), (77, 45, 24), (1000, 209, 16),
                                          (33, 21, 3), (9, 30, 13)])
def test_compact_nhwc_bit_exact(pixels, C, pad):
    """pad: 0 = dense rows; 8 = pitches rounded up to 8; 16 / 24 = output pitch with whole spare vectors behind the
    last one; other values = output pitch Cp + pad (rows neither aligned nor a multiple of 8).  Padding channels up
    to the next multiple of 8 are written as zero, the rest of the row is left alone."""
    from gpu_util import DEV, pitch8
    rng = np.random.Generator(np.random.PCG64(pixels + C))
    x = rng.integers(0, 65536, size=(pixels, C)).astype(np.uint16)
    idx = np.sort(rng.choice(C, max(1, int(C * 0.6)), replace=False)).astype(np.int32)
    xp = pitch8(C) if pad % 8 == 0 and pad else C
    op = idx.size if pad == 0 else (pitch8(idx.size) + pad - 8 if pad % 8 == 0 else idx.size + pad)
    xfull = np.full((pixels, xp), 0xDEAD, dtype=np.uint16)
    xfull[:, :C] = x
    xd = torch.from_numpy(xfull.view(np.int16)).to(DEV).view(torch.bfloat16)
    out = torch.empty((pixels, op), dtype=torch.bfloat16, device=DEV)
    out.view(torch.int16).fill_(0x1234)
    B.compact_nhwc(xd, pixels, C, xp, torch.from_numpy(idx).to(DEV), idx.size, out, op)
    torch.cuda.synchronize()
    got = out.view(torch.int16).cpu().numpy().view(np.uint16)
    assert np.array_equal(got[:, : idx.size], oracle.compact_nhwc(x, idx))
    zero_to = min(op, (idx.size + 7) // 8 * 8)
    assert np.all(got[:, idx.size:zero_to] == 0)
    assert np.all(got[:, zero_to:] == 0x1234)


def test_cfg1_reconfiguration_end_to_end():
    """cfg1: norms -> zero masks -> keep -> plan -> compact weights and activations; then the
    compacted layer's forward output equals the kept channels of the full layer's output (GPU vs GPU,
    bit for bit: dropped terms are exact zeros and the survivors are accumulated in the same order
    only if the tiling matches, so compare against the oracle within the conv tolerance instead)."""
    from gpu_util import CONV_TOL, DEV, dev_bf16, host_bf16, rel_err, run_conv_all
    c = wl.cfg1(0)
    spec, w = c["spec"], c["w_master"]
    wd, on, inn, sh = _norms_gpu(w, shadow=True)
    zo = torch.zeros(16, dtype=torch.uint8, device=DEV)
    zi = torch.zeros(16, dtype=torch.uint8, device=DEV)
    B.zero_groups(on, 16, c["thr"], zo)
    B.zero_groups(inn, 16, c["thr"], zi)
    torch.cuda.synchronize()
    assert np.flatnonzero(zo.cpu().numpy()).tolist() == c["zero_out"].tolist()
    assert np.flatnonzero(zi.cpu().numpy()).tolist() == c["zero_in"].tolist()
    keep_k = torch.zeros(16, dtype=torch.uint8, device=DEV)
    keep_c = torch.zeros(16, dtype=torch.uint8, device=DEV)
    B.reconcile_edge([zo], [], 16, keep_k)
    B.reconcile_edge([], [zi], 16, keep_c)
    ik = torch.zeros(16, dtype=torch.int32, device=DEV)
    ic = torch.zeros(16, dtype=torch.int32, device=DEV)
    nk = torch.zeros(1, dtype=torch.int32, device=DEV)
    nc = torch.zeros(1, dtype=torch.int32, device=DEV)
    B.compact_plan(keep_k, 16, ik, nk)
    B.compact_plan(keep_c, 16, ic, nc)
    torch.cuda.synchronize()
    assert nk.item() == 12 and nc.item() == 12
    w2 = torch.empty((12, 9, 12), dtype=torch.float32, device=DEV)
    B.compact_weights(wd, 16, 9, 16, 16, ik, 12, ic, 12, w2, 12)
    xd = dev_bf16(c["x"])
    x2 = torch.empty((4, 16, 16, 12), dtype=torch.bfloat16, device=DEV)
    B.compact_nhwc(xd, 4 * 16 * 16, 16, 16, ic, 12, x2, 12)
    torch.cuda.synchronize()
    rik, ric = ik.cpu().numpy()[:12], ic.cpu().numpy()[:12]
    assert np.array_equal(w2.cpu().numpy().reshape(12, 3, 3, 12), oracle.compact_weights(w, rik, ric).astype(np.float32))
    assert np.array_equal(host_bf16(x2), c["x"][..., ric])
    # compacted layer on the GPU vs the oracle's full layer restricted to kept channels
    spec2 = wl.ConvSpec("cfg1c", 4, 16, 16, 12, 12, 3, 3, 1, 1, None, None)
    wc = wl.to_bf16_grid(w2.cpu().numpy().reshape(12, 3, 3, 12))
    y2, dx2, dw2 = run_conv_all(spec2, host_bf16(x2), wc, c["dy"][..., rik])
    s = oracle.shape_of(spec)
    assert rel_err(y2, oracle.conv_fwd(s, c["x"], c["w"])[..., rik]) <= CONV_TOL
    assert rel_err(dx2, oracle.conv_bwd_data(s, c["dy"], c["w"])[..., ric]) <= CONV_TOL
    assert rel_err(dw2, oracle.conv_bwd_weight(s, c["x"], c["dy"])[rik][..., ric]) <= CONV_TOL


def test_multi_job_reconfiguration_equals_single_calls_and_oracle():
    """A small network with a residual-style shared edge, swept once through the multi-job calls and once
    through the single-tensor calls: identical masks, plans and compacted tensors, and both equal the oracle."""
    from paper_1901_09290_amd import harness as hz
    specs = [
        wl.ConvSpec("m0", 2, 12, 12, 3, 300, 3, 3, 1, 1, None, 0, first=True),
        wl.ConvSpec("m1", 2, 12, 12, 300, 37, 1, 1, 1, 0, 0, 1),
        wl.ConvSpec("m2", 2, 12, 12, 37, 300, 3, 3, 1, 1, 1, 0),
        wl.ConvSpec("m3", 2, 12, 12, 300, 1100, 1, 1, 1, 0, 0, 2),
        wl.ConvSpec("m4", 2, 12, 12, 1100, 9, 1, 1, 1, 0, 2, None),
    ]
    edges = [wl.Edge("e0", 300, [0, 2], [1, 3]), wl.Edge("e1", 37, [1], [2]), wl.Edge("e2", 1100, [3], [4])]
    rng = np.random.Generator(np.random.PCG64(77))
    zero_sets = wl.zeroed_channel_sets(edges, 0.35, rng)
    weights = wl.network_weights(specs, edges, zero_sets, rng)
    a = hz.ReconfigModel(specs, edges, weights, seed=8)
    b = hz.ReconfigModel(specs, edges, weights, seed=8)
    a.detect(1e-6)
    a.compact()
    b.detect_per_call(1e-6)
    b.compact(per_call=True)
    torch.cuda.synchronize()
    assert np.array_equal(a.new_counts, b.new_counts)
    assert a.new_counts.tolist() == [e.n - z.size for e, z in zip(edges, zero_sets)]
    for ta, tb in zip(a.keep + a.zo + a.zi + a.w_out + a.mom_out + a.act_out + [v for vs in a.bn_out for v in vs],
                      b.keep + b.zo + b.zi + b.w_out + b.mom_out + b.act_out + [v for vs in b.bn_out for v in vs]):
        assert torch.equal(ta, tb)
    for e in range(len(edges)):
        n = int(a.new_counts[e])
        keep = np.ones(edges[e].n, dtype=np.uint8)
        keep[zero_sets[e]] = 0
        assert np.array_equal(a.keep[e].cpu().numpy(), keep)
        assert np.array_equal(a.idx[e].cpu().numpy()[:n], oracle.compact_plan(keep))
        assert np.array_equal(b.idx[e].cpu().numpy()[:n], oracle.compact_plan(keep))
    for i, s in enumerate(specs):
        ik = oracle.compact_plan(a.keep[s.out_edge].cpu().numpy()) if s.out_edge is not None else None
        ic = oracle.compact_plan(a.keep[s.in_edge].cpu().numpy()) if s.in_edge is not None else None
        Kp = s.K if ik is None else ik.size
        Cp = s.C if ic is None else ic.size
        op = hz.pitch8(Cp)
        got = a.w_out[i].reshape(-1)[: Kp * s.R * s.S * op].reshape(Kp, s.R, s.S, op).cpu().numpy()[..., :Cp]
        assert np.array_equal(got, oracle.compact_weights(weights[i], ik, ic).astype(np.float32))
        if ik is not None:
            for v, o in zip(a.bn[i], a.bn_out[i]):
                assert np.array_equal(o.cpu().numpy()[:Kp], oracle.compact_vector(v.cpu().numpy(), ik))


def test_more_jobs_than_one_launch_holds():
    """A chain of 130 tiny layers: more edges, weight-shaped tensors, per-channel vectors and activations than the job
    tables of one launch hold (64 / 112 / 224 / 64), so every multi-job call splits; results equal the single calls."""
    from paper_1901_09290_amd import harness as hz
    rng = np.random.Generator(np.random.PCG64(91))
    n_layers = 130
    widths = [int(rng.integers(9, 41)) for _ in range(n_layers)]
    specs, edges = [], []
    c_in = 3
    for i, k in enumerate(widths):
        specs.append(wl.ConvSpec(f"c{i}", 1, 5, 5, c_in, k, 1, 1, 1, 0, None if i == 0 else i - 1,
                                 i if i + 1 < n_layers else None, first=(i == 0)))
        if i + 1 < n_layers:
            edges.append(wl.Edge(f"e{i}", k, [i], [i + 1]))
        c_in = k
    zero_sets = wl.zeroed_channel_sets(edges, 0.3, rng)
    weights = wl.network_weights(specs, edges, zero_sets, rng)
    a = hz.ReconfigModel(specs, edges, weights, seed=5)
    b = hz.ReconfigModel(specs, edges, weights, seed=5)
    a.detect(1e-6)
    a.compact()
    b.detect_per_call(1e-6)
    b.compact(per_call=True)
    torch.cuda.synchronize()
    assert a.new_counts.tolist() == [e.n - z.size for e, z in zip(edges, zero_sets)]
    assert np.array_equal(a.new_counts, b.new_counts)
    for ta, tb in zip(a.keep + a.idx + a.zo + a.zi + a.w_out + a.mom_out + a.act_out + [v for vs in a.bn_out for v in vs],
                      b.keep + b.idx + b.zo + b.zi + b.w_out + b.mom_out + b.act_out + [v for vs in b.bn_out for v in vs]):
        assert torch.equal(ta, tb)
    for i in (0, 63, 64, 111, 112, 129):      # layers on either side of the table boundaries, against the oracle
        s = specs[i]
        ik = oracle.compact_plan(a.keep[s.out_edge].cpu().numpy()) if s.out_edge is not None else None
        ic = oracle.compact_plan(a.keep[s.in_edge].cpu().numpy()) if s.in_edge is not None else None
        Kp = s.K if ik is None else ik.size
        Cp = s.C if ic is None else ic.size
        op = hz.pitch8(Cp)
        got = a.w_out[i].reshape(-1)[: Kp * op].reshape(Kp, 1, 1, op).cpu().numpy()[..., :Cp]
        assert np.array_equal(got, oracle.compact_weights(weights[i], ik, ic).astype(np.float32))


def test_regulariser_value_matches_oracle_and_is_deterministic():
    """GroupLassoReg over a whole network (ResNet-32 shapes + a 100-layer stack that needs two launches):
    device fp64 sum of the device's fp32 norms vs the oracle's fp64 sum of fp64 norms, 1e-5 relative; exact
    against the fp64 sum of the device's own norms; identical on a second run; first-layer exemption honoured."""
    from gpu_util import DEV, F32_TOL
    specs, _ = wl.resnet32_layers(N=2)
    specs = list(specs) + [wl.ConvSpec(f"x{i}", 1, 4, 4, 5 + i % 7, 3 + i % 11, 1, 1, 1, 0, None, None) for i in range(100)]
    rng = np.random.Generator(np.random.PCG64(91))
    jobs, ref_layers, dev_sum, keep = [], [], 0.0, []
    for i, s in enumerate(specs):
        w = wl.master_weights(s, rng)
        flags = 1 if s.first else 3
        wd, on, inn, _ = _norms_gpu(w, shadow=False)
        keep += [wd, on, inn]
        jobs.append(B.layer_penalty(on, inn, s.K, s.C, flags))
        a, b = oracle.group_norms(w)
        ref_layers.append((a, b, flags))
        dev_sum += float(on.double().sum()) + (float(inn.double().sum()) if flags & 2 else 0.0)
    out = torch.full((1,), float("nan"), dtype=torch.float64, device=DEV)
    B.group_lasso_penalty_batched(jobs, out)
    torch.cuda.synchronize()
    got = out.item()
    ref = oracle.group_lasso_penalty(ref_layers)
    assert abs(got - ref) <= F32_TOL * ref
    assert abs(got - dev_sum) <= 1e-12 * ref          # the reduction itself is fp64
    out2 = torch.zeros(1, dtype=torch.float64, device=DEV)
    B.group_lasso_penalty_batched(jobs, out2)
    torch.cuda.synchronize()
    assert out2.item() == got
    B.group_lasso_penalty_batched([], out2)            # no layers: the value is 0
    torch.cuda.synchronize()
    assert out2.item() == 0.0
    # the coefficient that makes the regulariser 25 % of the total loss at a classification loss of 6.9
    lam = B.lasso_set_coeff(6.9, got, 0.25)
    assert abs(lam * got / (6.9 + lam * got) - 0.25) < 1e-12


@pytest.mark.parametrize("pixels,C,pad", [(4 * 16 * 16, 16, False), (3 * 7 * 7, 203, True), (1000, 64, True),
                                          (129, 811, True), (50, 5, False), (1, 8, False), (70000, 72, True)])
def test_scatter_nhwc_bit_exact_and_inverts_the_gather(pixels, C, pad):
    from gpu_util import DEV, pitch8
    rng = np.random.Generator(np.random.PCG64(5000 + pixels + C))
    idx = np.sort(rng.choice(C, max(1, int(C * 0.6)), replace=False)).astype(np.int32)
    Cp = idx.size
    x = rng.integers(1, 65536, size=(pixels, Cp)).astype(np.uint16)
    xp = pitch8(Cp) if pad else Cp
    op = pitch8(C) if pad else C
    xfull = np.full((pixels, xp), 0xDEAD, dtype=np.uint16)
    xfull[:, :Cp] = x
    xd = torch.from_numpy(xfull.view(np.int16)).to(DEV).view(torch.bfloat16)
    idd = torch.from_numpy(idx).to(DEV)
    out = torch.empty((pixels, op), dtype=torch.bfloat16, device=DEV)
    out.view(torch.int16).fill_(0x1234)
    B.scatter_nhwc(xd, pixels, Cp, xp, idd, C, out, op)
    back = torch.empty((pixels, xp), dtype=torch.bfloat16, device=DEV)
    back.view(torch.int16).fill_(0x4321)
    B.compact_nhwc(out, pixels, C, op, idd, Cp, back, xp)
    torch.cuda.synchronize()
    got = out.view(torch.int16).cpu().numpy().view(np.uint16)
    assert np.array_equal(got[:, :C], oracle.scatter_nhwc(x, idx, C))
    assert np.all(got[:, C:] == 0x1234)                                     # pitch padding untouched
    assert np.array_equal(back.view(torch.int16).cpu().numpy().view(np.uint16)[:, :Cp], x)


@pytest.mark.parametrize("shape,pad", [((16, 3, 3, 16), False), ((40, 1, 1, 203), True), ((7, 7, 7, 3), False),
                                       ((300, 3, 3, 37), True), ((5, 1, 1, 2048), False)])
def test_group_maxabs_is_exact(shape, pad):
    from gpu_util import DEV, dev_f32, pitch8
    rng = np.random.Generator(np.random.PCG64(6000 + sum(shape)))
    w = rng.standard_normal(shape).astype(np.float32)
    w[1] = 0.0
    w[..., 0] = 0.0
    K, C = shape[0], shape[-1]
    RS = shape[1] * shape[2]
    pitch = pitch8(C) if pad else C
    wd = dev_f32(w, pitch)                      # padding is NaN: it must not enter the maxima
    om = torch.full((K,), float("nan"), device=DEV)
    im = torch.full((C,), float("nan"), device=DEV)
    B.group_maxabs(wd, K, RS, C, pitch, om, im)
    torch.cuda.synchronize()
    rom, rim = oracle.group_maxabs(w)
    assert np.array_equal(om.cpu().numpy(), rom.astype(np.float32))          # fp32 maxima of fp32 data: exact
    assert np.array_equal(im.cpu().numpy(), rim.astype(np.float32))
    z = torch.zeros(K, dtype=torch.uint8, device=DEV)
    B.zero_groups(om, K, 1e-4, z)
    torch.cuda.synchronize()
    assert np.array_equal(z.cpu().numpy(), oracle.zero_groups(rom, 1e-4))


def test_apply_zero_bit_exact():
    from gpu_util import DEV, dev_f32, pitch8
    rng = np.random.Generator(np.random.PCG64(7001))
    for shape, pad in (((12, 3, 3, 10), True), ((5, 1, 1, 64), False), ((33, 2, 2, 7), False)):
        w = rng.standard_normal(shape).astype(np.float32)
        K, C = shape[0], shape[-1]
        RS = shape[1] * shape[2]
        zo = (rng.random(K) < 0.3).astype(np.uint8)
        zi = (rng.random(C) < 0.3).astype(np.uint8)
        pitch = pitch8(C) if pad else C
        for mo, mi in ((zo, zi), (None, zi), (zo, None)):
            wd = dev_f32(w, pitch)
            B.apply_zero(wd, K, RS, C, pitch, None if mo is None else torch.from_numpy(mo).to(DEV),
                         None if mi is None else torch.from_numpy(mi).to(DEV))
            torch.cuda.synchronize()
            got = wd.cpu().numpy()
            assert np.array_equal(got[..., :C], oracle.apply_zero(w, mo, mi).astype(np.float32))
            if pitch != C:
                assert np.isnan(got[..., C:]).all()                            # padding untouched


@pytest.mark.parametrize("n", [2, 11])
def test_optimizer_step_of_many_layers_equals_the_layers_one_by_one(n):
    """A launch of more than 256 MB of w, dw and mom takes a form of its own: bit for bit what calls of one layer (26 MB)
    leave, padding untouched (rows that end inside a vector included)."""
    from gpu_util import DEV
    K, RS, lam, lr, mu, wd = 650, 9, 1e-3, 0.1, 0.9, 1e-4
    calls = {}
    for single in (True, False):
        jobs = calls.setdefault(single, ([], []))
        gen = torch.Generator(device=DEV).manual_seed(n)
        for i in range(n):
            C, pitch = 369 + i, 376 if i < 8 else 384
            t = [torch.randn((K, RS, pitch), device=DEV, generator=gen) for _ in range(3)]
            for x in t:
                x[..., C:] = 7.0
            norms = [torch.rand(k, device=DEV, generator=gen) + 0.5 for k in (K, C)]
            jobs[0].append((t, norms))
            jobs[1].append(B.layer_update(*t, *norms, K, RS, C, pitch, 3))
        for part in [[j] for j in jobs[1]] if single else [jobs[1]]:
            B.sgd_momentum_lasso_batched(part, lam, lr, mu, wd)
    torch.cuda.synchronize()
    for (one, _), (many, _) in zip(calls[True][0], calls[False][0]):
        assert all(torch.equal(a, b) for a, b in zip(one, many))


def test_optimizer_step_matches_oracle():
    """One launch updates several layers (vector and element-wise loaders, padded pitches, first-layer
    exemption): weights and momentum against the fp64 oracle at 1e-5; dw and pitch padding untouched; a second
    step from the device's own state also matches (momentum carries over)."""
    from gpu_util import DEV, F32_TOL, dev_f32, pitch8, rel_err
    rng = np.random.Generator(np.random.PCG64(8100))
    shapes = [((16, 3, 3, 3), False, 1), ((40, 1, 1, 203), True, 3), ((64, 3, 3, 64), True, 3), ((7, 5, 5, 11), False, 3),
              ((300, 1, 1, 37), True, 2)]
    lam, lr, mu, wd = 1e-3, 0.1, 0.9, 1e-4
    state = []
    for shape, pad, flags in shapes:
        K, C = shape[0], shape[-1]
        RS = shape[1] * shape[2]
        w = (rng.standard_normal(shape) * 0.1).astype(np.float32)
        w[0] = 0.0                                   # an exactly zero filter
        dw = (rng.standard_normal(shape) * 0.01).astype(np.float32)
        dw[0] = 0.0
        m = (rng.standard_normal(shape) * 0.01).astype(np.float32)
        m[0] = 0.0
        pitch = pitch8(C) if pad else C
        wd_, on, inn, _ = _norms_gpu(w, pitch if pad else None, shadow=False)
        state.append(dict(shape=shape, K=K, RS=RS, C=C, pitch=pitch, flags=flags, w=w, dw=dw, m=m,
                          wd=wd_, dwd=dev_f32(dw, pitch), md=dev_f32(m, pitch), on=on, inn=inn))
    for step in range(2):
        jobs = [B.layer_update(s["wd"], s["dwd"], s["md"], s["on"], s["inn"], s["K"], s["RS"], s["C"], s["pitch"],
                               s["flags"]) for s in state]
        B.sgd_momentum_lasso_batched(jobs, lam, lr, mu, wd)
        torch.cuda.synchronize()
        for s in state:
            on64, in64 = oracle.group_norms(s["w"])
            w_ref, m_ref = oracle.sgd_momentum_lasso(s["w"], s["dw"], s["m"], on64, in64, lam, lr, mu, wd, s["flags"])
            gw, gm = s["wd"].cpu().numpy(), s["md"].cpu().numpy()
            C = s["C"]
            assert rel_err(gw[..., :C], w_ref) <= F32_TOL and rel_err(gm[..., :C], m_ref) <= F32_TOL, s["shape"]
            assert not gw[0, ..., :C].any() and not gm[0, ..., :C].any()          # the zero filter stays exactly zero
            assert np.array_equal(s["dwd"].cpu().numpy()[..., :C], s["dw"])       # the loss gradient is read-only
            if s["pitch"] != C:
                assert np.isnan(gw[..., C:]).all() and np.isnan(gm[..., C:]).all()
            # next step starts from the device's fp32 state and fresh norms of it
            s["w"], s["m"] = gw[..., :C].copy(), gm[..., :C].copy()
            ws = workspace_for(s)
            B.group_norms(s["wd"], s["K"], s["RS"], C, s["pitch"], s["on"], s["inn"], None, ws)
        torch.cuda.synchronize()


def workspace_for(s):
    from gpu_util import workspace
    return workspace(B.group_norms_workspace_bytes(s["K"], s["RS"], s["C"]))


def test_norms_with_zero_masks_in_one_call():
    """pt_group_norms_detect_batched: norms bit-identical to pt_group_norms_batched's, masks bit-identical to
    pt_zero_groups on those norms and to the oracle's (groups are exactly zero or far above the threshold), at
    several thresholds including the ones that mark nothing."""
    from gpu_util import DEV, dev_f32, pitch8
    rng = np.random.Generator(np.random.PCG64(77))
    shapes = [(64, 3, 3, 64), (203, 1, 1, 811), (37, 3, 3, 51), (655, 1, 1, 207), (16, 7, 7, 3), (64, 3, 3, 37)]
    host, devs = [], []
    for i, sh in enumerate(shapes):
        w = rng.standard_normal(sh, dtype=np.float32) * np.float32(0.05)
        K, C = sh[0], sh[-1]
        zo = rng.choice(K, max(1, K // 3), replace=False)
        zi = rng.choice(C, max(1, C // 4), replace=False)
        w = wl.zero_groups_in_weights(w, zo, zi)
        pitch = C if i == len(shapes) - 1 else pitch8(C)          # the last layer is stored unaligned
        t = dict(w=dev_f32(w, pitch), K=K, RS=sh[1] * sh[2], C=C, pitch=pitch)
        for name, n, dt in (("on", K, torch.float32), ("inn", C, torch.float32), ("on2", K, torch.float32),
                            ("inn2", C, torch.float32), ("zo", K, torch.uint8), ("zi", C, torch.uint8),
                            ("zo2", K, torch.uint8), ("zi2", C, torch.uint8)):
            t[name] = torch.full((n,), 7, dtype=dt, device=DEV)
        host.append(w)
        devs.append(t)
    jobs_d = [B.layer_detect(t["w"], t["K"], t["RS"], t["C"], t["pitch"], t["on"], t["inn"], t["zo"], t["zi"]) for t in devs]
    jobs_n = [B.layer_weights(t["w"], t["K"], t["RS"], t["C"], t["pitch"], t["on2"], t["inn2"], None) for t in devs]
    ws = torch.empty(B.group_norms_detect_batched_workspace_bytes(jobs_d), dtype=torch.uint8, device=DEV)
    assert ws.numel() == B.group_norms_batched_workspace_bytes(jobs_n)
    B.group_norms_batched(jobs_n, ws)
    for thr in (1e-6, 1e-4, 0.0, -1.0, 1e9):
        B.group_norms_detect_batched(jobs_d, thr, ws)
        for t in devs:
            B.zero_groups(t["on2"], t["K"], thr, t["zo2"])
            B.zero_groups(t["inn2"], t["C"], thr, t["zi2"])
        torch.cuda.synchronize()
        for w, t in zip(host, devs):
            assert torch.equal(t["on"], t["on2"]) and torch.equal(t["inn"], t["inn2"])
            assert torch.equal(t["zo"], t["zo2"]) and torch.equal(t["zi"], t["zi2"])
            ron, rin = oracle.group_norms(w)
            assert np.array_equal(t["zo"].cpu().numpy(), oracle.zero_groups(ron.astype(np.float32), thr))
            assert np.array_equal(t["zi"].cpu().numpy(), oracle.zero_groups(rin.astype(np.float32), thr))
            if 0.0 < thr < 1.0:
                assert int(t["zo"].sum()) == max(1, t["K"] // 3) and int(t["zi"].sum()) == max(1, t["C"] // 4)


@pytest.mark.parametrize("C,keep_n", [(8, 1), (37, 7), (64, 8), (65, 9), (260, 255), (2048, 2047), (2048, 2048), (40, 0)])
def test_planned_compaction_reads_the_counts_on_the_device(C, keep_n):
    """All three kinds of gather with the counts left on the device by the plan: equal to plain indexing, nothing beyond
    the counted part written (a count of 0 writes nothing at all)."""
    from gpu_util import DEV
    rng = np.random.Generator(np.random.PCG64(C * 7 + keep_n))
    kept = np.sort(rng.permutation(C)[:keep_n]).astype(np.int32)
    idx = torch.full((C,), 0, dtype=torch.int32, device=DEV)
    idx[:keep_n] = torch.from_numpy(kept).to(DEV)
    n_dev = torch.tensor([keep_n], dtype=torch.int32, device=DEV)
    pixels, RS, K, pitch, op = 133, 3, C, (C + 7) // 8 * 8, (keep_n + 7) // 8 * 8
    x = torch.randn((pixels, pitch), device=DEV).to(torch.bfloat16)
    w = torch.randn((K, RS, pitch), device=DEV)
    v = torch.randint(0, 255, (K,), dtype=torch.uint8, device=DEV)
    xo, wo, w1 = torch.full_like(x, 3.0), torch.full_like(w, 3.0), torch.full_like(w, 3.0)
    vo = torch.full_like(v, 7)
    B.compact_planned([B.planned_nhwc(x, pixels, C, pitch, idx, n_dev, xo),
                       B.planned_weights(w, K, RS, C, pitch, idx, n_dev, idx, n_dev, wo),
                       B.planned_weights(w, K, RS, C, pitch, None, None, idx, n_dev, w1),
                       B.planned_vector(v, 1, K, idx, n_dev, vo)])
    torch.cuda.synchronize()
    sel = idx[:keep_n].long()
    got = xo.view(-1)[: pixels * op].view(pixels, op)
    assert torch.equal(got[:, :keep_n], x[:, sel]) and not got[:, keep_n:].any()
    assert (xo.view(-1)[pixels * op:] == 3.0).all()
    for out, src in ((wo, w[sel]), (w1, w)):
        n = src.shape[0] * RS * op
        assert torch.equal(out.view(-1)[:n].view(src.shape[0], RS, op)[..., :keep_n], src[..., sel])
        assert (out.view(-1)[n:] == 3.0).all()
    assert torch.equal(vo[:keep_n], v[sel]) and (vo[keep_n:] == 7).all()


@pytest.mark.parametrize("sizes", [[(1, 40), (40000, 264), (1, 8), (7, 2048), (9, 2048), (3000, 2048), (2, 16), (20000, 104)],
                                   [(100, 1000 + 8 * i) for i in range(60)]])
def test_activation_gather_over_many_tensors(sizes):
    """Runs of a launch's tensors are handed out with a fixed stride: a workgroup's next run may lie several tensors on,
    or in a tensor of less than one run (8 rows of 4 KB, an odd count of them, a single row)."""
    from gpu_util import DEV
    jobs, want = [], []
    for i, (pixels, C) in enumerate(sizes):
        gen = np.random.Generator(np.random.PCG64(i))
        n = max(1, C * 2 // 3)
        idx = torch.from_numpy(np.sort(gen.choice(C, n, replace=False)).astype(np.int32)).to(DEV)
        x = torch.randint(-32768, 32767, (pixels, C), dtype=torch.int16, device=DEV)
        out = torch.full((pixels, (n + 7) // 8 * 8 + 8), 7, dtype=torch.int16, device=DEV)
        cnt = torch.tensor([n], dtype=torch.int32, device=DEV)
        jobs.append(B.planned_nhwc(x.view(torch.bfloat16), pixels, C, C, idx, cnt, out.view(torch.bfloat16)))
        want.append((x, idx, out, n, cnt))
    B.compact_planned(jobs)
    torch.cuda.synchronize()
    for x, idx, out, n, _ in want:
        op, pixels = (n + 7) // 8 * 8, x.shape[0]
        got = out.view(-1)[: pixels * op].view(pixels, op)
        assert torch.equal(got[:, :n], x[:, idx.long()]) and not got[:, n:].any()
        assert (out.view(-1)[pixels * op:] == 7).all()


@pytest.mark.parametrize("n", range(9, 17))
@pytest.mark.parametrize("C,pixels", [(16, 1024 * 512 * 5 + 1), (1000, 17)])
def test_activation_gather_last_vector_and_many_runs(C, pixels, n):
    """One to eight channels in the last vector of a row; five runs a workgroup and one row more, and two runs in all."""
    from gpu_util import DEV
    idx = torch.from_numpy(np.sort(np.random.Generator(np.random.PCG64(n)).choice(C, n, replace=False)).astype(np.int32)).to(DEV)
    x = torch.randint(-32768, 32767, (pixels, (C + 7) // 8 * 8), dtype=torch.int16, device=DEV)
    out = torch.full((pixels + 1, 16), 7, dtype=torch.int16, device=DEV)
    B.compact_nhwc(x.view(torch.bfloat16), pixels, C, x.shape[1], idx, n, out.view(torch.bfloat16), 16)
    torch.cuda.synchronize()
    assert torch.equal(out[:pixels, :n], x[:, idx.long()]) and not out[:pixels, n:].any() and (out[pixels] == 7).all()


@pytest.mark.parametrize("runs", [768, 769, 1024, 1025])
@pytest.mark.parametrize("tensors", [1, 6, 7])
def test_activation_gather_of_about_two_runs_a_workgroup(runs, tensors):
    """Either side of the lines between which a workgroup reads both of its runs ahead of the first store: runs of 256 pixels of
    64 channels, the last one of a tensor a pixel short."""
    from gpu_util import DEV
    C, n = 64, 45
    share = [runs // tensors + (i < runs % tensors) for i in range(tensors)]
    idx = torch.from_numpy(np.sort(np.random.Generator(np.random.PCG64(runs)).choice(C, n, replace=False)).astype(np.int32)).to(DEV)
    xs = [torch.randint(-32768, 32767, (256 * r - 1, C), dtype=torch.int16, device=DEV) for r in share]
    outs = [torch.full((x.shape[0] + 1, 48), 7, dtype=torch.int16, device=DEV) for x in xs]
    B.compact_nhwc_batched([B.gather_nhwc(x.view(torch.bfloat16), x.shape[0], C, C, idx, n, o.view(torch.bfloat16), 48) for x, o in zip(xs, outs)])
    torch.cuda.synchronize()
    for x, o in zip(xs, outs):
        assert torch.equal(o[:-1, :n], x[:, idx.long()]) and not o[:-1, n:].any() and (o[-1] == 7).all()


@pytest.mark.parametrize("n_counts,zero_at", [(1, 0), (1, None), (64, 63), (65, 64), (130, 127), (130, None), (0, None)])
def test_guarded_compaction_writes_all_or_nothing(n_counts, zero_at):
    """One count of 0 anywhere (before, at and past the 64 that one load covers) keeps all three kinds of gather from
    writing; with none the call is the plain one."""
    from gpu_util import DEV
    C, RS, pixels = 72, 3, 700           # several runs of the streaming gather
    idx = torch.arange(0, C, 2, dtype=torch.int32, device=DEV)
    n_dev = torch.tensor([idx.numel()], dtype=torch.int32, device=DEV)
    counts = torch.full((n_counts,), 5, dtype=torch.int32, device=DEV)
    if zero_at is not None:
        counts[zero_at] = 0
    x = torch.randn((pixels, C), device=DEV).to(torch.bfloat16)
    w, v = torch.randn((C, RS, C), device=DEV), torch.randn(C, device=DEV)
    src = (x, w, v)

    def outputs(run):
        out = [torch.full_like(t, 3.0) for t in src]
        run([B.planned_nhwc(x, pixels, C, C, idx, n_dev, out[0]), B.planned_weights(w, C, RS, C, C, idx, n_dev, idx, n_dev, out[1]),
             B.planned_vector(v, 4, C, idx, n_dev, out[2])])
        torch.cuda.synchronize()
        return out
    plain = outputs(B.compact_planned)
    guarded = outputs(lambda jobs: B.compact_planned_guarded(jobs, counts))
    for a, b in zip(plain, guarded):
        assert not (a == 3.0).all()
        assert (b == 3.0).all() if zero_at is not None else torch.equal(a, b)


def test_sweep_refused_for_an_empty_edge_leaves_the_outputs():
    """An edge all of whose groups are zero: the sweep raises, and no compacted tensor has been touched."""
    from paper_1901_09290_amd import harness as hz
    specs = [wl.ConvSpec("s0", 2, 8, 8, 3, 24, 3, 3, 1, 1, None, 0, first=True), wl.ConvSpec("s1", 2, 8, 8, 24, 40, 1, 1, 1, 0, 0, 1),
             wl.ConvSpec("s2", 2, 8, 8, 40, 16, 1, 1, 1, 0, 1, None)]
    edges = [wl.Edge("e0", 24, [0], [1]), wl.Edge("e1", 40, [1], [2])]
    rng = np.random.Generator(np.random.PCG64(3))
    weights = wl.network_weights(specs, edges, [np.arange(5, dtype=np.int32), np.arange(40, dtype=np.int32)], rng)
    m = hz.ReconfigModel(specs, edges, weights, seed=4)
    outs = m.w_out + m.mom_out + m.act_out + [v for vs in m.bn_out for v in vs]
    for t in outs:
        t.fill_(3.0)
    with pytest.raises(B.PruneTrainError) as e:
        m.sweep(1e-6)
    torch.cuda.synchronize()
    assert e.value.status == -2 and m.new_counts.tolist() == [19, 0]
    assert all((t == 3.0).all() for t in outs)


@pytest.mark.parametrize("shape", [(64, 4, 4, 16), (205, 5, 1, 16), (114, 3, 3, 16), (4096, 1, 1, 4), (511, 2, 1, 5), (1, 1, 1, 1),
                                   (32, 1, 1, 256), (33, 1, 1, 256), (4, 2, 2, 2048), (700, 3, 3, 200)])
def test_norms_of_a_layer_by_itself(shape):
    """One chunk (norms finished by the workgroup that reads the layer), one row more, and many chunks: against the oracle, and
    bit for bit the same however often they are taken."""
    from gpu_util import F32_TOL, pitch8, rel_err
    w = np.random.Generator(np.random.PCG64(sum(shape))).standard_normal(shape, dtype=np.float32) * np.float32(0.05)
    w[0] = 0.0
    pitch = pitch8(shape[-1])
    _, on, inn, _ = _norms_gpu(w, pitch, shadow=True)
    ron, rin = oracle.group_norms(w)
    assert rel_err(on.cpu().numpy(), ron) <= F32_TOL and rel_err(inn.cpu().numpy(), rin) <= F32_TOL and on[0].item() == 0.0
    _, on2, inn2, _ = _norms_gpu(w, pitch)
    assert torch.equal(on, on2) and torch.equal(inn, inn2)


@pytest.mark.parametrize("shape", [(513, 1, 1, 16), (4096, 1, 1, 16), (4097, 1, 1, 16), (128, 1, 1, 300), (129, 1, 1, 300),
                                   (17, 1, 1, 300), (33, 1, 1, 300), (8, 1, 1, 2048), (9, 1, 1, 2048)])
def test_norms_around_the_sizes_where_the_chunks_change(shape):
    """Chunks of one batch of rows up to eight batches, of two batches beyond: by itself and in a call of several layers,
    against the oracle and each other."""
    from gpu_util import DEV, F32_TOL, rel_err, workspace
    K, R, S, C = shape
    w = np.random.Generator(np.random.PCG64(K + C)).standard_normal(shape, dtype=np.float32)
    pitch = (C + 7) // 8 * 8
    wd, on, inn, _ = _norms_gpu(w, pitch, shadow=True)
    ron, rin = oracle.group_norms(w)
    assert rel_err(on.cpu().numpy(), ron) <= F32_TOL and rel_err(inn.cpu().numpy(), rin) <= F32_TOL
    on2, inn2 = (torch.zeros((3, k), device=DEV) for k in (K, C))
    layers = [B.layer_weights(wd, K, R * S, C, pitch, on2[i], inn2[i], None) for i in range(3)]
    B.group_norms_batched(layers, workspace(B.group_norms_batched_workspace_bytes(layers)))
    torch.cuda.synchronize()
    for i in range(3):
        assert rel_err(on2[i].cpu().numpy(), ron) <= F32_TOL and rel_err(inn2[i].cpu().numpy(), rin) <= F32_TOL
        assert torch.equal(on2[i], on2[0]) and torch.equal(inn2[i], inn2[0])


@pytest.mark.parametrize("shape,pitch", [((64, 3, 3, 16), 16), ((205, 5, 1, 16), 16), ((114, 3, 3, 16), 16), ((32, 3, 3, 61), 64),
                                         ((33, 1, 1, 256), 256), ((8, 1, 1, 2047), 2048), ((129, 1, 1, 300), 304),
                                         ((64, 3, 3, 128), 128), ((40, 3, 3, 21), 21)])
def test_norms_of_one_layer_are_bit_for_bit_those_of_the_batched_call(shape, pitch):
    """One to two chunks (one launch when the layer is by itself), more, and unaligned rows: norms taken alone, in a call of
    three layers and by detection are the same bits, so a group at the threshold is zero by every route or by none."""
    from gpu_util import DEV, workspace
    K, R, S, C = shape
    RS = R * S
    w = np.random.Generator(np.random.PCG64(K * C)).standard_normal(shape, dtype=np.float32)
    wd, on, inn, _ = _norms_gpu(w, pitch)
    on3, inn3 = (torch.zeros((3, k), device=DEV) for k in (K, C))
    layers = [B.layer_weights(wd, K, RS, C, pitch, on3[i], inn3[i], None) for i in range(3)]
    B.group_norms_batched(layers, workspace(B.group_norms_batched_workspace_bytes(layers)))
    torch.cuda.synchronize()
    for i in range(3):
        assert torch.equal(on3[i], on) and torch.equal(inn3[i], inn)
    for thr in (float(on[K // 2]), float(inn[C // 2])):
        for n in (1, 2):
            on2, inn2 = (torch.zeros((n, k), device=DEV) for k in (K, C))
            zo, zi = (torch.full((n, k), 7, dtype=torch.uint8, device=DEV) for k in (K, C))
            jobs = [B.layer_detect(wd, K, RS, C, pitch, on2[i], inn2[i], zo[i], zi[i]) for i in range(n)]
            B.group_norms_detect_batched(jobs, thr, workspace(B.group_norms_detect_batched_workspace_bytes(jobs)))
            torch.cuda.synchronize()
            for i in range(n):
                assert torch.equal(on2[i], on) and torch.equal(inn2[i], inn)
                assert torch.equal(zo[i], (on < thr).to(torch.uint8)) and torch.equal(zi[i], (inn < thr).to(torch.uint8))


def test_first_optimizer_step_inside_a_graph():
    """A network whose first optimizer step is captured: every replay carries the momentum on, as eager steps do."""
    from gpu_util import DEV
    from paper_1901_09290_amd import harness as hz
    specs, _ = wl.resnet32_layers(2, 8)
    nets = [hz.Network(hz.build_network(specs[:5], seed=3)) for _ in range(2)]
    gen = torch.Generator(device=DEV)
    gen.manual_seed(4)
    for l, m in zip(*(n.layers for n in nets)):
        l.dw.normal_(generator=gen)
        m.dw.copy_(l.dw)
        l.out_norm.fill_(1.0), l.in_norm.fill_(1.0), m.out_norm.fill_(1.0), m.in_norm.fill_(1.0)
    step = lambda net: net.optimizer_step(1e-4, 0.1, 0.9, 1e-4)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step(nets[1])
    for i in range(4):
        step(nets[0])
        graph.replay()
        torch.cuda.synchronize()
        for l, m, a, b in zip(nets[0].layers, nets[1].layers, nets[0].mom, nets[1].mom):
            assert torch.equal(l.w_master, m.w_master) and torch.equal(a, b), i


@pytest.mark.parametrize("C,total", [(300, 2 << 20), (300, 3 << 20), (300, 6 << 20), (300, 12 << 20), (2045, 3 << 20), (5, 1 << 20)])
def test_optimizer_step_for_every_chunk_size(C, total):
    """One layer in chunks of 1 K to 16 K elements by its size: against the plain update in float64 at the tolerance of the
    oracle's test, dw untouched."""
    from gpu_util import DEV, F32_TOL
    RS, lam, lr, mu, wd = 3, 1e-3, 0.1, 0.9, 1e-4
    pitch = (C + 7) // 8 * 8
    K = total // (RS * pitch) + 1
    gen = torch.Generator(device=DEV).manual_seed(C)
    w, dw, mom = (torch.randn((K, RS, pitch), device=DEV, generator=gen) for _ in range(3))
    on, inn = (torch.rand(k, device=DEV, generator=gen) + 0.5 for k in (K, C))
    W, G, M = (t[..., :C].double() for t in (w, dw, mom))
    dw0 = dw.clone()
    M = mu * M + G + wd * W + lam * W * (1.0 / on.double()[:, None, None] + 1.0 / inn.double())
    W = W - lr * M
    B.sgd_momentum_lasso_batched([B.layer_update(w, dw, mom, on, inn, K, RS, C, pitch, 3)], lam, lr, mu, wd)
    torch.cuda.synchronize()
    for got, ref in ((w, W), (mom, M)):
        assert ((got[..., :C].double() - ref).norm() / ref.norm()).item() <= F32_TOL
    assert torch.equal(dw, dw0)


@pytest.mark.parametrize("total", [41 << 19, 43 << 19])
def test_optimizer_step_of_the_largest_chunks(total):
    """21.5 M elements, the most that chunks of 16 K take, and 22.5 M, in chunks of 32 K that pass by the caches."""
    test_optimizer_step_for_every_chunk_size(300, total)


@pytest.mark.parametrize("C,total", [(300, 1 << 20), (300, 3 << 20), (300, 6 << 20), (300, 12 << 20), (300, 21 << 20), (2045, 3 << 20),
                                     (5, 1 << 20)])
@pytest.mark.parametrize("n", [1, 2])
def test_gradient_for_every_chunk_size(C, total, n):
    """A layer by itself and two in one call, in chunks of 1 K to 16 K elements by their size: against the plain sum in
    float64 at the tolerance of the oracle's test."""
    from gpu_util import DEV, F32_TOL
    RS, lam = 3, 0.5
    pitch = (C + 7) // 8 * 8
    K = total // (RS * pitch * n) + 1
    gen = torch.Generator(device=DEV).manual_seed(C + n)
    w, dw = (torch.randn((n, K, RS, pitch), device=DEV, generator=gen) for _ in range(2))
    on, inn = (torch.rand((n, k), device=DEV, generator=gen) + 0.5 for k in (K, C))
    ref = dw[..., :C].double() + lam * w[..., :C].double() * (1.0 / on.double()[:, :, None, None] + 1.0 / inn.double()[:, None, None, :])
    pad = dw[..., C:].clone()
    if n == 1:
        B.group_lasso_grad(w, on, inn, lam, 3, dw, K, RS, C, pitch)
    else:
        B.group_lasso_grad_batched([B.layer_lasso(w[i], on[i], inn[i], dw[i], K, RS, C, pitch, 3) for i in range(n)], lam)
    torch.cuda.synchronize()
    assert ((dw[..., :C].double() - ref).norm() / ref.norm()).item() <= F32_TOL
    assert torch.equal(dw[..., C:], pad)
