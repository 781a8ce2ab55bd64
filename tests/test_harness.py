"""Host side of the harness without a GPU: tensors live in host memory, streams and events are stand-ins, and every
library call that would launch something is recorded instead.  Queries (workspaces, plans) go to the real library."""
import contextlib
import ctypes as C

import numpy as np
import pytest
import torch

from paper_1901_09290_amd import binding as B
from paper_1901_09290_amd import harness as hz
from paper_1901_09290_amd import workloads as wl


def _pointers(v, out):
    """Every address in a call's argument: plain integers, void pointers, fields of structures, elements of arrays."""
    if isinstance(v, (int, C.c_void_p)):
        out.append(v if isinstance(v, int) else v.value)
    elif isinstance(v, C.Array):
        for e in v:
            _pointers(e, out)
    elif isinstance(v, C.Structure):
        for name, typ in v._fields_:
            if typ is C.c_void_p:
                out.append(getattr(v, name))


class _Recorder:
    """Stands in for the loaded library: launching calls are noted as (name, addresses) and answered by `status`."""

    def __init__(self, real):
        self.real, self.calls, self.status = real, [], lambda name, args: 0

    def __getattr__(self, name):
        if name.endswith("_bytes") or name.endswith("_plan") and name != "pt_compact_plan" or name.startswith("pt_last"):
            return getattr(self.real, name)

        def call(*args):
            seen = []
            for a in args:
                _pointers(a, seen)
            self.calls.append((name, seen))
            return self.status(name, args)
        return call

    def seen(self, prefix=""):
        return {p for name, ps in self.calls if name.startswith(prefix) for p in ps}


class _Stream:
    cuda_stream = 0

    def wait_stream(self, other):
        pass

    def wait_event(self, event):
        pass


class _Event:
    def record(self, stream=None):
        pass

    def synchronize(self):
        pass


@pytest.fixture
def recorded(monkeypatch):
    rec = _Recorder(B.lib())
    monkeypatch.setattr(B, "lib", lambda: rec)
    monkeypatch.setattr(B, "_raw_stream", lambda: 0)
    monkeypatch.setattr(hz, "DEV", "cpu")
    main = _Stream()
    monkeypatch.setattr(torch.cuda, "Stream", _Stream)
    monkeypatch.setattr(torch.cuda, "Event", _Event)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: main)
    monkeypatch.setattr(torch.cuda, "stream", lambda s: contextlib.nullcontext())
    return rec


def residual_block(N=2):
    """A first layer, a residual block with a shortcut convolution and a strided layer behind it."""
    return [
        wl.ConvSpec("first", N, 16, 16, 3, 24, 3, 3, 1, 1, None, 0, first=True),
        wl.ConvSpec("b_a", N, 16, 16, 24, 16, 1, 1, 1, 0, 0, 1),
        wl.ConvSpec("b_b", N, 16, 16, 16, 16, 3, 3, 1, 1, 1, 2),
        wl.ConvSpec("b_c", N, 16, 16, 16, 40, 1, 1, 1, 0, 2, 3),
        wl.ConvSpec("b_proj", N, 16, 16, 24, 40, 1, 1, 1, 0, 0, 3),
        wl.ConvSpec("last", N, 16, 16, 40, 33, 3, 3, 2, 1, 3, None),
    ]


TENSORS = ("x", "dy", "w_master", "w_bf16", "w_crsk", "y", "dx", "dw", "out_norm", "in_norm")


@pytest.mark.parametrize("grouped", [True, False])
@pytest.mark.parametrize("overlap,fuse", [(True, True), (True, False), (False, False)])
def test_network_reads_the_layers_tensors_at_every_call(recorded, monkeypatch, grouped, overlap, fuse):
    """Every tensor of every layer is replaced between two iterations: the second one must hand the library the new
    tensors and none of the old ones, whose memory may belong to something else by then."""
    if not grouped:
        monkeypatch.setattr(hz, "WGRAD_GROUP_MAX_BYTES", 0)
    net = hz.Network(hz.build_network(residual_block(), seed=1))
    assert net.fork == {1: 4} and net.grouped == grouped and len(net.groups) == (3 if grouped else 6)
    net.overlap_wgrad, net.fuse_lasso = overlap, fuse

    def iteration():
        net.train_step(1e-3)
        net.regulariser_value()
        net.optimizer_step(1e-3, 0.1, 0.9, 0.0)

    iteration()
    old = {(i, a): getattr(l, a) for i, l in enumerate(net.layers) for a in TENSORS}
    assert {t.data_ptr() for t in old.values() if t is not None} <= recorded.seen()
    for (i, a), t in old.items():
        if t is not None:
            setattr(net.layers[i], a, t.clone())
    net.layers[1].lasso_flags = 0
    recorded.calls.clear()
    iteration()
    seen = recorded.seen()
    assert not {k for k, t in old.items() if t is not None and t.data_ptr() in seen}
    assert {getattr(net.layers[i], a).data_ptr() for (i, a), t in old.items() if t is not None} <= seen
    if overlap:
        assert [j.flags for j in net.wgrad_jobs] == [l.lasso_flags for l in reversed(net.layers)]


def test_network_enlarges_a_weight_gradient_workspace(recorded):
    """A tensor may be replaced by one that is aligned worse and whose plan needs more partial sums: the call's refusal
    for want of workspace is answered with a larger one, any other status is passed on."""
    net = hz.Network(hz.build_network(residual_block(), seed=1))
    sizes = [w.numel() for w in net.ws_sides]
    refused = []

    def status(name, args):
        if name == "pt_conv_bwd_weight_batched" and not refused:
            refused.append(args[5])
            return B.ERR_WORKSPACE
        return 0
    recorded.status = status
    net.train_step(1e-3)
    calls = [ps for name, ps in recorded.calls if name == "pt_conv_bwd_weight_batched"]
    assert refused == sizes and len(calls) == len(net.groups) + 1
    recorded.status = lambda name, args: B.ERR_UNSUPPORTED if name == "pt_conv_bwd_weight_batched" else 0
    with pytest.raises(B.PruneTrainError) as e:
        net.train_step(1e-3)
    assert e.value.status == B.ERR_UNSUPPORTED


def _reconfig_model(with_activations=True):
    specs = [
        wl.ConvSpec("m0", 1, 6, 6, 3, 30, 3, 3, 1, 1, None, 0, first=True),
        wl.ConvSpec("m1", 1, 6, 6, 30, 37, 1, 1, 1, 0, 0, 1),
        wl.ConvSpec("m2", 1, 6, 6, 37, 30, 3, 3, 1, 1, 1, 0),
        wl.ConvSpec("m3", 1, 6, 6, 30, 9, 1, 1, 1, 0, 0, None),
    ]
    edges = [wl.Edge("e0", 30, [0, 2], [1, 3]), wl.Edge("e1", 37, [1], [2])]
    rng = np.random.Generator(np.random.PCG64(5))
    weights = wl.network_weights(specs, edges, wl.zeroed_channel_sets(edges, 0.3, rng), rng)
    model = hz.ReconfigModel(specs, edges, weights, seed=2, with_activations=with_activations)
    model.counts.copy_(torch.tensor([20, 25], dtype=torch.int32))   # as the recorded plan would leave them
    return model


@pytest.mark.parametrize("with_activations", [True, False])
def test_compaction_reads_the_models_tensors_at_every_call(recorded, monkeypatch, with_activations):
    """The gathers of compact() after every tensor was replaced (some behind the same tensor object): job by job what the
    calls for single jobs make of the tensors the model holds now."""
    zeros = torch.zeros
    monkeypatch.setattr(torch, "zeros", lambda *a, pin_memory=False, **kw: zeros(*a, **kw))
    m = _reconfig_model(with_activations)
    tables = []

    def status(name, args):
        if name == "pt_compact_planned_guarded":
            tables.append([bytes(j) for j in args[0][: args[1]]])
        return 0
    recorded.status = status

    def expected():
        small, acts = [], []
        for i, s in enumerate(m.specs):
            ik, nk = (None, None) if s.out_edge is None else (m.idx[s.out_edge], m.counts[s.out_edge:])
            ic, nc = (None, None) if s.in_edge is None else (m.idx[s.in_edge], m.counts[s.in_edge:])
            for src, dst in ((m.w[i], m.w_out[i]), (m.mom[i], m.mom_out[i])):
                small.append(B.planned_weights(src, s.K, s.R * s.S, s.C, hz.pitch8(s.C), ik, nk, ic, nc, dst))
            if ik is not None:
                small += [B.planned_vector(v, 4, s.K, ik, nk, o) for v, o in zip(m.bn[i], m.bn_out[i])]
            if m.act and ic is not None:
                acts.append(B.planned_nhwc(m.act[i], s.N * s.H * s.W, s.C, hz.pitch8(s.C), ic, nc, m.act_out[i]))
        # (fields a kind does not read may hold anything)
        return [sorted(map(_planned_fields, map(bytes, jobs))) for jobs in ([acts] if acts else []) + [small]]

    for again in range(3):
        tables.clear()
        recorded.calls.clear()
        m.compact()
        assert all(m.counts.data_ptr() in ps for _, ps in recorded.calls)   # the counts that must be positive
        assert [sorted(map(_planned_fields, t)) for t in tables] == expected()
        assert m.new_counts.tolist() == [20, 25]
        if again == 0:      # every tensor is another one
            for name in ("w", "mom", "act", "w_out", "mom_out", "act_out", "idx"):
                setattr(m, name, [t.clone() for t in getattr(m, name)])
            m.bn, m.bn_out, m.counts = [[v.clone() for v in vs] for vs in m.bn], [[v.clone() for v in vs] for vs in m.bn_out], m.counts.clone()
        else:               # the same objects, other memory
            for t in (*m.w, *m.act_out, *m.bn[0], *m.idx):
                t.data = t.data.clone()


@pytest.mark.parametrize("how", ["detect", "detect_separate", "detect_per_call"])
def test_detection_writes_the_plan_that_the_compaction_reads(recorded, monkeypatch, how):
    """Weights, survivor lists, counts and keep masks replaced between two sweeps: the second one reads and writes the new
    ones (a list that the plan did not write would be read as indices by the gathers)."""
    zeros = torch.zeros
    monkeypatch.setattr(torch, "zeros", lambda *a, pin_memory=False, **kw: zeros(*a, **kw))
    m = _reconfig_model()

    def tensors():
        return [*m.w, *m.idx, *m.keep, m.counts]
    getattr(m, how)(1e-6)
    old = tensors()
    assert {t.data_ptr() for t in old} <= recorded.seen()
    m.w, m.idx, m.keep, m.counts = ([t.clone() for t in m.w], [t.clone() for t in m.idx], [t.clone() for t in m.keep],
                                    m.counts.clone())
    recorded.calls.clear()
    getattr(m, how)(1e-6)
    assert {t.data_ptr() for t in tensors()} <= recorded.seen()
    assert not {t.data_ptr() for t in old} & recorded.seen()


def test_compaction_of_activations_that_do_not_stream(recorded, monkeypatch):
    """The planned gathers refuse an activation (as they do one that is not 16-byte aligned): compact() takes the calls with
    the counts on the host.  Another refusal is passed on."""
    zeros = torch.zeros
    monkeypatch.setattr(torch, "zeros", lambda *a, pin_memory=False, **kw: zeros(*a, **kw))
    m = _reconfig_model()
    recorded.status = lambda name, args: B.ERR_UNSUPPORTED if name == "pt_compact_planned_guarded" else 0
    m.compact()
    assert [name for name, _ in recorded.calls] == ["pt_compact_planned_guarded", "pt_compact_nhwc_batched",
                                                    "pt_compact_weights_batched", "pt_compact_vector_batched"]
    assert {t.data_ptr() for t in m.act[1:] + m.act_out[1:]} <= recorded.seen("pt_compact_nhwc_batched")
    assert {t.data_ptr() for t in m.w + m.mom + m.w_out + m.mom_out} <= recorded.seen("pt_compact_weights_batched")
    assert m.new_counts.tolist() == [20, 25]
    recorded.status = lambda name, args: -2 if name == "pt_compact_planned_guarded" else 0
    with pytest.raises(B.PruneTrainError):
        m.compact()


def test_edge_without_survivors_is_refused_on_either_route(recorded, monkeypatch):
    """The counts that come back hold a 0: the planned gathers (which write nothing then) end in the error that the calls
    with the counts on the host return.  A model with an edge of no layer, whose count is nobody's business, takes those."""
    zeros = torch.zeros
    monkeypatch.setattr(torch, "zeros", lambda *a, pin_memory=False, **kw: zeros(*a, **kw))
    m = _reconfig_model()
    m.counts[1] = 0
    with pytest.raises(B.PruneTrainError) as e:
        m.compact()
    assert e.value.status == -2 and {name for name, _ in recorded.calls} == {"pt_compact_planned_guarded"}
    m = _reconfig_model()
    m = hz.ReconfigModel(m.specs, m.edges + [wl.Edge("unused", 8, [0], [])], [w.numpy()[..., : s.C] for w, s in zip(m.w, m.specs)], 2)
    m.counts.copy_(torch.tensor([20, 25, 0], dtype=torch.int32))
    recorded.calls.clear()
    m.compact()
    assert m.new_counts.tolist() == [20, 25, 0] and "pt_compact_planned_guarded" not in {name for name, _ in recorded.calls}


def _planned_fields(job):
    j = B.PlannedGather.from_buffer_copy(job)
    used = {B.PLANNED_WEIGHTS: ("src", "out", "idxK", "nK_dev", "idxC", "nC_dev", "K", "RS", "C", "cpitch"),
            B.PLANNED_NHWC: ("src", "out", "idxC", "nC_dev", "rows", "C", "cpitch"),
            B.PLANNED_VECTOR: ("src", "out", "idxK", "nK_dev", "K", "elem_bytes")}[j.kind]
    return (j.kind, *((getattr(j, f) or 0) for f in used))


@pytest.mark.gpu
@pytest.mark.parametrize("grouped", [True, False])
def test_train_step_after_tensors_were_replaced_against_oracle(monkeypatch, grouped):
    """The next batch arrives in other tensors, the gradients are wanted elsewhere, and one input is only 8-byte aligned:
    the second step's outputs against the oracle, and the first step's tensors left as they were."""
    import oracle
    from gpu_util import CONV_TOL, host_bf16, rel_err
    if not grouped:
        monkeypatch.setattr(hz, "WGRAD_GROUP_MAX_BYTES", 0)
    specs = residual_block(N=8)
    rng = np.random.Generator(np.random.PCG64(21))
    batches = [[wl.conv_tensors(s, rng) for s in specs] for _ in range(2)]
    net = hz.Network([hz.ConvLayer(s, host=t) for s, t in zip(specs, batches[0])])
    assert net.grouped == grouped
    lam = 1e-2
    net.train_step(lam)
    torch.cuda.synchronize()
    first = [(l.x, l.dy, l.dw, l.dw.clone(), l.y, l.y.clone()) for l in net.layers]
    for l, t in zip(net.layers, batches[1]):
        l.x, l.dy = hz._to_dev_bf16(t["x"], l.xp), hz._to_dev_bf16(t["dy"], l.yp)
        l.dw, l.y = torch.zeros_like(l.dw), torch.zeros_like(l.y)
        if l.dx is not None:
            l.dx = torch.zeros_like(l.dx)
    x = net.layers[-1].x
    apart = torch.zeros(x.numel() + 4, dtype=x.dtype, device=x.device)[4:].view(x.shape)
    apart.copy_(x)
    net.layers[-1].x = apart
    assert apart.data_ptr() % 16 == 8
    net.train_step(lam)
    torch.cuda.synchronize()
    for l, t, w in zip(net.layers, batches[1], (b["w"] for b in batches[0])):
        s, o = l.spec, oracle.shape_of(l.spec)
        ron, rin = oracle.group_norms(w)
        assert rel_err(host_bf16(l.y, s.K), oracle.conv_fwd(o, t["x"], w)) <= CONV_TOL, s
        if l.dx is not None:
            assert rel_err(host_bf16(l.dx, s.C), oracle.conv_bwd_data(o, t["dy"], w)) <= CONV_TOL, s
        ref = oracle.group_lasso_grad(w, ron, rin, lam, l.lasso_flags, oracle.conv_bwd_weight(o, t["x"], t["dy"]))
        assert rel_err(l.dw.cpu().numpy()[..., : s.C], ref) <= CONV_TOL, s
    for _, _, dw, dw0, y, y0 in first:
        assert torch.equal(dw, dw0) and torch.equal(y, y0)


@pytest.mark.gpu
def test_sweep_with_a_misaligned_activation():
    """One saved activation starts 2 bytes off a 16-byte boundary: the sweep takes it, and every output equals plain
    indexing."""
    m = _reconfig_model()
    a = m.act[2]
    m.act[2] = torch.zeros(a.numel() + 1, dtype=a.dtype, device=a.device)[1:].view(a.shape)
    m.act[2].copy_(a)
    m.sweep(1e-6)
    torch.cuda.synchronize()
    kept = [m.idx[e][: int(n)].long() for e, n in enumerate(m.new_counts)]
    assert [k.numel() for k in kept] == [21, 26]
    for i, s in enumerate(m.specs):
        ik = torch.arange(s.K, device=a.device) if s.out_edge is None else kept[s.out_edge]
        ic = torch.arange(s.C, device=a.device) if s.in_edge is None else kept[s.in_edge]
        pitch = hz.pitch8(ic.numel())
        for src, out in ((m.w[i], m.w_out[i]), (m.mom[i], m.mom_out[i])):
            got = out.reshape(-1)[: ik.numel() * s.R * s.S * pitch].view(ik.numel(), s.R, s.S, pitch)
            assert torch.equal(got[..., : ic.numel()], src[ik][..., ic])
        if s.in_edge is not None:
            got = m.act_out[i].reshape(-1)[: s.N * s.H * s.W * pitch].view(s.N, s.H, s.W, pitch)
            assert torch.equal(got[..., : ic.numel()], m.act[i][..., ic])
        if s.out_edge is not None:
            for v, o in zip(m.bn[i], m.bn_out[i]):
                assert torch.equal(o[: ik.numel()], v[ik])
