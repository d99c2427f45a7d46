"""Statistics that the workgroups put together themselves (launches in which up to 5/4 workgroups per CU have a
share; the fused step up to 5/2, large layers in calls of 24 MB beside as many chunks without one) and those of a launch of their own, on both sides of the rule's lines: against the oracle, the same bits on every
repetition, the same bits for the allocation-free entry point (which never folds), and through a captured graph that is
replayed between eager calls."""
import numpy as np
import pytest
import torch

from paper_2502_11058_amd import workloads as W
from paper_2502_11058_amd.harness import DeviceReplica

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per_layer", [[1], [3, 5], [64] * 4, [319], [320], [321], [200, 1, 119], [1] * 40, [900, 2],
                                       [127], [128], [129], [70, 1, 57], [70, 1, 58], [33] * 3, [2] * 64, [2] * 65])
def test_both_sides_of_the_line(oracle, per_layer):
    assert torch.cuda.is_available(), "no GPU visible"
    n = 4
    ts = [W.TensorSpec(f"l{l}", l, 1024 * k - (l % 3)) for l, k in enumerate(per_layer)]
    w = W.Workload(f"fold{len(per_layer)}_{per_layer[0]}", ts, n_replicas=n, period=1, optimizer="sgdm", param_dtype="f32", lr=1e-2,
                   sigma_drift=1e-3, policy="every")
    rep = DeviceReplica(w, 0, options={"update_chunk": 1024, "mean_chunk": 1024})
    rep.init_params()
    rep.fill_grads(0)
    wk = oracle.Worker(rep.layer_of, [t.cpu().numpy() for t in rep.sync], "sgdm", dict(lr=w.lr, momentum=w.momentum), False)
    flat, off, order, total = wk.pack_slot(rep.sets[0])
    local = torch.from_numpy(flat).to(rep.dev)
    rep.fill_peers_from(local, 0, total)
    reps = [flat] + [p[:total].cpu().numpy() for p in rep.peers]
    mean = oracle.mean(reps)
    ref = np.array([v for b, e in wk.layer_ranges(rep.sets[0], off, order) for v in oracle.layer_stats(reps, mean, b, e)])
    k = 2 * len(per_layer)
    out = torch.zeros_like(rep.flat)
    src = torch.zeros_like(rep.flat)
    src[:total] = local

    def call(fn):
        rep.stats.fill_(-1.0)
        fn(0, src, rep._peers_arr, n, 0, out, rep.stats)
        return rep.stats.cpu().numpy()[:k].copy()

    first = call(rep.ctx.ddp_partial_average)
    np.testing.assert_allclose(first, ref, rtol=1e-10)
    for _ in range(3):
        assert np.array_equal(call(rep.ctx.ddp_partial_average), first)
    assert np.array_equal(call(rep.ctx.ddp_partial_average_static), first)

    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            rep.ctx.ddp_partial_average(0, src, rep._peers_arr, n, 0, out, rep.stats, s)
    for _ in range(3):
        rep.stats.fill_(-1.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(rep.stats.cpu().numpy()[:k], first)
        assert np.array_equal(call(rep.ctx.ddp_partial_average), first)

    saved = [a.clone() for a in (rep.a_sync, rep.a_s0)]
    seen = []
    for layers in (None, None, 1, 3):                              # whole model twice, then range by range
        rep.a_sync.copy_(saved[0])
        rep.a_s0.copy_(saved[1])
        rep.stats.fill_(-1.0)
        if layers is None:
            rep.fused_step(0)
        else:
            for lo in range(0, len(per_layer), layers):
                rep.ctx.ddp_fused_sync_update_layers(0, lo, min(layers, len(per_layer) - lo), rep.peers, 0, 0, n, 0, rep.stats,
                                                     rep.opt_struct(1))
        seen.append(rep.stats.cpu().numpy()[:k].copy())
        np.testing.assert_allclose(seen[-1], ref, rtol=1e-10)
    assert all(np.array_equal(x, seen[0]) for x in seen)
    rep.close()


@pytest.mark.parametrize("default", [False, True])
@pytest.mark.parametrize("dense_path", [1, 0])
@pytest.mark.parametrize("per_layer", [[60, 4097, 3, 120, 7, 300], [60, 4096, 3, 120, 7, 300], [60, 8193, 3, 120, 7, 300], [60, 8192, 3, 120, 7, 300]])
def test_small_layers_beside_a_large_one(per_layer, dense_path, default):
    """One layer on either side of the number of partials (8192) from which a slot's statistics take the two-stage reduction: the
    small layers' statistics have the same bits from the whole-model call and from every partition into ranges.  In chunks of 1024
    elements that the caller gives, and in those that the fused step takes by itself, halves of chunks of 2048 (with 4096, whole ones)."""
    assert torch.cuda.is_available(), "no GPU visible"
    ts = [W.TensorSpec(f"l{l}", l, 1024 * k) for l, k in enumerate(per_layer)]
    w = W.Workload(f"order{per_layer[1]}", ts, n_replicas=3, period=1, optimizer="sgdm", param_dtype="f32", lr=1e-2, sigma_drift=1e-3,
                   policy="every")
    given = {} if default else {"update_chunk": 1024, "mean_chunk": 1024}
    rep = DeviceReplica(w, 0, options=dict(given, dense_path=dense_path))
    rep.init_params()
    rep.fill_grads(0)
    S = rep.sets[0]
    flat = torch.cat([rep.sync[l] for l in S])
    rep.fill_peers_from(flat, 0, flat.numel())
    saved = [a.clone() for a in (rep.a_sync, rep.a_s0)]
    seen = []
    for layers in (None, 1, 2, 3, len(per_layer)):
        rep.a_sync.copy_(saved[0])
        rep.a_s0.copy_(saved[1])
        rep.stats.fill_(-1.0)
        if layers is None:
            rep.fused_step(0)
        else:
            for lo in range(0, len(per_layer), layers):
                rep.ctx.ddp_fused_sync_update_layers(0, lo, min(layers, len(per_layer) - lo), rep.peers, 0, 0, 3, 0, rep.stats,
                                                     rep.opt_struct(1))
        seen.append(rep.stats.cpu().numpy()[:2 * len(per_layer)].copy())
        assert (seen[-1] >= 0.0).all()
        assert np.array_equal(seen[-1], seen[0]), layers
    rep.close()


@pytest.mark.parametrize("default", [False, True])
@pytest.mark.parametrize("dense_path", [1, 0])
@pytest.mark.parametrize("per_layer", [[30] * 12, [128, 1, 127, 64, 3, 100]])
def test_ranges_in_flight_on_two_streams(per_layer, dense_path, default):
    """Range calls that put their statistics together themselves, disjoint ones in flight at the same time on two streams (each
    layer has its own counter and partials): the bits of the calls one after the other, on every repetition.  In chunks that the
    caller gives and in halves of the default ones."""
    assert torch.cuda.is_available(), "no GPU visible"
    L = len(per_layer)
    ts = [W.TensorSpec(f"l{l}", l, 1024 * k - (l % 3)) for l, k in enumerate(per_layer)]
    w = W.Workload(f"streams{L}", ts, n_replicas=4, period=1, optimizer="sgdm", param_dtype="f32", lr=1e-2, sigma_drift=1e-3, policy="every")
    given = {} if default else {"update_chunk": 1024, "mean_chunk": 1024}
    rep = DeviceReplica(w, 0, options=dict(given, dense_path=dense_path))
    rep.init_params()
    rep.fill_grads(0)
    flat = torch.cat([rep.sync[l] for l in rep.sets[0]])
    rep.fill_peers_from(flat, 0, flat.numel())
    saved = [a.clone() for a in (rep.a_sync, rep.a_s0)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    opt = rep.opt_struct(1)
    seen = []
    for turn in range(12):
        rep.a_sync.copy_(saved[0])
        rep.a_s0.copy_(saved[1])
        rep.stats.fill_(-1.0)
        torch.cuda.synchronize()
        for l in range(L):
            s = streams[l % 2] if turn else streams[0]
            rep.ctx.ddp_fused_sync_update_layers(0, l, 1, rep._peers_arr, 0, 0, 4, 0, rep.stats, opt, s)
        torch.cuda.synchronize()
        seen.append([rep.stats.clone(), rep.a_sync.clone(), rep.a_s0.clone()])
        assert all(torch.equal(a, b) for a, b in zip(seen[-1], seen[0])), turn
    rep.close()


@pytest.mark.parametrize("dense_path", [1, 0])
def test_both_wires_in_flight_on_two_streams(dense_path):
    """Range calls of one worker on fp32 and on bf16 peers, in flight at the same time on two streams, with default options in a model for which
    eleven fp32 replicas take halves of chunks and eleven bf16 ones whole chunks: the bits of the calls one after the other."""
    assert torch.cuda.is_available(), "no GPU visible"
    n, L = 11, 12
    ts = [W.TensorSpec(f"l{l}", l, 300_001 + 1000 * l) for l in range(L)]                # 3.67 M elements, 7 chunks of 2048 per CU
    w = W.Workload("wires", ts, n_replicas=n, period=1, optimizer="sgdm", param_dtype="f32", lr=1e-2, sigma_drift=1e-3, policy="every")
    rep = DeviceReplica(w, 0, options={"dense_path": dense_path}, wire16=True)
    rep.init_params()
    rep.fill_grads(0)
    flat = torch.cat([rep.sync[l] for l in rep.sets[0]])
    rep.fill_peers16_from(flat, 0, flat.numel())
    saved = [a.clone() for a in (rep.a_sync, rep.a_s0)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    opt = rep.opt_struct(1)
    seen = []
    for turn in range(12):
        rep.a_sync.copy_(saved[0])
        rep.a_s0.copy_(saved[1])
        rep.stats.fill_(-1.0)
        torch.cuda.synchronize()
        for l in range(L):
            wire = l % 2
            rep.ctx.ddp_fused_sync_update_layers(0, l, 1, rep._peers16_arr if wire else rep._peers_arr, wire, 0, n, 0, rep.stats, opt,
                                                 streams[wire] if turn else streams[0])
        torch.cuda.synchronize()
        seen.append([rep.stats.clone(), rep.a_sync.clone(), rep.a_s0.clone()])
        assert (seen[-1][0][:2 * L] > 0.0).all()
        assert all(torch.equal(a, b) for a, b in zip(seen[-1], seen[0])), turn
    rep.close()


@pytest.mark.parametrize("per_layer", [[200, 256, 1, 64, 65, 255], [1] * 330, [256, 256], [63, 127, 128, 129, 192, 193], [256] * 40])
def test_narrow_and_wide_workgroups(per_layer):
    """Layers of up to 256 partial pairs, which a launch of its own adds up by workgroups of 256 threads; beside one layer of 257, by workgroups
    of 1024: the same bits, from the average and from the fused step."""
    assert torch.cuda.is_available(), "no GPU visible"
    n, seen = 3, []
    sizes = [1024 * k - (l % 3) for l, k in enumerate(per_layer)]
    total = sum(sizes)
    data = [torch.randn(total + 257 * 1024, device="cuda", generator=torch.Generator("cuda").manual_seed(k)) for k in range(n)]
    for numel in (sizes, sizes + [257 * 1024]):
        L = len(numel)
        ts = [W.TensorSpec(f"l{l}", l, k) for l, k in enumerate(numel)]
        w = W.Workload(f"wide{len(sizes)}_{L}", ts, n_replicas=n, period=1, optimizer="sgdm", param_dtype="f32", lr=1e-2, sigma_drift=1e-3, policy="every")
        rep = DeviceReplica(w, 0, options={"update_chunk": 1024, "mean_chunk": 1024})
        rep.install_schedule([0, L], list(range(L)))
        rep.fill_grads(0)
        at = 0
        for l, k in enumerate(numel):
            rep.sync[l].copy_(data[0][at:at + k])
            at += k
        src, out = torch.zeros_like(rep.flat), torch.zeros_like(rep.flat)
        src[:at] = data[0][:at]
        for p, d in zip(rep.peers, data[1:]):
            p[:at] = d[:at]
        rep.stats.fill_(-1.0)
        rep.ctx.ddp_partial_average(0, src, rep._peers_arr, n, 0, out, rep.stats)
        seen.append(rep.stats.cpu().numpy()[:2 * len(sizes)].copy())
        rep.stats.fill_(-1.0)
        rep.fused_step(0)
        seen.append(rep.stats.cpu().numpy()[:2 * len(sizes)].copy())
        rep.close()
    a = torch.stack([d[:total] for d in data]).double()
    mean = a.sum(0) / n
    ref = [((a - mean) ** 2).sum(0) / n, mean ** 2]
    ref = np.array([r[b:b + k].sum().item() for b, k in zip(np.cumsum([0] + sizes), sizes) for r in ref])
    for s in seen:
        np.testing.assert_allclose(s, ref, rtol=1e-5)            # (the device's mean is rounded to 32 bits: 2^-24 of it in each difference)
    assert np.array_equal(seen[0], seen[2]) and np.array_equal(seen[1], seen[3])
