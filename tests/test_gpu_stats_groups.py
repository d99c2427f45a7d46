"""Statistics that the workgroups put together themselves, counted in groups of 32 partial pairs: layers on both sides of a full
group, of several groups, and of the line in pairs (320, 5/4 workgroups per CU), beside layers of one pair; and in the fused step, up to
640 pairs (5/2 per CU; layers beyond 320 in calls of 24 MB beside as many chunks without one), the most groups a layer has (20)."""
import numpy as np
import pytest
import torch

import test_gpu_stats_fold as fold
from paper_2502_11058_amd import workloads as W
from paper_2502_11058_amd.harness import DeviceReplica

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per_layer", [[15], [16], [17], [16, 17, 1, 31, 32, 33], [255], [256], [257], [320], [321], [256, 64], [256, 65], [160, 1, 159],
                                       [20] * 16, [1] * 320, [1] * 321, [63], [64], [65], [32, 33, 1, 63, 64, 65], [288, 32], [287, 33]])
def test_groups(oracle, per_layer):
    fold.test_both_sides_of_the_line(oracle, per_layer)


@pytest.mark.parametrize("default", [False, True])
@pytest.mark.parametrize("dense_path", [1, 0])
@pytest.mark.parametrize("n,pairs", [(6, p) for p in ([321], [608], [609], [639], [640], [641], [320, 320], [320, 321], [577, 63], [1] * 20 + [600, 20])] +
                         [(8, p) for p in ([585], [586], [640], [641], [320, 320], [1] * 20 + [600, 20])])
def test_groups_beside_unscheduled_layers(oracle, n, pairs, dense_path, default):
    """A slot of half the model: whole, its statistics are folded up to 640 pairs; range by range, where every chunk has a pair, layers beyond 320 only in
    calls of less than 24 MB (eight replicas: up to 585 pairs), else by a launch of their own.  All of them give the same bits, and the oracle's
    values to 1e-10.  In chunks of 1024 elements that the caller gives, and in the halves that the fused step takes by itself (128 and 160 bytes
    a vector)."""
    assert torch.cuda.is_available(), "no GPU visible"
    L = len(pairs)
    sizes = [1024 * k - (l % 3) for l, k in enumerate(pairs)]
    rest = 2_400_000 if default else sum(sizes) + 2048          # (2.4 to 3.1 M elements: past the small models, short of whole chunks)
    ts = [W.TensorSpec(f"l{l}", l, k) for l, k in enumerate(sizes)] + [W.TensorSpec("rest", L, rest)]
    w = W.Workload(f"beside{L}_{pairs[0]}", ts, n_replicas=n, period=1, optimizer="sgdm", param_dtype="f32", lr=1e-2, sigma_drift=1e-3, policy="every")
    given = {} if default else {"update_chunk": 1024, "mean_chunk": 1024}
    rep = DeviceReplica(w, 0, options=dict(given, dense_path=dense_path))
    slot = list(range(L - 1, -1, -1))
    rep.install_schedule([0, L], slot)                          # the last layer is in no slot
    rep.init_params()
    rep.fill_grads(0)
    wk = oracle.Worker(rep.layer_of, [t.cpu().numpy() for t in rep.sync], "sgdm", dict(lr=w.lr, momentum=w.momentum), False)
    flat, off, order, total = wk.pack_slot(slot)
    rep.fill_peers_from(torch.from_numpy(flat).to(rep.dev), 0, total)
    reps = [flat] + [p[:total].cpu().numpy() for p in rep.peers]
    mean = oracle.mean(reps)
    ref = np.array([v for b, e in wk.layer_ranges(slot, off, order) for v in oracle.layer_stats(reps, mean, b, e)])
    saved, seen = [a.clone() for a in (rep.a_sync, rep.a_s0)], []
    for layers in (None, None, 1, 3):
        rep.a_sync.copy_(saved[0])
        rep.a_s0.copy_(saved[1])
        rep.stats.fill_(-1.0)
        if layers is None:
            rep.fused_step(0)
        else:
            for lo in range(0, L + 1, layers):
                rep.ctx.ddp_fused_sync_update_layers(0, lo, min(layers, L + 1 - lo), rep.peers, 0, 0, n, 0, rep.stats, rep.opt_struct(1))
        seen.append(rep.stats.cpu().numpy()[:2 * L].copy())
        np.testing.assert_allclose(seen[-1], ref, rtol=1e-10)
        assert np.array_equal(seen[-1], seen[0]), layers
    rep.close()
