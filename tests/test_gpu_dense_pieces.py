"""The fused step over dense arenas cuts the model into pieces that share a launch: more layers than one launch takes, layers
of one element to several chunks, odd starts, one layer much wider than the rest, all layers scheduled, every other one, or
none; whole-model calls and ranges of layers.  Every element against the oracle, bit for bit."""
import pytest
import torch

from paper_2502_11058_amd import workloads as W
from paper_2502_11058_amd.harness import DeviceReplica
from test_gpu_parity import run_trajectory

pytestmark = pytest.mark.gpu

SIZES = [1, 1023, 5, 2048, 4097, 3, 1024, 9000, 2, 6143]


def _workload(n_layers, wide, optimizer, dtype, n, policy, period):
    ts = [W.TensorSpec(f"l{l}", l, wide if l == n_layers // 2 else SIZES[l % len(SIZES)]) for l in range(n_layers)]
    return W.Workload(f"pieces{n_layers}_{wide}_{n}", ts, n_replicas=n, period=period, optimizer=optimizer, param_dtype=dtype, lr=1e-3,
                      sigma_drift=1e-3, iterations=3, policy=policy)


@pytest.mark.parametrize("layerwise", [0, 1, 40])
@pytest.mark.parametrize("n_layers,policy,period", [(1, "full", 2), (3, "enp", 3), (40, "every", 1), (70, "round_robin", 2), (70, "enp", 4)])
@pytest.mark.parametrize("optimizer,dtype,n,wire16", [("sgdm", "f32", 5, False), ("adamw", "bf16", 8, True)])
def test_pieces(oracle, n_layers, policy, period, optimizer, dtype, n, wire16, layerwise):
    w = _workload(n_layers, 400_003, optimizer, dtype, n, policy, period)
    t = run_trajectory(oracle, w, iters=3, fused=True, wire16=wire16, layerwise=layerwise, options={"update_chunk": 1024})
    assert t.frac() == 1.0


@pytest.mark.parametrize("n_layers,period,policy", [(20, 1, "every"), (21, 1, "every"), (300, 1, "every"), (41, 2, "round_robin")])
@pytest.mark.parametrize("optimizer,dtype,n,wire16", [("sgdm", "f32", 4, False), ("adamw", "bf16", 3, True)])
def test_more_segments_than_a_launch_takes(oracle, n_layers, period, policy, optimizer, dtype, n, wire16):
    """Small models on both sides of the number of segments from which their slots take the table: layers of several tensors,
    whole-model calls and ranges of layers, every element against the oracle and the same statistics whatever the ranges."""
    ts = [W.TensorSpec(f"l{l}.{j}", l, SIZES[(l + j) % len(SIZES)]) for l in range(n_layers) for j in range(1 + l % 3)]
    w = W.Workload(f"segments{n_layers}", ts, n_replicas=n, period=period, optimizer=optimizer, param_dtype=dtype, lr=1e-3, sigma_drift=1e-3,
                   iterations=2, policy=policy)
    for layerwise in (0, 1, 7):
        assert run_trajectory(oracle, w, iters=2, fused=True, wire16=wire16, layerwise=layerwise, options={"update_chunk": 1024}).frac() == 1.0
    seen = []
    for dense_path in (1, 0):
        rep = DeviceReplica(w, 0, options={"update_chunk": 1024, "dense_path": dense_path}, wire16=wire16)
        rep.init_params()
        rep.fill_grads(0)
        flat = torch.cat([t for l in rep.sets[0] for t, k in zip(rep.sync, rep.layer_of) if k == l])
        (rep.fill_peers16_from if wire16 else rep.fill_peers_from)(flat, 0, flat.numel())
        streams = [a for a in (rep.a_sync, rep.a_s0, rep.a_s1, rep.a_model) if a is not None]
        saved = [a.clone() for a in streams]
        for layers in (n_layers, 1, 7):
            for a, b in zip(streams, saved):
                a.copy_(b)
            rep.stats.fill_(-1.0)
            for lo in range(0, n_layers, layers):
                rep.ctx.ddp_fused_sync_update_layers(0, lo, min(layers, n_layers - lo), rep.peers16 if wire16 else rep.peers, int(wire16), 0, n, 0,
                                                     rep.stats, rep.opt_struct(1))
            seen.append([rep.stats.cpu()] + [a.cpu() for a in streams])
        rep.close()
    assert all(torch.equal(a, b) for got in seen[1:] for a, b in zip(got, seen[0]))


@pytest.mark.parametrize("chunks", [16383, 16385])
def test_long_table_launches(chunks):
    """AdamW launches of the table-driven kernels on both sides of the length from which they ask for less at a time: the bits of
    the table-free kernels, for the update alone and for the fused step."""
    w = W.Workload(f"long{chunks}", [W.TensorSpec("a", 0, 1024 * (chunks - 3) + 5), W.TensorSpec("b", 1, 2051)], n_replicas=2, period=2,
                   optimizer="adamw", param_dtype="bf16", lr=1e-3, sigma_drift=1e-3, policy="round_robin")
    got = []
    for dense_path in (1, 0):
        rep = DeviceReplica(w, 0, options={"update_chunk": 1024, "dense_path": dense_path})
        rep.init_params()
        for r in (0, 1):                                # the long layer scheduled, then the short one
            rep.fill_grads(r)
            rep.ctx.ddp_pack(r, rep.flat)
            rep.fill_peers_from(rep.flat, r, rep.slot_numel[r])
            rep.fused_step(r)
            rep.ctx.ddp_local_update(rep.opt_struct(r + 2))
        got.append([a.cpu() for a in (rep.a_sync, rep.a_s0, rep.a_s1, rep.a_model, rep.stats)])
        rep.close()
    assert all(torch.equal(a, b) for a, b in zip(*got))
