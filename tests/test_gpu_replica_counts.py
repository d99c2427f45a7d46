"""Replica counts around every kernel that serves a range of counts (1..3, 5..7, 9..15, 17..31) and its neighbours, each with
the local replica first, last and in between: average and fused step, fp32 and bf16 exchange, with and without statistics,
every element against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2502_11058_amd import workloads as W
from paper_2502_11058_amd.harness import DeviceReplica

pytestmark = pytest.mark.gpu


def _host(t):
    return t.view(torch.int16).cpu().numpy().view(np.uint16) if t.dtype == torch.bfloat16 else t.cpu().numpy()


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 8, 9, 12, 15, 16, 17, 25, 31, 32, 33])
@pytest.mark.parametrize("wire16", [False, True])
def test_counts_and_ranks(oracle, n, wire16):
    assert torch.cuda.is_available(), "no GPU visible"
    sizes = [[2050, 3], [1, 1023], [4097], [5]]
    ts = [W.TensorSpec(f"{l}.{j}", l, k) for l, ks in enumerate(sizes) for j, k in enumerate(ks)]
    for optimizer, dtype in (("adamw", "bf16"), ("sgdm", "f32")):
        w = W.Workload(f"counts{n}", ts, n_replicas=n, period=2, optimizer=optimizer, param_dtype=dtype, lr=1e-2, sigma_drift=1e-3)
        rep = DeviceReplica(w, 0, wire16=wire16)
        hyper = dict(lr=w.lr, momentum=w.momentum, beta1=w.beta1, beta2=w.beta2, eps=w.eps, weight_decay=w.weight_decay)
        rep.init_params()
        rep.sync[0][5] = -0.0                                  # the sum must keep the sign of a zero
        wk = oracle.Worker(rep.layer_of, [_host(t) for t in rep.sync], optimizer, hyper, rep.bf16)
        for r, rank in enumerate(sorted({0, n // 2, n - 1})):
            S = rep.sets[r % 2]
            flat, _, _, total = wk.pack_slot(S)
            base = torch.from_numpy(flat).to(rep.dev)
            (rep.fill_peers16_from if wire16 else rep.fill_peers_from)(base, r, total)
            peers = [p[:total] for p in (rep.peers16 if wire16 else rep.peers)]
            for p in peers:
                p[base == 0.0] = -0.0
            rep.fill_grads(r)
            host_peers = [_host(p) for p in peers]
            local = oracle.bf16_rne(flat) if wire16 else flat
            reps = host_peers[:rank] + [local] + host_peers[rank:]
            want = (oracle.mean_wire16 if wire16 else oracle.mean)(reps)
            if wire16:
                rep.ctx.ddp_pack_wire16(r % 2, rep.flat16)
                rep.ctx.ddp_partial_average_wire16(r % 2, rep.flat16, rep.peers16, n, rank, rep.flat, rep.stats)
            else:
                rep.ctx.ddp_pack(r % 2, rep.flat)
                rep.ctx.ddp_partial_average(r % 2, rep.flat, rep.peers, n, rank, rep.flat, rep.stats)
            assert np.array_equal(_host(rep.flat[:total]).view(np.int32), want.view(np.int32)), (n, rank)
            by_average = rep.stats.cpu().numpy().copy()
            rep.stats.fill_(-1.0)                              # whatever the fused step leaves out stays visible
            _, ref = wk.sync(S, host_peers, rank, wire16=wire16)
            wk.local_update([_host(g) for g in rep.grad], r + 1)
            rep.fused_step(r, rank, with_stats=r != 1, wire16=wire16)          # without statistics in between
            by_fused = rep.stats.cpu().numpy()
            if r == 1:
                assert (by_fused == -1.0).all(), (n, rank)
            for i, (gam, msq) in enumerate(ref):
                for got in (by_average,) if r == 1 else (by_average, by_fused):
                    assert got[2 * i] == pytest.approx(gam, rel=1e-10, abs=1e-300) and got[2 * i + 1] == pytest.approx(msq, rel=1e-10)
            for a, b in zip(rep.sync, wk.p):
                assert np.array_equal(_host(a).view(np.int32), b.view(np.int32)), (optimizer, n, rank)
        rep.close()
