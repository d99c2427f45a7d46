"""The average of 17 to 32 replicas, and over small slots of 12 to 16 fp32 ones, cuts chunks in two: layers that end on either
side of a cut or of a chunk and start anywhere in a line, on both sides of the rule's lines (replica count, wire, slot size).
Every element against the oracle, bit for bit; the allocation-free entry point gives the same bits and statistics."""
import pytest
import torch

from paper_2502_11058_amd import workloads as W
from paper_2502_11058_amd.harness import DeviceReplica
from test_gpu_parity import run_trajectory

pytestmark = pytest.mark.gpu

SIZES = [1, 511, 512, 513, 449, 575, 1023, 1024, 1025, 3 * 1024 + 7, 64 * 33 - 1, 2]


@pytest.mark.parametrize("n,wire16", [(11, False), (12, False), (16, False), (16, True), (17, True), (24, False), (24, True), (31, False), (32, False), (32, True), (33, True)])
@pytest.mark.parametrize("wide", [0, 2100 * 1024 + 5])
def test_cut(oracle, n, wire16, wide):
    sizes = SIZES + ([wide] if wide else [])
    ts = [W.TensorSpec(f"l{l}", l, k) for l, k in enumerate(sizes)]
    w = W.Workload(f"cut{n}_{wide}", ts, n_replicas=n, period=1, optimizer="sgdm", param_dtype="f32", lr=1e-3, sigma_drift=1e-3, iterations=1,
                   policy="every")
    options = {"mean_chunk": 1024}
    assert run_trajectory(oracle, w, iters=1, fused=False, wire16=wire16, options=options).frac() == 1.0
    if wire16:
        return
    rep = DeviceReplica(w, 0, options=options)
    rep.init_params()
    rep.ctx.ddp_pack(0, rep.flat)
    rep.fill_peers_from(rep.flat, 0, rep.slot_numel[0])
    got = []
    for fn in (rep.ctx.ddp_partial_average, rep.ctx.ddp_partial_average_static):
        out = torch.zeros_like(rep.flat)
        rep.stats.fill_(-1.0)
        fn(0, rep.flat, rep._peers_arr, n, 0, out, rep.stats)
        got.append((out, rep.stats.clone()))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    rep.close()
