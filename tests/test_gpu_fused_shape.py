"""The fused step's chunks of 1024 elements, the update's and the unscheduled pieces' of two of them, with default options: layers around
one and several of both, and statistics of up to and beyond 5/2 workgroups per CU with a pair; the four calls and the fused step, whole
and layer by layer, dense and through the table.  Every element against the oracle, bit for bit, statistics to 1e-10."""
import numpy as np
import pytest
import torch

from paper_2502_11058_amd import workloads as W
from paper_2502_11058_amd.harness import DeviceReplica
from test_gpu_parity import run_trajectory

pytestmark = pytest.mark.gpu

AROUND = [1023, 1024, 1025, 2047, 2048, 2049, 3071, 3072, 3073, 1, 64 * 17, 4096 + 61, 2, 5 * 1024 + 3]


@pytest.mark.parametrize("dense_path", [1, 0])
@pytest.mark.parametrize("fused,layerwise", [(False, 0), (True, 0), (True, 1), (True, 4)])
@pytest.mark.parametrize("chunks", [AROUND, [640], [641], [640 - 7, 3, 4], [700, 1, 5]])
@pytest.mark.parametrize("n,wire16", [(2, True), (6, False)])
def test_chunks_and_pairs(oracle, n, wire16, chunks, fused, layerwise, dense_path):
    sizes = chunks if chunks is AROUND else [1024 * k - (l % 3) for l, k in enumerate(chunks)]
    ts = [W.TensorSpec(f"l{l}", l, k) for l, k in enumerate(sizes)]
    w = W.Workload(f"shape{len(sizes)}_{sizes[0]}", ts, n_replicas=n, period=3 if chunks is AROUND else 1, optimizer="sgdm", param_dtype="f32",
                   lr=1e-2, sigma_drift=1e-3, iterations=3, policy="round_robin" if chunks is AROUND else "every")
    iters = 3 if chunks is AROUND else 1
    assert run_trajectory(oracle, w, iters=iters, fused=fused, wire16=wire16, layerwise=layerwise, options={"dense_path": dense_path}).frac() == 1.0


@pytest.mark.parametrize("dense_path", [1, 0])
@pytest.mark.parametrize("given", [{"update_wg_per_cu": 2}, {"update_lds": 64512}])
def test_a_given_residency_is_one_of_whole_chunks(given, dense_path):
    """update_wg_per_cu or update_lds without update_chunk: the fused step keeps the chunks of 2048 elements that the option is stated for.  The
    statistics' partial sums are a chunk's, so their last bits tell."""
    assert torch.cuda.is_available(), "no GPU visible"
    ts = [W.TensorSpec(f"l{l}", l, k) for l, k in enumerate([100_003, 250_007, 65_537, 180_001])]
    w = W.Workload("given", ts, n_replicas=4, period=1, optimizer="sgdm", param_dtype="f32", lr=1e-2, sigma_drift=1e-3, policy="every")

    def stats(options):
        rep = DeviceReplica(w, 0, options=dict(options, dense_path=dense_path))
        rep.init_params()
        rep.fill_grads(0)
        flat = torch.cat([rep.sync[l] for l in rep.sets[0]])
        rep.fill_peers_from(flat, 0, flat.numel())
        rep.fused_step(0)
        out = rep.stats.cpu().numpy()[:2 * len(ts)].copy()
        rep.close()
        return out

    whole, halves = stats({"update_chunk": 2048}), stats({})
    np.testing.assert_allclose(halves, whole, rtol=1e-12)
    assert not np.array_equal(halves, whole)             # seen for these seeded inputs: the shapes can be told apart
    assert np.array_equal(stats(given), whole)


@pytest.mark.parametrize("dense_path", [1, 0])
def test_captured_ranges_in_halves(dense_path):
    """Range calls with default options in a captured graph, replayed between eager calls: the bits of the eager ones, statistics too."""
    assert torch.cuda.is_available(), "no GPU visible"
    ts = [W.TensorSpec(f"l{l}", l, k) for l, k in enumerate([1021, 100_003, 2049, 250_007, 64, 65_537])]
    L, n = len(ts), 5
    w = W.Workload("captured", ts, n_replicas=n, period=2, optimizer="sgdm", param_dtype="f32", lr=1e-2, sigma_drift=1e-3, policy="round_robin")
    rep = DeviceReplica(w, 0, options={"dense_path": dense_path})
    rep.init_params()
    rep.fill_grads(0)
    rep.fill_peers_from(torch.cat([rep.sync[l] for l in rep.sets[1]]), 1, rep.slot_numel[1])
    saved, opt, s = [a.clone() for a in (rep.a_sync, rep.a_s0)], rep.opt_struct(1), torch.cuda.Stream()

    def calls(stream):
        for l in range(L - 1, -1, -1):
            rep.ctx.ddp_fused_sync_update_layers(1, l, 1, rep.peers, 0, 0, n, 0, rep.stats, opt, stream)

    def fresh():
        rep.a_sync.copy_(saved[0])
        rep.a_s0.copy_(saved[1])
        rep.stats.fill_(-1.0)
        torch.cuda.synchronize()

    def result():
        torch.cuda.synchronize()
        return [a.clone() for a in (rep.a_sync, rep.a_s0, rep.stats)]

    fresh()
    calls(None)
    first = result()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        calls(s)
    for _ in range(3):
        fresh()
        g.replay()
        assert all(torch.equal(a, b) for a, b in zip(result(), first))
        fresh()
        calls(None)
        assert all(torch.equal(a, b) for a, b in zip(result(), first))
    rep.close()


@pytest.mark.parametrize("layerwise", [0, 2])
@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("n,wire16,chunks", [(16, False, 1439), (16, False, 1440), (32, True, 1791), (32, True, 1792)])
def test_small_models_by_their_workgroups(oracle, n, wire16, chunks, order, layerwise):
    """Small models over the table, on both sides of the lines in workgroups (45/8 and 7 per CU of 256) from which three and four of them take a CU."""
    sizes = [1024 * k - (l % 3) for l, k in enumerate([1, chunks - 703, 2, 700])]
    ts = [W.TensorSpec(f"l{l}", l, k) for l, k in enumerate(sizes)]
    w = W.Workload(f"small{chunks}", ts, n_replicas=n, period=2, optimizer="sgdm", param_dtype="f32", lr=1e-2, sigma_drift=1e-3, iterations=2, policy="round_robin")
    assert run_trajectory(oracle, w, iters=2, fused=True, wire16=wire16, layerwise=layerwise, order=order, options={"dense_path": 0}).frac() == 1.0


@pytest.mark.parametrize("dense_path", [1, 0])
@pytest.mark.parametrize("layerwise", [0, 1])
@pytest.mark.parametrize("optimizer", ["sgdm", "adamw"])
@pytest.mark.parametrize("period", [10, 5, 2])
def test_slots_of_all_sizes(oracle, period, optimizer, layerwise, dense_path):
    """A model of 7.6 chunks of 2048 elements per CU: slots of 0.8, 1.5 and 3.8, which take halves of chunks, whole ones, and either by the optimizer."""
    ts = [W.TensorSpec(f"l{l}", l, 400_001 + 7 * l) for l in range(10)]
    w = W.Workload(f"slots{period}", ts, n_replicas=4, period=period, optimizer=optimizer, param_dtype="bf16" if optimizer == "adamw" else "f32", lr=1e-3,
                   sigma_drift=1e-3, iterations=1, policy="round_robin")
    assert run_trajectory(oracle, w, iters=1, fused=True, layerwise=layerwise, options={"dense_path": dense_path}).frac() == 1.0
