"""The fused step over dense arenas cuts the model into pieces that share a launch: more layers than one launch takes, layers
of one element to several chunks, odd starts, one layer much wider than the rest, all layers scheduled, every other one, or
none; whole-model calls and ranges of layers.  Every element against the oracle, bit for bit."""
import pytest

from paper_2502_11058_amd import workloads as W
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
