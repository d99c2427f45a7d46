"""Chunks end on cache lines (multiples of 64 elements): layers of a line and one element more or less, of whole chunks and a
line more or less, that start anywhere in a line; the four calls and the fused step over dense arenas, whole and layer by
layer, and through the table.  Every element against the oracle, bit for bit."""
import pytest

from paper_2502_11058_amd import workloads as W
from test_gpu_parity import run_trajectory

pytestmark = pytest.mark.gpu

SIZES = [61, 64, 63, 1, 1024 - 61, 1024, 1025, 3 * 1024 + 7, 64 * 33 - 1, 2048 - 64, 2048 + 63, 4096 - 3, 128, 65, 960, 2]


@pytest.mark.parametrize("dense_path", [1, 0])
@pytest.mark.parametrize("fused,layerwise", [(False, 0), (True, 0), (True, 1), (True, 3)])
@pytest.mark.parametrize("optimizer,dtype,n,wire16", [("sgdm", "f32", 3, False), ("adamw", "bf16", 8, True)])
def test_layers_around_lines_and_chunks(oracle, optimizer, dtype, n, wire16, fused, layerwise, dense_path):
    ts = [W.TensorSpec(f"l{l}", l, k) for l, k in enumerate(SIZES)]
    w = W.Workload("lines", ts, n_replicas=n, period=2, optimizer=optimizer, param_dtype=dtype, lr=1e-3, sigma_drift=1e-3, iterations=2,
                   policy="round_robin")
    options = {"update_chunk": 1024, "mean_chunk": 1024, "copy_chunk": 1024, "dense_path": dense_path}
    assert run_trajectory(oracle, w, iters=2, fused=fused, wire16=wire16, layerwise=layerwise, options=options).frac() == 1.0


@pytest.mark.parametrize("dense_path", [1, 0])
@pytest.mark.parametrize("layerwise", [0, 1, 3])
@pytest.mark.parametrize("n,wire16", [(3, False), (8, True), (12, False), (32, True)])
def test_default_halves_around_lines_and_chunks(oracle, n, wire16, layerwise, dense_path):
    ts = [W.TensorSpec(f"l{l}", l, k) for l, k in enumerate(SIZES)]
    w = W.Workload("lines_default", ts, n_replicas=n, period=2, optimizer="sgdm", param_dtype="f32", lr=1e-3, sigma_drift=1e-3, iterations=2,
                   policy="round_robin")
    assert run_trajectory(oracle, w, iters=2, fused=True, wire16=wire16, layerwise=layerwise, options={"dense_path": dense_path}).frac() == 1.0
