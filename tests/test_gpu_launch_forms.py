"""Unscheduled layers that start anywhere in a vector, called layer by layer and in ranges, and averages of 9 to 16 replicas on both sides
of the line where the two sums of a launch are formed one after the other (8192 chunks): every element against the oracle, bit for bit,
statistics to 1e-10."""
import pytest

from paper_2502_11058_amd import workloads as W
from test_gpu_parity import run_trajectory

pytestmark = pytest.mark.gpu


def _run(oracle, sizes, n, period, policy, adam=False, **kw):
    ts = [W.TensorSpec(f"l{l}", l, k) for l, k in enumerate(sizes)]
    w = W.Workload(f"forms{len(sizes)}_{sizes[0]}", ts, n_replicas=n, period=period, optimizer="adamw" if adam else "sgdm", param_dtype="bf16" if adam else "f32",
                   lr=1e-3 if adam else 1e-2, sigma_drift=1e-3, iterations=period, policy=policy)
    assert run_trajectory(oracle, w, iters=period, **kw).frac() == 1.0


@pytest.mark.parametrize("adam", [False, True])
@pytest.mark.parametrize("layerwise", [1, 3])
@pytest.mark.parametrize("sizes", [[1, 1023, 2, 2047, 3, 2049, 61, 64], [3 * 2048 + 1, 509 * 510, 127, 65, 4097, 2, 5 * 1024 + 3, 1]])
def test_unscheduled_layers_anywhere(oracle, sizes, layerwise, adam):
    _run(oracle, sizes, 3, 4, "round_robin", adam, fused=True, layerwise=layerwise)


@pytest.mark.parametrize("n,chunks", [(9, 8191), (9, 8192), (16, 8192)])
def test_long_average(oracle, n, chunks):
    _run(oracle, [2048 * chunks - 1], n, 1, "every")
