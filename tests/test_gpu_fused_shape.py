"""The fused step's chunks of 1024 elements, the update's and the unscheduled pieces' of two of them, with default options: layers around
one and several of both, and statistics of up to and beyond 5/2 workgroups per CU with a pair; the four calls and the fused step, whole
and layer by layer, dense and through the table.  Every element against the oracle, bit for bit, statistics to 1e-10."""
import pytest

from paper_2502_11058_amd import workloads as W
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
