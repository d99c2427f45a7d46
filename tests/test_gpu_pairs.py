"""Fused steps with many bf16 peers on both sides of the rule for two vectors in flight per thread (three scheduled chunks of at least
2048 elements per compute unit, in a call on 4.5): chunks with one vector per thread, with two and with three (two, then one), remainders of a
vector, a thread and a line; replica counts that have such kernels and those beside them; whole and by ranges of layers, which
may lie on the other side.  Every element against the oracle, bit for bit."""
import pytest
import torch

from paper_2502_11058_amd import workloads as W
from test_gpu_parity import run_trajectory

pytestmark = pytest.mark.gpu

SIZES = [3, 1021, 1024, 2044, 2048, 2051, 3 * 1024 + 1, 5 * 1024 + 64]


@pytest.mark.parametrize("optimizer,dtype,dense_path,layerwise", [("sgdm", "f32", 1, 0), ("adamw", "bf16", 1, 3), ("adamw", "bf16", 0, 0)])
@pytest.mark.parametrize("n,chunk", [(8, 2048), (9, 2048), (12, 3072), (16, 2048), (17, 3072), (24, 2048), (24, 1024), (31, 2048), (32, 2048), (33, 2048)])
@pytest.mark.parametrize("above", [False, True])
def test_vectors_in_flight(oracle, above, n, chunk, optimizer, dtype, dense_path, layerwise):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    ts = [W.TensorSpec(f"l{l}", l, k) for l, k in enumerate(SIZES + [cus * 9 // 2 * chunk - 5 if above else cus * 3 * chunk - 5 - sum(SIZES) - 9 * chunk])]
    w = W.Workload(f"pairs{n}", ts, n_replicas=n, period=1, optimizer=optimizer, param_dtype=dtype, lr=1e-3, sigma_drift=1e-3, iterations=1,
                   policy="every")
    options = {"update_chunk": chunk, "dense_path": dense_path}
    assert run_trajectory(oracle, w, iters=1, fused=True, wire16=True, layerwise=layerwise, options=options).frac() == 1.0
