"""Models (and layer ranges of larger ones) on both sides of the sizes that take the small models' chunks and residency, with default options: the four calls, the
fused step whole and layer by layer, dense and through the table.  Every element against the oracle, bit for bit."""
import pytest
import torch

from paper_2502_11058_amd import workloads as W
from test_gpu_parity import run_trajectory

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fused,layerwise", [(False, 0), (True, 0), (True, 1)])
@pytest.mark.parametrize("optimizer,dtype,n,wire16", [("sgdm", "f32", 3, False), ("adamw", "bf16", 9, True)])
@pytest.mark.parametrize("per_cu,more", [(1.25, 0), (1.25, 1), (4.5, 0), (4.5, 1), (6.0, 3)])
@pytest.mark.parametrize("whole", [True, False])      # layers that start on a vector (the table-free update of a range) or inside one
def test_both_sides_of_the_lines(oracle, whole, per_cu, more, optimizer, dtype, n, wire16, fused, layerwise):
    total = int(per_cu * torch.cuda.get_device_properties(0).multi_processor_count) * 2048 + more
    sizes = [4, 2052, total // 3 // 4 * 4, 1024] if whole else [5, 2051, total // 3, 1023]
    sizes.append(total - sum(sizes))
    ts = [W.TensorSpec(f"l{l}", l, k) for l, k in enumerate(sizes)]
    w = W.Workload(f"small{total}", ts, n_replicas=n, period=2, optimizer=optimizer, param_dtype=dtype, lr=1e-3, sigma_drift=1e-3, iterations=2,
                   policy="round_robin")
    for dense_path in (1, 0):
        assert run_trajectory(oracle, w, iters=2, fused=fused, wire16=wire16, layerwise=layerwise, options={"dense_path": dense_path}).frac() == 1.0
