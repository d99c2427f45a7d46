"""Unscheduled layers that start anywhere in a vector, called layer by layer and in ranges, updates of ranges alone, and averages of 9 to 16 replicas on both sides
of the line where the two sums of a launch are formed one after the other (8192 chunks): every element against the oracle, bit for bit,
statistics to 1e-10."""
import pytest
import torch

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


@pytest.mark.parametrize("options", [{}, {"nontemporal": 0}, {"update_chunk": 1024}])
@pytest.mark.parametrize("adam", [False, True])
@pytest.mark.parametrize("layers", [1, 2, 3])
@pytest.mark.parametrize("sizes", [[1, 1023, 2, 2047, 3, 2049, 61, 64], [3 * 2048 + 1, 509 * 510, 127, 65, 4097, 2, 5 * 1024 + 3, 600_001]])
def test_update_ranges_anywhere(sizes, layers, adam, options):
    """The local update range by range, starting anywhere in a vector, table-free: the bits of the whole model's through the table, which
    test_gpu_parity has against the oracle."""
    from paper_2502_11058_amd.harness import DeviceReplica
    assert torch.cuda.is_available(), "no GPU visible"
    ts = [W.TensorSpec(f"l{l}", l, k) for l, k in enumerate(sizes)]
    w = W.Workload(f"ranges{len(sizes)}_{sizes[0]}", ts, n_replicas=2, period=1, optimizer="adamw" if adam else "sgdm", param_dtype="bf16" if adam else "f32",
                   lr=1e-3, policy="every")
    reps = [DeviceReplica(w, 0, options=dict(options, dense_path=d)) for d in (0, 1)]
    for rep in reps:
        rep.init_params()
    for r in range(2):
        for rep in reps:
            rep.fill_grads(r)
        reps[0].ctx.ddp_local_update(reps[0].opt_struct(r + 1))
        for lo in range(0, len(sizes), layers):
            reps[1].ctx.ddp_local_update_layers(lo, min(layers, len(sizes) - lo), reps[1].opt_struct(r + 1))
    for name in ("a_sync", "a_s0", "a_s1", "a_model"):
        a, b = getattr(reps[0], name), getattr(reps[1], name)
        assert a is None or torch.equal(a.view(torch.int16), b.view(torch.int16)), name
    for rep in reps:
        rep.close()
