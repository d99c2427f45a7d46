"""Streams that lie differently against their own vectors: every stream of every tensor has a start of its own (fp32 at any
multiple of 4 bytes, bf16 at any multiple of 2), and the flat offsets of the slot are odd too.  The vector accesses of the
table-driven kernels then start at any element.  Every element against the oracle, bit for bit, and no element outside the
tensors touched."""
import numpy as np
import pytest
import torch

from paper_2502_11058_amd import binding as B

pytestmark = pytest.mark.gpu

LAYERS = [[1021, 5], [1], [2047, 2050], [4099, 3], [6151, 7]]     # below, at and above one and several chunks of 1024


def _bits(t):
    return t.detach().cpu().view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32).numpy()


OWN = {"update_chunk": 1024, "mean_chunk": 1024}


@pytest.mark.parametrize("starts", [(0, 0, 0, 1, 1), (1, 2, 3, 1, 2), (3, 0, 1, 3, 0), (2, 1, 0, 2, 3)])
@pytest.mark.parametrize("adam,bf16,n_replicas,wire16", [(True, True, 2, False), (True, True, 5, True), (False, False, 8, True),
                                                         (False, True, 17, False), (True, False, 40, True)])
def test_every_stream_at_its_own_offset(oracle, starts, adam, bf16, n_replicas, wire16):
    _run(oracle, LAYERS, starts, adam, bf16, n_replicas, wire16, OWN)


# several tensors a layer around one and two of the halves of 1024 elements that the fused step takes by default, less where a line starts
HALVES = [[1024, 960, 1023], [1025, 64], [1024 - 61, 2048 - 16, 2048], [2049, 1, 3 * 1024 - 3, 5], [4096 + 61, 2 * 1024 + 7]]


@pytest.mark.parametrize("starts", [(0, 0, 0, 1, 1), (1, 2, 3, 1, 2), (3, 0, 1, 3, 0), (2, 1, 0, 2, 3)])
@pytest.mark.parametrize("bf16,n_replicas,wire16", [(False, 2, False), (True, 3, True), (False, 6, False), (False, 12, True), (True, 17, False), (True, 32, True), (False, 40, True)])
def test_default_chunks_at_their_own_offsets(oracle, starts, bf16, n_replicas, wire16):
    _run(oracle, HALVES, starts, False, bf16, n_replicas, wire16, {})


@pytest.mark.parametrize("starts", [(1, 2, 3, 1, 2), (2, 1, 0, 2, 3)])
@pytest.mark.parametrize("bf16,n_replicas,wire16", [(True, 5, False), (True, 16, True), (False, 32, False)])
def test_default_chunks_with_a_second_moment(oracle, starts, bf16, n_replicas, wire16):
    _run(oracle, HALVES + [[2_400_001, 1021]], starts, True, bf16, n_replicas, wire16, {})     # (past the small models)


def _run(oracle, layers, starts, adam, bf16, n_replicas, wire16, options):
    assert torch.cuda.is_available(), "no GPU visible"
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(n_replicas)
    layer_of = [l for l, ns in enumerate(layers) for _ in ns]
    numel = [n for ns in layers for n in ns]
    half = torch.bfloat16 if bf16 else torch.float32
    names = ["sync", "s0", "s1", "grad", "model"]
    dtypes = [torch.float32, torch.float32, torch.float32, half, torch.bfloat16]
    arena, views = {}, {}
    for name, dt, first in zip(names, dtypes, starts):
        at, pos = [], 0
        for j, n in enumerate(numel):            # each tensor somewhere else, a stretch that nobody owns in between
            pos = (pos + 15) // 16 * 16 + 16 + (first + j) % 4
            at.append(pos)
            pos += n
        arena[name] = torch.empty(pos + 32, dtype=torch.float32, device=dev).normal_(0.0, 1e-3, generator=g).to(dt)
        views[name] = [arena[name][a:a + n] for a, n in zip(at, numel)]
    if not bf16:
        views["model"] = None
    for x in views["s0"] + views["s1"]:
        x.zero_()
    if bf16:
        for a, b in zip(views["model"], views["sync"]):
            a.copy_(b)
    before = {k: v.clone() for k, v in arena.items()}
    sets = [[4, 2, 0], list(range(5, len(layers))) + [3, 1]]
    hyper = dict(lr=1e-2, momentum=0.9, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1)
    wk = oracle.Worker(layer_of, [x.cpu().numpy() for x in views["sync"]], "adamw" if adam else "sgdm", hyper, bf16)
    ctx = B.Context(0)
    for k, v in options.items():
        ctx.ddp_set_option(k, v)
    ctx.ddp_register_model(len(layers), layer_of, numel, B.DDP_BF16 if bf16 else B.DDP_F32, B.DDP_BF16 if bf16 else B.DDP_F32, views["sync"],
                           views["model"], views["grad"], views["s0"], views["s1"] if adam else None)
    ctx.ddp_set_schedule(*B.csr_from_sets(sets))
    host = lambda t: t.view(torch.int16).cpu().numpy().view(np.uint16) if t.dtype == torch.bfloat16 else t.cpu().numpy()  # noqa: E731
    stats = torch.zeros(2 * len(layers), dtype=torch.float64, device=dev)
    for r in range(2):
        S, rank = sets[r], (7 * r + 1) % n_replicas
        flat = torch.cat([views["sync"][t] for l in S for t in range(len(numel)) if layer_of[t] == l])
        peers = [flat + torch.empty_like(flat).normal_(0.0, 1e-3, generator=g) for _ in range(n_replicas - 1)]
        if wire16:
            peers = [p.bfloat16() for p in peers]
        opt = B.make_opt("adamw" if adam else "sgdm", hyper["lr"], r + 1, momentum=0.9, weight_decay=0.1)
        if wire16:
            ctx.ddp_fused_sync_update_wire16(r, peers, n_replicas, rank, stats, opt)
        else:
            ctx.ddp_fused_sync_update(r, peers, n_replicas, rank, stats, opt)
        _, ref = wk.sync(S, [host(p) for p in peers], rank, wire16=wire16)
        wk.local_update([host(x) for x in views["grad"]], r + 1)
        got = stats.cpu().numpy()
        for i, (gam, msq) in enumerate(ref):
            assert got[2 * i] == pytest.approx(gam, rel=1e-10) and got[2 * i + 1] == pytest.approx(msq, rel=1e-10)
    opt = B.make_opt("adamw" if adam else "sgdm", hyper["lr"], 3, momentum=0.9, weight_decay=0.1)
    ctx.ddp_local_update(opt)
    wk.local_update([host(x) for x in views["grad"]], 3)
    refs = {"sync": wk.p, "s0": wk.s0, "s1": wk.s1 if adam else None, "model": wk.model if bf16 else None}
    for name, ref in refs.items():
        if ref is None:
            continue
        for t, b in enumerate(ref):
            want = b.view(np.int16) if b.dtype == np.uint16 else b.view(np.int32)
            assert np.array_equal(_bits(views[name][t]), want), (name, t)
    for name in names:                            # what lies between the tensors is as it was
        mask = torch.ones(arena[name].numel(), dtype=torch.bool, device=dev)
        for x in views[name] or []:
            o = x.storage_offset()
            mask[o:o + x.numel()] = False
        assert np.array_equal(_bits(arena[name][mask]), _bits(before[name][mask])), name
    ctx.close()
