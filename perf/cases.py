"""Workloads that the step's performance is measured on, each through the framework's public entry points.

A case is one worker of one job: the model (shapes of the repository's own configurations, or generic ones of the same
families), the number of replicas, the schedule, the optimizer, the precision of the model and of the exchange, and the way
the iteration is called.  One pass is one iteration of that worker with the gradients and the peers' buffers already in
HBM:

    four      DeviceReplica.step: ddp_pack, ddp_partial_average, ddp_unpack, ddp_local_update (or the bf16-wire forms)
    fused     DeviceReplica.fused_step, or Context.ddp_fused_sync_update[_wire16] on tensors of the caller's own
    layers    one Context.ddp_fused_sync_update_layers call per layer in backward order, as the autograd hooks make them
    average   Context.ddp_partial_average alone, what a worker runs that exchanges and averages without stepping

`arenas` says how the tensors lie: "dense" is the framework's own slab (every stream one flat arena), "separate" gives every
tensor a start of its own at a multiple of 512 bytes and something else in between, as a caching allocator places tensors
that were created one by one.
"""
from __future__ import annotations

import math

import torch

from paper_2502_11058_amd import binding as B
from paper_2502_11058_amd import workloads as W
from paper_2502_11058_amd.harness import DeviceReplica

# Common values, overridden by the cases.  `iteration` is in the middle of a run: the moments hold earlier gradients, and
# the slot that is synchronised is iteration mod period.
_DEFAULT = {"replicas": 8, "period": 4, "policy": "enp", "iteration": 1001, "rank": 0, "optimizer": "sgdm", "dtype": "f32",
            "call": "four", "wire": "f32", "stats": True, "arenas": "dense"}


def _case(**kw):
    return dict(_DEFAULT, **kw)


def _mlp(layers, width):
    return {"family": "mlp", "layers": layers, "width": width}


def _gpt2(blocks, d, vocab=50257, context=1024, biases=False):
    return {"family": "gpt2", "layers": blocks, "width": d, "vocab": vocab, "context": context, "biases": biases}


def _llama(blocks, d, ffn, vocab, kv):
    return {"family": "llama", "layers": blocks, "width": d, "ffn": ffn, "vocab": vocab, "kv": kv}


def listed():
    adam = {"optimizer": "adamw", "dtype": "bf16"}
    return [
        # the smallest configuration (8 layers of 256 x 256, 4 workers): every call is a handful of microseconds, so launches
        # and latency are what a user waits for; both ways to call an iteration
        _case(name="tiny_four", **_mlp(8, 256), replicas=4),
        _case(name="tiny_fused", **_mlp(8, 256), replicas=4, call="fused"),
        # a small network whose sizes are no multiples of anything (one odd bias shifts everything behind it), driven layer by
        # layer from backward hooks: many short calls
        _case(name="ragged_mlp_layers", **_mlp(8, 509), replicas=5, call="layers"),
        # the same kind of network larger, in mixed precision, all of it in one call
        _case(name="ragged_mlp_fused", **_mlp(16, 1533), replicas=8, call="fused", **adam),
        # GPT-2 small as configured (fp32, SGD with momentum, 8 workers): the four calls on the framework's slab
        _case(name="gpt2_four", **_gpt2(12, 768)),
        # the same model with biases and its final norm as an ordinary program holds it: tensors allocated one by one
        _case(name="gpt2_separate_fused", **_gpt2(12, 768, biases=True), call="fused", arenas="separate"),
        # the same in mixed precision with half the bytes on the wire, layer by layer from backward hooks
        _case(name="gpt2_layers_wire16", **_gpt2(12, 768), call="layers", wire="bf16", **adam),
        # a worker of the paper's largest cluster (32) and a mid-size network, bf16 on the wire, four calls
        _case(name="mlp_32_workers_wire16", **_mlp(12, 1536), replicas=32, wire="bf16"),
        # TinyLlama-1.1B as configured, four calls and with bf16 peers through the fused call
        _case(name="tinyllama_four", **_llama(22, 2048, 5632, 32000, 4), **adam),
        _case(name="tinyllama_fused_wire16", **_llama(22, 2048, 5632, 32000, 4), call="fused", wire="bf16", **adam),
        # averaging alone: one block of Llama-3-8B and its 16 workers
        _case(name="llama3_block_average", **_llama(2, 4096, 14336, 16000, 8), replicas=16, call="average", **adam),
        # the largest: blocks, embedding and head of Llama-2-7B (a quarter of its depth), fused
        _case(name="llama2_blocks_fused", **_llama(8, 4096, 11008, 32000, 32), call="fused", **adam),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        family = rng.choice(["mlp", "mlp", "gpt2", "llama"])
        if family == "mlp":
            m = _mlp(rng.randint(3, 16), _log_int(rng, 128, 4096) + rng.choice([0, 1]))
        elif family == "gpt2":
            m = _gpt2(rng.randint(2, 16), 64 * _log_int(rng, 2, 24), vocab=_log_int(rng, 1000, 50257), context=rng.choice([256, 512, 1024]),
                      biases=rng.random() < 0.5)
        else:
            d = 128 * _log_int(rng, 2, 32)
            m = _llama(rng.randint(2, 22), d, 16 * int(d * rng.uniform(2.5, 3.6) / 16), _log_int(rng, 1000, 32000), rng.choice([4, 8, 32]))
        n = rng.choice([2, 3, 4, 5, 6, 8, 8, 12, 16, 24, 32])
        c = _case(**m, replicas=n, period=rng.choice([2, 4, 4, 8]), policy=rng.choice(["enp", "enp", "round_robin"]),
                  iteration=rng.randint(100, 20000), rank=rng.randrange(n), call=rng.choice(["four", "four", "fused", "fused", "layers", "average"]),
                  wire=rng.choice(["f32", "f32", "bf16"]), stats=rng.random() < 0.85, arenas=rng.choice(["dense", "dense", "separate"]))
        if rng.random() < (0.8 if family == "llama" else 0.4):
            c.update(optimizer="adamw", dtype="bf16")
        if c["call"] == "average" and c["wire"] == "bf16":
            c["wire"] = "f32"
        if 3e6 < work(c)["bytes"] < 6e10 and _state_bytes(c) < 4.5e10:
            return c


# ---- shapes ---------------------------------------------------------------------------------------------------------

def _workload(case):
    """The framework's description of the job, from the dimensions of the case."""
    f, name = case["family"], "case"
    adam = case["optimizer"] == "adamw"
    cfg = {"family": f, "n_replicas": case["replicas"], "period": case["period"], "optimizer": case["optimizer"], "param_dtype": case["dtype"],
           "lr": 3e-4 if adam else 0.01, "weight_decay": 0.1, "policy": case["policy"], "sigma_drift": 1e-4 if adam else 1e-3,
           "sigma_grad": 1e-3 if adam else 1e-2}
    if f == "mlp":
        cfg.update(n_layers=case["layers"], width=case["width"])
    elif f == "gpt2":
        cfg.update(n_blocks=case["layers"], d=case["width"], ffn=4 * case["width"], vocab=case["vocab"], context=case["context"])
    else:
        cfg.update(n_blocks=case["layers"], d=case["width"], ffn=case["ffn"], vocab=case["vocab"], n_heads=32, n_kv=case["kv"])
    return W.from_config(name, cfg, with_biases=bool(case.get("biases")))


def _slot_layers(case, n_layers):
    """The layers that the schedule synchronises in this iteration, in backward order."""
    H = case["period"]
    slot = case["iteration"] % H
    if case["policy"] == "round_robin":
        return [l for l in range(n_layers - 1, -1, -1) if l % H == slot]
    base, extra = divmod(n_layers, H)                       # equal numbers, the remainder to the earliest slots
    first = slot * base + min(slot, extra)
    return [n_layers - 1 - i for i in range(first, first + base + (slot < extra))]


def _layout(case):
    """(numel, layer of each tensor, start of each tensor in its arena, arena length, tensors of the slot in flat order,
    layers of the slot)"""
    w = _workload(case)
    numel, layer = [t.numel for t in w.tensors], [t.layer for t in w.tensors]
    starts, pos = [], 0
    for n in numel:
        starts.append(pos)
        pos += n if case["arenas"] == "dense" else -(-n // 256) * 256 + 256      # 256 bf16 elements = 512 bytes
    layers = _slot_layers(case, w.n_layers)
    order = [t for l in layers for t in range(len(numel)) if layer[t] == l]
    return numel, layer, starts, pos, order, layers


def work(case):
    numel, _, _, _, order, _ = _layout(case)
    P, S, N = sum(numel), sum(numel[t] for t in order), case["replicas"]
    wire = 2 if case["wire"] == "bf16" else 4
    model = 2 if case["dtype"] == "bf16" else 0
    step = (2 if model else 4) + (24 if case["optimizer"] == "adamw" else 16) + model        # gradient, parameter and moments, model copy
    flops_step = 16 if case["optimizer"] == "adamw" else 4
    flops_mean = N + (3 * N + 2 if case["stats"] else 0)
    if case["call"] == "average":
        return {"bytes": 4.0 * (N + 1) * S, "flops": float(flops_mean * S)}
    if case["call"] == "four":       # what each of the four calls takes and gives
        b = (4 + wire) * S + (wire * N + 4) * S + (8 + model) * S + step * P
    else:
        b = wire * (N - 1) * S + step * P
    return {"bytes": float(b), "flops": float(flops_mean * S + flops_step * P)}


def _state_bytes(case):
    numel, _, _, arena, order, _ = _layout(case)
    S = max(sum(numel[t] for t in order), 1)
    per = 4 * (3 if case["optimizer"] == "adamw" else 2) + (4 if case["dtype"] == "bf16" else 4)
    return per * arena + (6 if case["wire"] == "bf16" else 4) * case["replicas"] * 2 * S


# ---- inputs ---------------------------------------------------------------------------------------------------------

def _arenas(case):
    names = [("sync", torch.float32), ("s0", torch.float32)]
    if case["optimizer"] == "adamw":
        names.append(("s1", torch.float32))
    names.append(("grad", torch.bfloat16 if case["dtype"] == "bf16" else torch.float32))
    if case["dtype"] == "bf16":
        names.append(("model", torch.bfloat16))
    return names


def _normal(out, sigma, seed):
    """N(0, sigma^2) draws in pieces, made in fp32 and rounded to the tensor's type."""
    g = torch.Generator(device=out.device)
    g.manual_seed(seed & ((1 << 62) - 1))
    if out.dtype == torch.float32:
        out.normal_(0.0, sigma, generator=g)
        return
    for piece in out.split(1 << 27):
        piece.copy_(torch.empty(piece.shape, dtype=torch.float32, device=out.device).normal_(0.0, sigma, generator=g))


def _fill(case, seed, a, peers):
    """Parameters, moments in the middle of a run, gradients; peers[k]: the slot's parameters plus their drift."""
    numel, _, starts, _, order, _ = _layout(case)
    adam = case["optimizer"] == "adamw"
    sg = 1e-3 if adam else 1e-2
    _normal(a["sync"], 0.02, 101 * seed + 1)
    _normal(a["grad"], sg, 101 * seed + 2)
    _normal(a["s0"], 0.3 * sg if adam else 3.0 * sg, 101 * seed + 3)
    if adam:
        _normal(a["s1"], sg, 101 * seed + 4)
        a["s1"].square_()
        a["s1"].add_(1e-4 * sg * sg)
    if case["arenas"] == "separate":             # nothing lies between the tensors
        for x in a.values():
            for n, s, e in zip(numel, starts, starts[1:] + [x.numel()]):
                x[s + n:e].zero_()
    if case["dtype"] == "bf16":
        a["model"].copy_(a["sync"])
    flat = torch.cat([a["sync"][starts[t]:starts[t] + numel[t]] for t in order]) if order else a["sync"][:0]
    tmp = torch.empty_like(flat)
    for k, p in enumerate(peers):
        _normal(tmp, 1e-4 if adam else 1e-3, 101 * seed + 10 + k)
        p[:flat.numel()].copy_(tmp.add_(flat))
    return flat


class _Own:
    """A worker on tensors that the program allocated itself, registered with the binding."""

    def __init__(self, case, w):
        numel, layer, starts, arena, order, _ = _layout(case)
        dev = torch.device("cuda")
        self.a = {n: torch.zeros(arena, dtype=t, device=dev) for n, t in _arenas(case)}
        views = {n: [x[s:s + k] for s, k in zip(starts, numel)] for n, x in self.a.items()}
        self.w = w
        sets = [_slot_layers(dict(case, iteration=s), w.n_layers) for s in range(case["period"])]
        lay = w.layer_numel()
        S = max(max(sum(lay[l] for l in s) for s in sets), 4)
        t16 = torch.bfloat16 if case["wire"] == "bf16" else torch.float32
        self.flat = torch.zeros(S, dtype=torch.float32, device=dev)
        self.flat16 = torch.zeros(S, dtype=t16, device=dev) if case["wire"] == "bf16" else None
        self.peers = self.peers16 = [torch.zeros(S, dtype=t16, device=dev) for _ in range(case["replicas"] - 1)]
        self._peers_arr = self._peers16_arr = B.device_pointer_array(self.peers)
        self.stats = torch.zeros(2 * w.n_layers + 2, dtype=torch.float64, device=dev)
        self.ctx = B.Context(dev.index or 0)
        bf = B.DDP_BF16 if case["dtype"] == "bf16" else B.DDP_F32
        self.ctx.ddp_register_model(w.n_layers, layer, numel, bf, bf, views["sync"], views.get("model"), views["grad"], views["s0"], views.get("s1"))
        self.ctx.ddp_set_schedule(*B.csr_from_sets(sets))
        self.sets = sets

    def opt_struct(self, step):
        w = self.w
        return B.make_opt(w.optimizer, w.lr, step, momentum=w.momentum, beta1=w.beta1, beta2=w.beta2, eps=w.eps, weight_decay=w.weight_decay)

    step, fused_step = DeviceReplica.step, DeviceReplica.fused_step


def prepare(case, seed):
    w = _workload(case)
    if case["arenas"] == "dense":
        rep = DeviceReplica(w, 0, placement_probe=False, wire16=case["wire"] == "bf16")
        a = {"sync": rep.a_sync, "s0": rep.a_s0, "s1": rep.a_s1, "grad": rep.a_grad, "model": rep.a_model}
        a = {n: a[n] for n, _ in _arenas(case)}
    else:
        rep = _Own(case, w)
        a = rep.a
    peers = rep.peers16 if case["wire"] == "bf16" else rep.peers
    flat = _fill(case, seed, a, peers)
    rep.flat[:flat.numel()].copy_(flat)
    _, _, _, _, order, layers = _layout(case)
    assert list(rep.sets[case["iteration"] % case["period"]]) == layers
    S = flat.numel()
    out = [a[n] for n, _ in _arenas(case) if n != "grad"]
    if case["call"] == "average":
        out = []
    if case["call"] in ("four", "average"):
        out.append(rep.flat[:S])
    if case["call"] == "four" and case["wire"] == "bf16":
        out.append(rep.flat16[:S])
    if case["stats"] and layers:
        out.append(rep.stats[:2 * len(layers)])
    return {"case": case, "rep": rep, "out": out, "peers": peers, "stats": rep.stats if case["stats"] else None}


def run(state):
    case, rep = state["case"], state["rep"]
    r, rank, wire16 = case["iteration"], case["rank"], case["wire"] == "bf16"
    if case["call"] == "four":
        rep.step(r, rank, case["stats"], wire16=wire16)
    elif case["call"] == "fused":
        rep.fused_step(r, rank, case["stats"], wire16=wire16)
    elif case["call"] == "average":
        rep.ctx.ddp_partial_average(r % case["period"], rep.flat, rep._peers_arr, case["replicas"], rank, rep.flat, state["stats"])
    else:
        opt = rep.opt_struct(r + 1)
        for l in range(rep.w.n_layers - 1, -1, -1):
            rep.ctx.ddp_fused_sync_update_layers(r % case["period"], l, 1, state["peers"], B.DDP_BF16 if wire16 else B.DDP_F32,
                                                 B.DDP_SYNC_THEN_UPDATE, case["replicas"], rank, state["stats"], opt)
    return state["out"]


# ---- what the results are compared with ------------------------------------------------------------------------------

def tolerance(case):
    """fp32 results lie up to 6.2e-8 (2-norm) from the 64-bit ones; a bf16 model copy rounded from a parameter that is off
    by that much differs from the unperturbed one by 1.5e-5 in the 2-norm, by one unit in the last place (7.4e-3 at most) where it differs.
    Four times the norms."""
    return {"rel": 2.5e-7} if case["dtype"] == "f32" else {"rel": 6e-5, "max": 8e-3}


def exact(case, seed):
    """The iteration in 64 bits (bf16 exchange: the mean of the rounded values, which is what that form defines)."""
    numel, _, starts, arena, order, layers = _layout(case)
    dev = torch.device("cuda")
    a = {n: torch.zeros(arena, dtype=t, device=dev) for n, t in _arenas(case)}
    S, N, rank = sum(numel[t] for t in order), case["replicas"], case["rank"]
    wire16 = case["wire"] == "bf16"
    peers = [torch.empty(max(S, 1), dtype=torch.bfloat16 if wire16 else torch.float32, device=dev) for _ in range(N - 1)]
    local = _fill(case, seed, a, peers)
    if wire16:
        local16 = local.bfloat16()
        local = local16
    xs = peers[:rank] + [local] + peers[rank:]
    f32 = lambda v: float(torch.tensor(v, dtype=torch.float32))  # noqa: E731  (the options are stated in fp32)
    mean = torch.zeros(S, dtype=torch.float64, device=dev)
    for x in xs:
        mean += x[:S]
    mean /= N
    stats, pos = [], 0
    layer_numel = _workload(case).layer_numel()
    for l in layers:
        m = mean[pos:pos + layer_numel[l]]
        stats += [sum(float((m - x[pos:pos + layer_numel[l]]).square_().sum()) for x in xs) / N, float(m.square().sum())]
        pos += layer_numel[l]
    stats = torch.tensor(stats, dtype=torch.float64)
    out = []
    if case["call"] != "average":
        p = a.pop("sync").double()
        pos = 0
        for t in order:
            p[starts[t]:starts[t] + numel[t]] = mean[pos:pos + numel[t]]
            pos += numel[t]
        g = a.pop("grad")
        if case["optimizer"] == "sgdm":
            s0 = a.pop("s0").double().mul_(f32(0.9)).add_(g)
            p.sub_(s0, alpha=f32(0.01))
            out = [p, s0]
        else:
            b1, b2, lr, wd, eps, t = f32(0.9), f32(0.95), f32(3e-4), f32(0.1), f32(1e-8), case["iteration"] + 1
            g = g.double()
            s0 = a.pop("s0").double().mul_(b1).add_(g, alpha=1 - b1)
            s1 = a.pop("s1").double().mul_(b2).add_(g.square_(), alpha=1 - b2)
            g = torch.sqrt(s1).div_(math.sqrt(1 - b2 ** t)).add_(eps)
            p.mul_(1 - lr * wd).sub_((s0 / g).mul_(lr / (1 - b1 ** t)))
            out = [p, s0, s1]
        if case["dtype"] == "bf16":
            out.append(p)
    if case["call"] in ("four", "average"):
        out.append(mean)
    if case["call"] == "four" and wire16:
        out.append(local16)
    if case["stats"] and layers:
        out.append(stats)
    return out
