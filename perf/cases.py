"""Performance cases: the work a user of this library has it do, through its public entry points.

Four ways in, as ``path`` names them:

``eager``       one all-reduce as two calls: the emulated peers write, then the reduction
                (``Sifar.produce`` + ``Sifar.reduce`` / ``Sifar.reduce_rmsnorm``)
``noalloc``     one all-reduce on the library's static scratch (``sifar_allreduce_noalloc``)
``graph``       one decode step of L chained all-reduces with ``persistent = 0``, the library's
                default: speculative validation, the peers one epoch ahead
``persistent``  one decode step with ``persistent = 1``: consumer waves against live peers

``epilogue`` adds the fused residual-add + RMSNorm, ``late`` is the probability that a rank's
stamp is late at an epoch (the stragglers of the speculation-stress and MoE workloads), ``wpg``
the handle's waves per workgroup. Values follow the workloads' recipe for decode activations.
"""
from __future__ import annotations

import numpy as np
import torch

import paper_2607_08973_amd as S

DEV = "cuda:0"
EPS = 1e-6
POOL_BYTES = 96 << 20   # a step's source pool: buffers that a serving program reuses


def _case(name, path, nranks, tokens, hidden, reduces=1, epilogue=0, late=0.0, wpg=1):
    c = dict(path=path, nranks=nranks, tokens=tokens, hidden=hidden, reduces=reduces,
             epilogue=epilogue, late=late, wpg=wpg)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one token's 8 KiB between two ranks, called by hand: host cost and launch latency
        _case("eager-n2-t1-h4096", "eager", 2, 1, 4096),
        # a prefill-sized block of 256 tokens, called by hand: memory bandwidth
        _case("eager-n8-t256-h8192", "eager", 8, 256, 8192),
        # a serving loop that must not allocate, at a batch of 16
        _case("noalloc-n8-t16-h4096", "noalloc", 8, 16, 4096),
        # the benchmark's decode step (dense 8B model, 32 layers x 2) at batch 1
        _case("persistent-n8-t1-h4096", "persistent", 8, 1, 4096, 64),
        # the same step at the largest batch the benchmark quotes
        _case("persistent-n8-t64-h4096", "persistent", 8, 64, 4096, 64),
        # odd batch and a hidden size of nine chunks
        _case("persistent-n8-t5-h4608", "persistent", 8, 5, 4608, 64),
        # the payload sweep's largest point
        _case("persistent-n8-t256-h8192", "persistent", 8, 256, 8192, 20),
        # the library's default configuration on the benchmark's shapes
        _case("graph-n8-t4-h4096", "graph", 8, 4, 4096, 64),
        # five ranks, ragged rows (the last chunk of a row is partly filled)
        _case("graph-n5-t64-h3896", "graph", 5, 64, 3896, 40),
        # MoE decode step (60 layers x 2) with the fused residual-add + RMSNorm
        _case("moe-persistent-n8-t8-h8192", "persistent", 8, 8, 8192, 120, epilogue=1),
        # the same through launches, at a batch of 32 with 5 % late stamps
        _case("moe-graph-n8-t32-h8192-late", "graph", 8, 32, 8192, 120, epilogue=1, late=0.05,
              wpg=4),
        # speculation stress: 10 % late stamps, so that a good third of the chunks retry
        _case("stress-graph-n8-t4-h4096-late", "graph", 8, 4, 4096, 64, late=0.1),
    ]


def _spread(rng, lo, hi):
    """A whole number of lo..hi, even over its logarithm."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    while True:
        path = rng.choice(["eager", "noalloc", "persistent", "persistent", "graph", "graph"])
        nranks = rng.choice([2, 4, 8, 8, rng.randint(1, 8)])
        # hidden sizes of models, and any multiple of the 8-element vector
        hidden = rng.choice([2048, 4096, 5120, 8192, 8 * _spread(rng, 64, 1024)])
        epilogue = int(path != "noalloc" and rng.random() < 0.3)
        tokens = _spread(rng, 1, {"noalloc": 64}.get(path, 32 if epilogue else 256))
        segs = (hidden + 511) // 512
        reduces = 1
        if path in ("graph", "persistent"):
            reduces = rng.choice([24, 64, 120]) if tokens <= 32 else 20
        late = 0.0
        if path in ("graph", "persistent") and rng.random() < 0.2:
            late = rng.choice([0.02, 0.05, 0.1])
        if path == "noalloc" and tokens * hidden > S.SIFAR_NOALLOC_MAX_ELEMS:
            continue
        if tokens * segs > (512 if epilogue else 4096):
            continue
        if nranks * tokens * hidden * reduces > 8 * 256 * 8192 * 20:
            continue  # no more than the largest listed case
        wpg = rng.choice([1, 4]) if epilogue and path != "persistent" else 1
        return _case(None, path, nranks, tokens, hidden, reduces, epilogue, late, wpg)


def _entries(case):
    """Source-pool entries: a divisor of the chain length (so that every step reads the same
    epochs' inputs), as many as the pool's budget holds, at least 4."""
    L = case["reduces"]
    one = case["nranks"] * case["tokens"] * case["hidden"] * 2
    fit = [d for d in range(1, L + 1) if L % d == 0 and d * one <= POOL_BYTES]
    return max(fit + [min(L, 4)])


def _inputs(case, seed):
    """The seeded inputs, on the GPU: decode activations N(0,1) * 0.5 with 0.1 % outliers x 50,
    a residual stream N(0,1) and a norm weight N(1, 0.02)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    N, T, H, E = case["nranks"], case["tokens"], case["hidden"], _entries(case)
    pool = torch.empty((E, N, T, H), dtype=torch.bfloat16, device=DEV)
    for e in range(E):
        x = torch.randn((N, T, H), generator=g, device=DEV) * 0.5
        out = torch.rand((N, T, H), generator=g, device=DEV) < 0.001
        pool[e] = torch.where(out, x * 50.0, x).to(torch.bfloat16)
    residual = torch.randn((T, H), generator=g, device=DEV).to(torch.bfloat16)
    weight = (1.0 + 0.02 * torch.randn((H,), generator=g, device=DEV)).to(torch.bfloat16)
    return pool, residual, weight


def _late_table(case, seed):
    r = np.random.default_rng([260708973, seed])
    bits = r.random((case["reduces"], case["nranks"])) < case["late"]
    return (bits * (1 << np.arange(case["nranks"]))).sum(axis=1).tolist()


def prepare(case, seed):
    N, T, H, L = case["nranks"], case["tokens"], case["hidden"], case["reduces"]
    pool, residual, weight = _inputs(case, seed)
    s = dict(case=case, pool=pool)
    if case["path"] == "noalloc":
        s["out"] = torch.zeros((T, H), dtype=torch.bfloat16, device=DEV)
        return s
    h = S.Sifar(nranks=N, hidden=H, max_tokens=T, reduces_per_step=L,
                validate="ordered" if case["path"] == "persistent" else "spec",
                persistent=int(case["path"] == "persistent"), epilogue=case["epilogue"],
                rms_eps=EPS, waves_per_group=case["wpg"], log_epochs=L)
    s["handle"] = h
    if case["epilogue"]:
        s.update(residual0=residual, residual=residual.clone(), weight=weight)
    out = torch.zeros((T, H) if case["path"] == "eager" else (L, T, H), dtype=torch.bfloat16,
                      device=DEV)
    s["out"] = out
    if case["path"] != "eager":
        if case["epilogue"]:
            h.bind_step(pool, residual=s["residual"], weight=weight, y_ring=out)
        else:
            h.bind_step(pool, out_ring=out)
        if case["late"]:
            h.set_injection(_late_table(case, seed))
    return s


def run(s):
    case = s["case"]
    T = case["tokens"]
    if case["path"] == "noalloc":
        pool = s["pool"]
        S.sifar_allreduce_noalloc(pool, pool.stride(1), case["nranks"], T, case["hidden"], s["out"])
        return s["out"]
    h = s["handle"]
    if case["epilogue"]:
        s["residual"].copy_(s["residual0"])  # the step's input: the tokens' embeddings
    if case["path"] == "eager":
        h.produce(s["pool"][0], T)
        if case["epilogue"]:
            h.reduce_rmsnorm(s["residual"], s["weight"], s["out"], T)
        else:
            h.reduce(s["out"], T)
    else:
        h.step(T)
    return (s["out"], s["residual"]) if case["epilogue"] else s["out"]


def work(case):
    """Per all-reduce: every rank's partial read, the sum written. With the epilogue the sum is
    not stored: y is; the residual is read and written once a pass, the weight read once."""
    N, K, L = case["nranks"], case["tokens"] * case["hidden"], case["reduces"]
    moved = L * (N + 1) * K * 2
    flops = L * (N - 1) * K
    if case["epilogue"]:
        moved += 2 * K * 2 + case["hidden"] * 2
        flops += L * 6 * K
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    """The sum's order and rounding are part of the contract: bit-exact, and so is the residual
    stream. The normalised output may differ where the fp32 sum of squares is added in another
    order: by one bf16 step (2^-7 of the value at most), at few elements."""
    if not case["epilogue"]:
        return "exact"
    return {"rel": 1e-4, "max": 0.0079}


def exact(case, seed):
    """The first pass in float64: no rounding between the all-reduces of a chain."""
    pool, residual, weight = _inputs(case, seed)
    E, L = pool.shape[0], case["reduces"]
    sums = torch.stack([pool[e].double().sum(0) for e in range(E)])
    if not case["epilogue"]:
        out = sums[torch.arange(L, device=DEV) % E]
        return out if case["path"] in ("graph", "persistent") else out[0]
    res, w, ys = residual.double(), weight.double(), []
    for i in range(L):
        res = res + sums[i % E]
        ys.append(res * w / torch.sqrt((res * res).mean(-1, keepdim=True) + EPS))
    return (torch.stack(ys) if case["path"] != "eager" else ys[0], res)
