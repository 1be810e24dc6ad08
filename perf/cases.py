"""The expert stage and the combine as a program calls them, over the sizes they are used at.

A stage case is one expert-parallel rank's pass: routed token copies of `ranks` source ranks
(`tokens` each, top-`k` of `experts * ranks` experts) that were dispatched to this rank's `experts`
local experts go through the gated FFN and come back in one buffer per source rank, the region of
that rank's receive buffer this owner fills (with room to spare).  `entry` names the call:

  run              overlapped stage, plan built on the host (routing in host arrays)
  run_devplan      overlapped stage, plan built on the GPU (routing in device tensors)
  serial           expert compute, then the whole return copy, host-built plan
  serial_devplan   the same with the plan built on the GPU
  serial_static    the same without a handle (callers that cannot allocate)
  combine          the weighted reduction of a source rank's returned rows

The overlapped calls run on a stream of their own, with the consumer beside the producer on 64
compute units; the others run on the current stream.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2607_19539_amd import binding as B

# hidden, ffn, local experts, source ranks, choices per token, router, tokens per rank at full size
FAMILIES = {
    "tiny": (256, 512, 2, 4, 2, "uniform", 64),
    "ragged": (320, 576, 2, 4, 2, "uniform", 200),
    "mixtral": (4096, 14336, 2, 4, 2, "uniform", 4096),
    "mixtral_zipf": (4096, 14336, 2, 4, 2, "zipf", 4096),
    "fine": (2048, 1408, 16, 4, 6, "bias", 8192),
    "large_fine": (7168, 2048, 32, 8, 8, "uniform", 4096),
    "layer_e4": (1024, 4096, 4, 4, 2, "uniform", 8192),
    "layer_e16": (1024, 4096, 16, 4, 2, "uniform", 8192),
    "layer_e64": (1024, 4096, 64, 4, 2, "uniform", 8192),
}
SELF_RANK = 0
WEIGHT_STD = 0.02
ZIPF_S = 1.2
CU_SPLIT = 64


def _stage(name, family, entry, tokens):
    H, F, E, R, k, router, _ = FAMILIES[family]
    return {"name": name, "kind": "stage", "entry": entry, "hidden": H, "ffn": F, "experts": E, "ranks": R, "k": k,
            "router": router, "tokens": tokens}


def _combine(name, hidden, tokens, k):
    return {"name": name, "kind": "combine", "entry": "combine", "hidden": hidden, "tokens": tokens, "k": k}


def listed():
    return [
        # The smallest call: a few hundred rows of a small model, inside a loop that may not allocate.
        _stage("tiny_static", "tiny", "serial_static", 64),
        # Sizes that fill no tile: hidden and ffn that are multiples of 64 only, ragged experts.
        _stage("ragged_small", "ragged", "serial", 200),
        # Decoding: a handful of rows per expert, so the pass is a read of the weights.
        _stage("mixtral_decode", "mixtral", "serial_devplan", 16),
        _stage("large_fine_decode", "large_fine", "run_devplan", 32),
        # A chunk of a prefill beside decoding: some hundred rows per expert, an odd number of tokens.
        _stage("fine_chunk", "fine", "run", 777),
        # Full prefill batches of the measured workloads.
        _stage("fine", "fine", "run", 8192),
        _stage("large_fine", "large_fine", "run_devplan", 4096),
        _stage("mixtral", "mixtral", "run", 4096),
        # The rank that owns the hot experts of a skewed router, without overlap.
        _stage("mixtral_zipf", "mixtral_zipf", "serial", 4096),
        # The widest point of the expert-count sweep: about one tile row per expert.
        _stage("layer_e64", "layer_e64", "serial", 8192),
        # The reduction on the source rank after a decode step and after a prefill batch.
        _combine("combine_decode", 7168, 48, 8),
        _combine("combine", 4096, 4096, 2),
    ]


def draw(rng):
    if rng.random() < 0.15:
        hidden = rng.choice([256, 320, 1024, 2048, 4096, 7168])
        tokens = int(round(math.exp(rng.uniform(math.log(3), math.log(8192)))))
        c = _combine("", hidden, tokens, rng.randint(1, 8))
    else:
        family = rng.choice(sorted(FAMILIES))
        entries = ["run", "run_devplan", "serial", "serial_devplan"]
        if family in ("tiny", "ragged"):
            entries.append("serial_static")
        full = FAMILIES[family][6]
        tokens = int(round(math.exp(rng.uniform(math.log(5), math.log(full)))))
        c = _stage("", family, rng.choice(entries), tokens)
    del c["name"]
    return c


# ------------------------------------------------------------------------------------ inputs

def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + stream) & 0x7FFFFFFFFFFF)
    return g


def _zipf_p(n):
    p = [(e + 1) ** -ZIPF_S for e in range(n)]
    return [v / sum(p) for v in p]


def _router_logits(case, seed):
    R, T, E_t = case["ranks"], case["tokens"], case["experts"] * case["ranks"]
    u = torch.rand((R, T, E_t), generator=_gen(seed, 1), device="cuda")
    if case["router"] == "uniform":
        return u
    if case["router"] == "zipf":  # Gumbel top-k: k distinct experts, popular ones first
        return torch.tensor(_zipf_p(E_t), device="cuda").log() - (-(u.clamp_min(1e-30)).log()).log()
    # N(0, 1) plus a bias per expert, the same spread of popular and unpopular experts on each rank
    q = (torch.arange(E_t, device="cuda", dtype=torch.float64) * 37 % E_t + 0.5) / E_t
    return torch.randn((R, T, E_t), generator=_gen(seed, 1), device="cuda") + torch.special.ndtri(q).float()


def _routing(case, seed):
    """expert_offsets, row_src_rank, row_slot of the rows dispatched to this rank (expert, then
    source rank, then token), and the rows each source rank gets back."""
    R, E, k = case["ranks"], case["experts"], case["k"]
    top = _router_logits(case, seed).topk(k, dim=-1).indices                      # [R, T, k]
    lo = SELF_RANK * E
    r, t, j = torch.nonzero((top >= lo) & (top < lo + E), as_tuple=True)
    e = top[r, t, j] - lo
    order = ((e * R + r) * case["tokens"] + t).argsort(stable=True)
    e, r = e[order], r[order]
    n = e.numel()
    by_rank = (r * n + torch.arange(n, device="cuda")).argsort()                  # (rank, expert, token)
    counts = torch.bincount(r, minlength=R)
    first = counts.cumsum(0) - counts
    slot = torch.empty(n, dtype=torch.int64, device="cuda")
    slot[by_rank] = torch.arange(n, device="cuda") - first[r[by_rank]]
    offsets = torch.zeros(E + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = torch.bincount(e, minlength=E).cumsum(0)
    return offsets.int(), r.int().contiguous(), slot.int()


def _return_rows(case):
    """Rows of each source rank's region: the mean, a quarter more and some, at most every copy."""
    mean = _rows(case) / case["ranks"]
    return min(case["tokens"] * min(case["k"], case["experts"]), int(mean * 1.25) + 64)


def _stage_inputs(case, seed):
    H, F, E = case["hidden"], case["ffn"], case["experts"]
    off, src, slot = _routing(case, seed)
    g = _gen(seed, 2)

    def normal(shape, std):
        t = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
        return t.normal_(0.0, std, generator=g)

    x = normal((int(src.numel()), H), 1.0)
    w1, w3, w2 = normal((E, F, H), WEIGHT_STD), normal((E, F, H), WEIGHT_STD), normal((E, H, F), WEIGHT_STD)
    return off, src, slot, x, w1, w3, w2


def _combine_inputs(case, seed):
    H, T, k = case["hidden"], case["tokens"], case["k"]
    g = _gen(seed, 3)
    recv = torch.empty((T * k, H), dtype=torch.bfloat16, device="cuda").normal_(0.0, 1.0, generator=g)
    slot = torch.randperm(T * k, generator=g, device="cuda").int().view(T, k)     # every row used once
    gate = torch.rand((T, k), generator=g, device="cuda").mul(4.0).softmax(-1)
    return recv, slot.contiguous(), gate.contiguous()


def _capacity(case):
    """Rows a program sizes its handle for: twice the mean, at most every copy there is."""
    copies = case["ranks"] * case["tokens"] * min(case["k"], case["experts"])
    return int(min(copies, max(512, 2 * _rows(case))))


def prepare(case, seed):
    if case["kind"] == "combine":
        recv, slot, gate = _combine_inputs(case, seed)
        out = torch.zeros((case["tokens"], case["hidden"]), dtype=torch.bfloat16, device="cuda")
        return {"entry": "combine", "args": (recv, slot, gate, out), "out": out}
    off, src, slot, x, w1, w3, w2 = _stage_inputs(case, seed)
    back = np.full(case["ranks"], _return_rows(case), np.int64)
    bufs = [torch.zeros((int(n), case["hidden"]), dtype=torch.bfloat16, device="cuda") for n in back]
    entry = case["entry"]
    if entry in ("run", "serial"):
        routing = [a.cpu().numpy() for a in (off, src, slot)]
    else:
        routing = [off, src, slot]
    state = {"entry": entry, "args": (x, *routing, w1, w3, w2, bufs, back), "out": bufs}
    shape = (case["hidden"], case["ffn"], case["experts"], case["ranks"], SELF_RANK, max(_capacity(case), x.shape[0]))
    if entry == "serial_static":
        state["cfg"] = B.make_config(*shape)
    else:
        state["stage"] = B.MoeStage(*shape, flags=B.MOE_LOCAL_DIRECT | B.MOE_SHARED_CUS)
        if entry in ("run", "run_devplan"):
            state["stream"] = torch.cuda.Stream()
    return state


def run(state):
    entry, args = state["entry"], state["args"]
    if entry == "combine":
        B.moe_combine(*args)
    elif entry == "run":
        state["stage"].run(*args, cu_split=CU_SPLIT, stream=state["stream"])
    elif entry == "run_devplan":
        state["stage"].run_devplan(*args, cu_split=CU_SPLIT, stream=state["stream"])
    elif entry == "serial":
        state["stage"].run_serial(*args)
    elif entry == "serial_devplan":
        state["stage"].run_serial_devplan(*args)
    else:
        B.moe_stage_run_serial_static(state["cfg"], *args)
    return state["out"]


# ------------------------------------------------------------------------------------ what a pass needs

def _rows(case):
    """Mean number of rows dispatched to this rank."""
    R, E, k = case["ranks"], case["experts"], case["k"]
    if case["router"] != "zipf":
        return R * case["tokens"] * k * E / (E * R)
    p = _zipf_p(E * R)  # the first two distinct experts drawn (k = 2)
    hit = [p[e] + sum(p[i] * p[e] / (1 - p[i]) for i in range(len(p)) if i != e) for e in range(E)]
    return R * case["tokens"] * sum(hit)


def work(case):
    H = case["hidden"]
    if case["kind"] == "combine":
        T, k = case["tokens"], case["k"]
        return {"bytes": 2 * H * T * (k + 1) + 8 * k * T, "flops": 2 * H * T * k}
    rows, E, F = _rows(case), case["experts"], case["ffn"]
    active = E * (1.0 - (1.0 - rows / (E * case["ranks"] * case["tokens"])) ** (case["ranks"] * case["tokens"]))
    return {"bytes": 2 * (3 * active * H * F + 2 * rows * H) + 12 * rows, "flops": 6 * rows * H * F}


def tolerance(case):
    # Both outputs are bf16: the rounding of the result is the whole of the difference from 64 bits
    # (1.7e-3 in the 2-norm), and a sum in another order moves some values by one unit in the last
    # place (2^-8 of the value at most).
    if case["kind"] == "combine":
        return {"rel": 5e-3, "max": 2e-2}
    return {"rel": 8e-3, "max": 4e-2}


def exact(case, seed):
    """The same pass in 64 bits; the activation between the two products is rounded to bf16 once,
    which is part of what the stage computes."""
    if case["kind"] == "combine":
        recv, slot, gate = _combine_inputs(case, seed)
        out = torch.zeros((case["tokens"], case["hidden"]), dtype=torch.float64, device="cuda")
        for j in range(case["k"]):
            out += gate[:, j:j + 1].double() * recv[slot[:, j].long()].double()
        return out
    off, src, slot, x, w1, w3, w2 = _stage_inputs(case, seed)
    bufs = [torch.zeros((_return_rows(case), case["hidden"]), dtype=torch.float64, device="cuda")
            for _ in range(case["ranks"])]
    o = off.tolist()
    for e in range(case["experts"]):
        if o[e + 1] == o[e]:
            continue
        xe = x[o[e]:o[e + 1]].double()
        g = xe @ w1[e].double().t()
        u = xe @ w3[e].double().t()
        a = (g / (1.0 + torch.exp(-g)) * u).to(torch.bfloat16).double()
        y = a @ w2[e].double().t()
        re, se = src[o[e]:o[e + 1]], slot[o[e]:o[e + 1]].long()
        for r in range(case["ranks"]):
            m = re == r
            bufs[r][se[m]] = y[m]
    return bufs
