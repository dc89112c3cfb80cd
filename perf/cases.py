"""What this framework is timed on: the calls a serving program makes, at the sizes it makes them.

Five kinds of work:
  forward       one rank's share of one MoE layer, a repeated `binding.RankForward` call on the
                heaviest rank of a planned deployment (plan, tables, weights resident)
  router        the gating network and top-k selection over one batch
  load          the expert-load histogram over a window of routing traces
  load_experts  what a rank does with experts it fetched: re-order (or quantise and re-order)
                their weights for the forward

A deployment (popularity, profiled loads, plan, heaviest rank) is a function of the case
alone; the seed draws the batch and the weights.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2603_28768_amd import binding, synth

DEV = "cuda:0"

# Layer shapes and deployments of synth.CONFIGS, by name.
_SHAPE_FIELDS = ("H", "I", "E", "k", "D")


def _shape(config: str, **more) -> dict:
    c = synth.CONFIGS[config]
    case = {f: getattr(c, f) for f in _SHAPE_FIELDS}
    case.update(T=c.T, replicas=c.replica_slots, zipf=c.zipf_s, hot=c.hot_experts, hot_factor=c.hot_factor,
                popularity=c.index)
    case.update(more)
    return case


def _forward(name: str, config: str, dtype: str = "bf16", weights: str = "packed", gate: bool = False, **more) -> dict:
    return dict(name=name, kind="forward", dtype=dtype, weights=weights, gate=gate, **_shape(config, **more))


def listed() -> list:
    return [
        # decode: the tokens of a few running requests, the layer's own gate included; a handful of
        # rows on the rank, so launches and the stream of a few experts' weights are everything
        _forward("decode_8_gate", "dsv3", gate=True, T=8),
        # decode: an ordinary running batch
        _forward("decode_64", "qwen3", T=64),
        # decode: a large running batch on 8-bit expert weights, not a multiple of anything
        _forward("decode_250_e4m3", "kimi", weights="e4m3", T=250),
        # the small fp32 layer that correctness work and bring-up run on
        _forward("tiny_f32", "tiny", dtype="f32", weights="rowmajor"),
        # a program that keeps its checkpoint's row-major matrices (no second, packed copy), ragged batch
        _forward("prefill_1777_rowmajor", "qwen3", weights="rowmajor", T=1777),
        # prefill chunks at the sizes of the layer configurations
        _forward("prefill_4096", "qwen3"),
        _forward("prefill_8192", "dsv3"),
        _forward("prefill_16384_e4m3", "kimi", weights="e4m3"),
        # the longest batch: one layer of the multi-layer stack
        _forward("prefill_32768", "dsv3_long"),
        # gate and top-k of a prefill chunk
        dict(name="router_8192", kind="router", T=8192, H=7168, E=256, k=8),
        # one rebalancing window of routing traces over all layers of the stack
        dict(name="load_window", kind="load", L=58, T=131072, k=8, E=256, batch=4096),
        # experts fetched at a rebalancing, stored in 8 bits
        dict(name="load_experts_e4m3", kind="load_experts", n=4, H=7168, I=2048, weights="e4m3"),
    ]


_MOST_FLOPS = 6e11      # of a drawn forward


def _log_uniform(rng, lo: float, hi: float) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng) -> dict:
    kind = rng.choice(["decode", "decode", "prefill", "prefill", "rowmajor", "f32", "router", "load", "load_experts"])
    if kind in ("decode", "prefill", "rowmajor"):
        D = rng.choice([8, 16, 32, 64])
        E = rng.choice([96, 128, 160, 256, 384])
        k = rng.choice([2, 4, 6, 8])
        T = _log_uniform(rng, 1, 512) if kind == "decode" else _log_uniform(rng, 512, 24576)
        case = dict(kind="forward", dtype="bf16",
                    weights="rowmajor" if kind == "rowmajor" else rng.choice(["packed", "packed", "e4m3"]),
                    gate=kind == "decode" and T <= 32 and rng.random() < 0.5,
                    T=T, H=rng.choice([1024, 2048, 2880, 4096, 5120, 7168]), I=rng.choice([512, 768, 1408, 1536, 2048]),
                    E=E, k=k, D=D, replicas=rng.choice([0, D // 2, D, 2 * D]), zipf=round(rng.uniform(0.6, 1.4), 2),
                    hot=rng.choice([0, 0, 4]), hot_factor=5.0, popularity=rng.randrange(10, 1000))
        # the heaviest rank sees a few rows of any batch worth sending there
        rows = float(_deployment(case).slot_rows.sum())
        case["T"] = T = max(T, math.ceil(6.0 / rows))
        # an uneven deployment can put most of a batch on one rank: no more work than the longest
        # listed batch, a quarter of it where the weights are row-major
        most = _MOST_FLOPS / (4 if kind == "rowmajor" else 1)
        case["T"] = max(1, int(T * min(1.0, most / work(case)["flops"])))
        return case
    if kind == "f32":
        return dict(kind="forward", dtype="f32", weights="rowmajor", gate=False, T=_log_uniform(rng, 64, 1024),
                    H=rng.choice([64, 128, 196, 256, 512]), I=rng.choice([100, 128, 256, 512]), E=rng.choice([8, 16, 24, 32]),
                    k=rng.choice([1, 2, 4]), D=4, replicas=rng.choice([0, 4]), zipf=round(rng.uniform(0.6, 1.4), 2),
                    hot=0, hot_factor=1.0, popularity=rng.randrange(10, 1000))
    if kind == "router":
        return dict(kind="router", T=_log_uniform(rng, 16, 16384), H=rng.choice([1024, 2048, 2880, 4096, 7168]),
                    E=rng.choice([64, 100, 128, 160, 256, 384]), k=rng.choice([2, 4, 6, 8]))
    if kind == "load":
        return dict(kind="load", L=rng.randint(4, 61), T=_log_uniform(rng, 3000, 131072), k=rng.choice([2, 4, 6, 8]),
                    E=rng.choice([64, 100, 128, 256, 384]), batch=rng.choice([1024, 4096, 5000, 8192]))
    return dict(kind="load_experts", n=rng.randint(1, 6), H=rng.choice([1024, 2048, 2880, 4096, 7168]),
                I=rng.choice([512, 768, 1408, 1536, 2048]), weights=rng.choice(["packed", "e4m3"]))


# ------------------------------------------------------------------- deployments

_PROFILE_TOKENS = 8192


class _Deployment:
    """Popularity, profiled loads, plan and heaviest rank of a forward case."""

    def __init__(self, E, k, D, replicas, zipf, hot, hot_factor, popularity):
        self.pop = synth.popularity(E, zipf, popularity, 0, hot, hot_factor)
        g = np.random.default_rng([popularity, E, k, D])
        scores = g.standard_normal((_PROFILE_TOKENS, E), dtype=np.float32) + np.log(self.pop).astype(np.float32)
        ids = np.argpartition(scores, E - k, axis=1)[:, E - k:]
        self.counts = np.bincount(ids.reshape(-1), minlength=E).astype(np.int64)
        self.plan = binding.Plan(self.counts[None, None], D, replicas)
        lay = self.plan.layer(0)
        _, self.rank = self.plan.rank_rows(0, self.counts)
        lo, hi = lay["rank_slot_off"][self.rank], lay["rank_slot_off"][self.rank + 1]
        self.slots = [int(e) for e in lay["slot_expert"][lo:hi]]
        share = np.bincount(self.slots, minlength=E) / lay["copies"]     # of an expert's tokens, to this rank
        self.token_share = float((1.0 - np.prod(1.0 - share[ids], axis=1)).mean())
        # expected rows of each slot, per token of a batch
        self.slot_rows = np.array([self.counts[e] / lay["copies"][e] for e in self.slots]) / _PROFILE_TOKENS


_DEPLOYMENT_FIELDS = ("E", "k", "D", "replicas", "zipf", "hot", "hot_factor", "popularity")


@functools.lru_cache(maxsize=32)
def _deployment_of(*fields) -> _Deployment:
    return _Deployment(*fields)


def _deployment(case: dict) -> _Deployment:
    return _deployment_of(*(case[f] for f in _DEPLOYMENT_FIELDS))


# ---------------------------------------------------------------------- prepare

def _generator(seed: int) -> torch.Generator:
    return torch.Generator(device=DEV).manual_seed(seed)


def _randn(g, shape, dtype, scale=1.0):
    # a slice at a time: the fp32 draws of a large matrix need no second copy of it
    out = torch.empty(shape, dtype=dtype, device=DEV)
    for part in out.view(-1).split(1 << 26):
        part.copy_(torch.randn(part.numel(), generator=g, device=DEV) * scale)
    return out


def _expert(g, H, I, dtype):
    return (_randn(g, (I, H), dtype, H ** -0.5), _randn(g, (I, H), dtype, H ** -0.5), _randn(g, (H, I), dtype, I ** -0.5))


def _prepare_forward(case, g):
    dep = _deployment(case)
    T, H, I = case["T"], case["H"], case["I"]
    td = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    experts, packed = {}, {}
    for e in dep.slots:
        if e not in experts:
            experts[e] = _expert(g, H, I, td)
            if case["weights"] == "packed":
                packed[e] = binding.pack_weights(*experts[e])
            elif case["weights"] == "e4m3":
                packed[e] = binding.pack_weights_e4m3(*experts[e])
    x = _randn(g, (T, H), td)
    bias = torch.from_numpy(np.log(dep.pop).astype(np.float32)).to(DEV)
    w_router = logits = None
    if case["gate"]:
        # scores N(0,1) plus the log-popularity, which comes in through a constant feature
        x[:, 0] = 1.0
        w_router = _randn(g, (case["E"], H), td, H ** -0.5)
        w_router[:, 0] = bias.to(td)
    else:
        logits = _randn(g, (T, case["E"]), torch.float32) + bias
    fwd = binding.RankForward(dep.plan, 0, dep.rank, case["dtype"], T, H, I, case["k"],
                              [experts[e][0] for e in dep.slots], [experts[e][1] for e in dep.slots],
                              [experts[e][2] for e in dep.slots],
                              packed=[packed[e] for e in dep.slots] if packed else None,
                              weight_format=binding.CRAFT_W_E4M3 if case["weights"] == "e4m3" else binding.CRAFT_W_BF16,
                              w_router=w_router)
    return dict(kind="forward", fwd=fwd, x=x, logits=logits)


def _prepare_router(case, g):
    x = _randn(g, (case["T"], case["H"]), torch.bfloat16)
    w = _randn(g, (case["E"], case["H"]), torch.bfloat16, case["H"] ** -0.5)
    return dict(kind="router", x=x, w=w, k=case["k"], workspace=binding.router_logits_workspace(x, w))


def _prepare_load(case, g):
    L, T, E, k = case["L"], case["T"], case["E"], case["k"]
    ids = torch.empty((L, T, k), dtype=torch.int32, device=DEV)
    exponents = synth.trace_layer_exponents(L, 5)
    for l in range(L):
        logp = torch.from_numpy(np.log(synth.popularity(E, exponents[l], 5, l)).astype(np.float32)).to(DEV)
        # the k largest of log-popularity + Gumbel noise: k draws without replacement
        noise = torch.empty((T, E), device=DEV).exponential_(generator=g)
        ids[l] = binding.route_topk(logp - torch.log(noise.clamp_(min=1e-20)), k)[0]
    return dict(kind="load", ids=ids, E=E, batch=case["batch"])


def _prepare_load_experts(case, g):
    return dict(kind="load_experts", experts=[_expert(g, case["H"], case["I"], torch.bfloat16) for _ in range(case["n"])],
                pack=binding.pack_weights_e4m3 if case["weights"] == "e4m3" else binding.pack_weights)


def prepare(case: dict, seed: int) -> dict:
    g = _generator(seed)
    return {"forward": _prepare_forward, "router": _prepare_router, "load": _prepare_load,
            "load_experts": _prepare_load_experts}[case["kind"]](case, g)


# -------------------------------------------------------------------------- run

def run(state: dict):
    if state["kind"] == "forward":
        return state["fwd"](state["x"], state["logits"])
    if state["kind"] == "router":
        logits = binding.router_logits(state["x"], state["w"], state["workspace"])
        ids, w = binding.route_topk(logits, state["k"])
        return logits, ids, w
    if state["kind"] == "load":
        return binding.expert_load(state["ids"], state["E"], state["batch"])
    return [state["pack"](*e) for e in state["experts"]]


# ------------------------------------------------------------------- work, tolerance

def work(case: dict) -> dict:
    if case["kind"] == "forward":
        dep = _deployment(case)
        T, H, I, E = case["T"], case["H"], case["I"], case["E"]
        es = 4 if case["dtype"] == "f32" else 2
        rows = dep.slot_rows * T
        live = float((1.0 - np.exp(-rows)).sum())            # slots that see a token
        weight = 3 * H * I * es if case["weights"] != "e4m3" else 3 * H * I + 4 * (2 * I + H)
        scores = E * H * es if case["gate"] else T * E * 4
        x_tokens = T if case["gate"] else T * dep.token_share
        flops = 6.0 * H * I * float(rows.sum()) + (2.0 * T * E * H if case["gate"] else 0.0)
        return {"bytes": live * weight + x_tokens * H * es + T * H * es + scores, "flops": flops}
    if case["kind"] == "router":
        T, H, E, k = case["T"], case["H"], case["E"], case["k"]
        return {"bytes": 2.0 * H * (T + E) + 4.0 * T * E + 8.0 * T * k, "flops": 2.0 * T * H * E}
    if case["kind"] == "load":
        L, T, k, E = case["L"], case["T"], case["k"], case["E"]
        n = L * T * k
        return {"bytes": 4.0 * n + 8.0 * L * E * math.ceil(T / case["batch"]), "flops": float(n)}
    n, H, I = case["n"], case["H"], case["I"]
    elements = 3.0 * n * H * I
    if case["weights"] == "packed":
        return {"bytes": 4.0 * elements, "flops": 0.0}
    return {"bytes": 3.0 * elements + 4.0 * n * (2 * I + H), "flops": 2.0 * elements}


def tolerance(case: dict):
    if case["kind"] in ("load", "load_experts"):
        return "exact"
    if case["kind"] == "router":
        # fp32 sums of H products in another order (2.5e-7 from float64 sums at H = 7168);
        # neighbouring scores may then change places
        return {"rel": 2e-6, "differ": 1e-4}
    # fp32: two chained contractions of a few hundred terms (4.2e-7 from float64).  bf16: the
    # activations between the GEMMs, the expert outputs and the result are each rounded to 8 bits
    # of mantissa (2.9e-3 from float64).
    return {"rel": 3e-6} if case["dtype"] == "f32" else {"rel": 1e-2}
