"""The calls whose speed matters, as a program that serves a model with this library makes them.

A case is a dict of plain values with a "kind":

  step    the four linear layers of one Llama-shaped decoder layer (QKV, O, gate+up, down) on M rows,
          each with its own input: what one layer asks of the library per token (decode) or per prompt
  linear  one rg_linear / rg_linear_bias / rg_linear_f32w call on any shape
  head    the LM head on M rows and the greedy decision over its logits
  attn    one decode-attention call on B sequences of ragged lengths

Weights are bf16 (or f32 where "weights" says so), activations f32.  Every output is fixed bit for
bit by the documented order, so the tolerance is "exact" everywhere.
"""
import math

import torch

import paper_2609_25624_amd as rg


def listed():
    llama = {"hidden": 4096, "qkv": 6144, "inter": 14336}
    return [
        # the smallest layer of the benchmark's configurations: launch and host cost count
        {"name": "linear m1 1024x1024", "kind": "linear", "M": 1, "N": 1024, "K": 1024, "weights": "bf16", "bias": False},
        # single-stream decode of the 8B-shaped model: the benchmark's own step
        {"name": "step m1", "kind": "step", "M": 1, **llama, "weights": "bf16"},
        # a few sequences decoded together
        {"name": "step m4", "kind": "step", "M": 4, **llama, "weights": "bf16"},
        # a served batch
        {"name": "step m16", "kind": "step", "M": 16, **llama, "weights": "bf16"},
        # the largest batch of the decode range
        {"name": "step m64", "kind": "step", "M": 64, **llama, "weights": "bf16"},
        # a prompt of ordinary, odd length
        {"name": "step prompt m333", "kind": "step", "M": 333, **llama, "weights": "bf16"},
        # a long prompt through the 70B-shaped down projection: the largest call
        {"name": "down70b prompt m2048", "kind": "linear", "M": 2048, "N": 8192, "K": 28672, "weights": "bf16", "bias": False},
        # the next token of one sequence: logits over the vocabulary and the greedy decision
        {"name": "head m1", "kind": "head", "M": 1, "N": 128256, "K": 4096},
        # the reproducibility probes with FP32 weights, on a served batch
        {"name": "step f32 m16", "kind": "step", "M": 16, **llama, "weights": "f32"},
        # sizes that no tile divides and rows that start at odd addresses, with a bias
        {"name": "linear ragged bias", "kind": "linear", "M": 5, "N": 2999, "K": 1003, "weights": "bf16", "bias": True},
        # decode attention of a served batch, 8B-shaped heads, ragged lengths
        {"name": "attn b16", "kind": "attn", "B": 16, "H": 32, "Hkv": 8, "L": 4096, "D": 128},
        # decode attention of one long sequence
        {"name": "attn long", "kind": "attn", "B": 1, "H": 32, "Hkv": 8, "L": 32768, "D": 128},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("step", "step", "linear", "linear", "linear", "head", "attn", "attn"))
    if kind == "step":
        # hidden sizes in multiples of 64, from small models to somewhat beyond the 8B shape
        hidden = 64 * _log(rng, 16, 84)
        inter = 64 * int(hidden * rng.uniform(2.0, 3.6) / 64)
        qkv = hidden + 256 * rng.randint(1, 8)
        weights = "f32" if rng.random() < 0.2 else "bf16"
        return {"kind": kind, "M": _log(rng, 1, 640), "hidden": hidden, "qkv": qkv, "inter": inter, "weights": weights}
    if kind == "head":
        return {"kind": kind, "M": _log(rng, 1, 64), "N": rng.randint(32000, 160000), "K": 8 * _log(rng, 128, 512)}
    if kind == "attn":
        Hkv = rng.choice((1, 2, 4, 8))
        G = rng.choice((1, 2, 4, 4, 5, 8, 8))
        D = rng.choice((64, 128, 128, 128, 256))
        B = _log(rng, 1, 64)
        longest = min(32768, int(4e8 / (B * Hkv * D)))   # at most 1.6 GB of keys and values
        return {"kind": kind, "B": B, "H": Hkv * G, "Hkv": Hkv, "L": _log(rng, 64, longest), "D": D}
    weights = "f32" if rng.random() < 0.25 else "bf16"
    bias = weights == "bf16" and rng.random() < 0.4
    if rng.random() < 0.25:
        # rows of W that start at odd addresses: small, unaligned models and test shapes
        return {"kind": kind, "M": _log(rng, 1, 64), "N": _log(rng, 64, 4096) | 1, "K": _log(rng, 64, 4096) | 1,
                "weights": weights, "bias": bias}
    K = 8 * _log(rng, 32, 3584)
    N = _log(rng, 256, min(57344, 5e8 / K))
    return {"kind": kind, "M": _log(rng, 1, min(2048, 9e11 / (2 * N * K))), "N": N, "K": K, "weights": weights, "bias": bias}


def _layers(case):
    """(N, K) of each linear layer of a case."""
    if case["kind"] == "step":
        h, q, i = case["hidden"], case["qkv"], case["inter"]
        return [(q, h), (h, h), (2 * i, h), (h, i)]
    return [(case["N"], case["K"])]


def _lens(case):
    """Sequence lengths: the longest is L, the others spread below it as in a batch that is being served."""
    B, L = case["B"], case["L"]
    return [max(1, L - (L * b) // (2 * B)) for b in range(B)]


def prepare(case, seed):
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)

    def normal(shape, std, dtype=torch.float32):
        return torch.empty(shape, dtype=dtype, device=dev).normal_(0.0, std, generator=g)

    if case["kind"] == "attn":
        B, H, Hkv, L, D = (case[k] for k in ("B", "H", "Hkv", "L", "D"))
        return {"kind": "attn",
                "q": normal((B, H, D), 1.0), "k": normal((B, Hkv, L, D), 1.0, torch.bfloat16),
                "v": normal((B, Hkv, L, D), 1.0, torch.bfloat16),
                "lens": torch.tensor(_lens(case), dtype=torch.int32, device=dev), "scale": 1.0 / math.sqrt(D),
                "out": torch.empty((B, H, D), dtype=torch.float32, device=dev),
                "ws": torch.empty(rg.rg_attn_workspace_size(B, H, L, D), dtype=torch.uint8, device=dev)}
    M = case["M"]
    wdtype = torch.float32 if case.get("weights") == "f32" else torch.bfloat16
    s = {"kind": case["kind"], "f32": wdtype == torch.float32, "layers": []}
    for N, K in _layers(case):
        x = normal((M, K), 1.0)
        w = normal((N, K), 0.02, wdtype)
        b = normal((N,), 1.0) if case.get("bias") else None
        s["layers"].append((x, w, b, torch.empty((M, N), dtype=torch.float32, device=dev)))
    if case["kind"] == "head":
        s["ids"] = torch.empty((M,), dtype=torch.int64, device=dev)
    return s


def run(state):
    if state["kind"] == "attn":
        return rg.rg_attn_decode(state["q"], state["k"], state["v"], state["lens"], state["out"], state["scale"],
                                 workspace=state["ws"])
    ys = []
    for x, w, b, y in state["layers"]:
        if b is not None:
            rg.rg_linear_bias(x, w, b, y)
        elif state["f32"]:
            rg.rg_linear_f32w(x, w, y)
        else:
            rg.rg_linear(x, w, y)
        ys.append(y)
    if state["kind"] == "head":
        return {"logits": ys[0], "ids": rg.rg_argmax_rows(ys[0], state["ids"])}
    return ys


def work(case):
    if case["kind"] == "attn":
        B, H, Hkv, D = (case[k] for k in ("B", "H", "Hkv", "D"))
        positions = sum(_lens(case))
        return {"bytes": 2 * positions * Hkv * D * 2 + 2 * B * H * D * 4 + B * 4, "flops": 4 * positions * H * D}
    M, wb = case["M"], 4 if case.get("weights") == "f32" else 2
    nbytes = sum(wb * N * K + 4 * M * K + 4 * M * N + (4 * N if case.get("bias") else 0) for N, K in _layers(case))
    if case["kind"] == "head":
        nbytes += 8 * M
    return {"bytes": nbytes, "flops": sum(2 * M * N * K for N, K in _layers(case))}


def tolerance(case):
    # the order of every sum is part of the interface: each output bit is fixed by the shape
    return "exact"


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] == "attn":
        B, H, Hkv, D = (case[k] for k in ("B", "H", "Hkv", "D"))
        out = torch.empty((B, H, D), dtype=torch.float64, device=s["q"].device)
        for b, n in enumerate(_lens(case)):
            for h in range(Hkv):
                q = s["q"][b].view(Hkv, H // Hkv, D)[h].double()
                t = (q @ s["k"][b, h, :n].double().t().contiguous()) * s["scale"]
                out[b].view(Hkv, H // Hkv, D)[h] = torch.softmax(t, dim=1) @ s["v"][b, h, :n].double()
        return out
    ys = []
    for x, w, b, _ in s["layers"]:
        y = x.double() @ w.double().t()
        ys.append(y if b is None else y + b.double())
    return {"logits": ys[0], "ids": None} if case["kind"] == "head" else ys
