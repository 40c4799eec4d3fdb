"""The work a rank's training or serving program has this library do, as timed cases.

Three kinds of pass, all through the package's public entry points:
  train   forward and backward of one rank's MoE layer (MoERankShape.step).  With n_ep = n_esp = 1 every
          expert is local and the pass is the complete layer; otherwise the buffers that the two AlltoAlls would
          deliver are stand-ins built beforehand from the rank's own data (MoERankShape.fill_stand_ins).
  infer   forward only, every expert local (MoERankLayer.forward / forward_fused_dispatch).
  route   what a rank computes when its experts live on other ranks: gate, dispatch and combine, forward and
          backward, around expert outputs and gradients that arrive from elsewhere.
Token activations and upstream gradients are N(0, 1), weights N(0, sigma_w), the routing is uniform or skewed by
a per-expert gate bias ("normal": N(0, 1); "zipf": -1.1 ln(1 + popularity rank)), as in the package's
synthetic configurations.
"""
import math

import torch

from paper_2407_00599_amd import api
from paper_2407_00599_amd.layer import MoERankLayer, MoERankShape

DEFAULTS = {"kind": "train", "dtype": "bf16", "S_total": 0, "M": 0, "H": 0, "E": 0, "k": 2, "f": 1.0, "n_mp": 1,
            "mp_idx": 0, "n_ep": 1, "n_esp": 1, "esp_idx": 0, "bias": "none", "norm": 1, "fused": True,
            "sigma_x": 1.0, "sigma_w": 0.02}


def _case(**kw):
    return dict(DEFAULTS, **kw)


def listed():
    return [
        # smallest training step (configuration "tiny_fp32"): launches and host calls are all of its time
        _case(name="tiny_fp32", dtype="f32", S_total=256, M=64, H=128, E=4, k=1, f=1.2, norm=0, sigma_x=0.02),
        # one decoding step of a small batch: 32 tokens, no token may drop; the expert weights are the traffic
        _case(name="decode_32", kind="infer", S_total=32, M=1024, H=4096, E=8, f=4.0),
        # a few hundred tokens against the largest configuration's experts (2.1 GB of weights at full hidden size)
        _case(name="prefill_256_wide", kind="infer", S_total=256, M=4096, H=14336, E=8, f=1.5, sigma_w=0.01),
        # ragged training step: no size is a multiple of a tile, top-3, skewed routing with drops
        _case(name="ragged_train", S_total=1003, M=520, H=1544, E=12, k=3, f=1.1, bias="normal"),
        # the layer shape of the paper's layer benchmark (configuration "layer_bf16"), every expert local
        _case(name="layer_bf16", S_total=4096, M=1024, H=4096, E=8, f=1.2),
        # the same layer serving 4096 tokens, with the dispatched buffer materialised
        _case(name="layer_infer", kind="infer", S_total=4096, M=1024, H=4096, E=8, f=1.2, fused=False),
        # fp32 training of a middle-sized layer
        _case(name="layer_fp32", dtype="f32", S_total=1024, M=512, H=2048, E=8, f=1.2),
        # configuration "mp4_ep": a quarter of the tokens, a quarter of the experts, skewed routing
        _case(name="mp4_ep", S_total=8192, M=768, H=3072, E=16, n_mp=4, mp_idx=1, n_ep=4, bias="normal"),
        # configuration "esp4": 64 experts over 8 ranks, 4 hidden shards, Zipf routing: most capacity is padding
        _case(name="esp4", S_total=16384, M=2048, H=8192, E=64, f=1.25, n_ep=8, n_esp=4, esp_idx=1, bias="zipf"),
        # a rank without experts of its own: 128 experts, top-4
        _case(name="route_128", kind="route", S_total=8192, M=2048, H=0, E=128, k=4, f=1.25),
        # configuration "large": the largest one-GPU share
        _case(name="large", S_total=32768, M=4096, H=14336, E=8, n_esp=2, sigma_w=0.01),
    ]


def _log_int(rng, lo, hi, mult=1):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / mult)) * mult))


def draw(rng):
    """One more case of the same ranges: token counts from a decoding step to a long batch, odd sizes among them."""
    while True:
        kind = rng.choice(["train", "train", "train", "infer", "infer", "rank", "rank", "route"])
        dtype = "bf16" if rng.random() < 0.75 else "f32"
        bias = rng.choice(["none", "none", "normal", "zipf"])
        M = _log_int(rng, 64, 4096, rng.choice([8, 64, 256]))
        H = _log_int(rng, 128, 14336, rng.choice([8, 64, 512]))
        n_mp = n_ep = n_esp = 1
        E = rng.choice([1, 2, 4, 4, 8, 8, 8, 12, 16, 16, 24, 32])
        S = _log_int(rng, 16, 8192)
        if kind == "rank":
            n_ep, n_esp, n_mp = rng.choice([1, 2, 4, 8]), rng.choice([1, 2, 4]), rng.choice([1, 1, 2, 4])
            E = n_ep * rng.choice([1, 2, 4, 8])
            H = max(128, H // (8 * n_esp) * (8 * n_esp))
            S = _log_int(rng, 256, 16384)
        elif kind == "route":
            E, H, S = rng.choice([16, 32, 48, 64, 128, 160, 256]), 0, _log_int(rng, 64, 16384)
        k = rng.choice([1, 2, 2, 2, 3, 4]) if kind != "route" else rng.choice([1, 2, 4, 6, 8])
        k = min(k, E)
        f = rng.choice([0.5, 1.0, 1.0, 1.2, 1.25, 1.5, 2.0] + ([4.0] if S <= 512 else []))
        case = _case(kind="train" if kind == "rank" else kind, dtype=dtype, S_total=S * n_mp, M=M, H=H, E=E, k=k, f=f,
                     n_mp=n_mp, mp_idx=rng.randrange(n_mp), n_ep=n_ep, n_esp=n_esp, esp_idx=rng.randrange(n_esp),
                     bias=bias, norm=0 if k == 1 else rng.choice([0, 1, 1]), fused=rng.random() < 0.7)
        C = api.moe_capacity(S, E, k, f)
        rows = E * C * (n_esp if kind == "rank" else 1)            # capacity-padded rows of the rank
        flops = 6 * 2.0 * rows * M * (H // n_esp)
        if flops <= (4e13 if dtype == "bf16" else 1e12) and rows * max(M, H // n_esp) <= 1 << 29 and E // n_ep * M * H <= 1 << 29:
            return case


def _gate_bias(case, gen, dev):
    E = case["E"]
    if case["bias"] == "normal":
        return torch.randn(E, generator=gen, device=dev)
    if case["bias"] == "zipf":
        return -1.1 * torch.log1p(torch.randperm(E, generator=gen, device=dev).float())
    return None


def prepare(case, seed):
    dev = "cuda:0"
    c = dict(DEFAULTS, **case)
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    S_total, M, H, E, k, f = (c[n] for n in ("S_total", "M", "H", "E", "k", "f"))

    def normal(*shape, sigma=1.0, dtype=dt):
        out = torch.empty(*shape, dtype=dtype, device=dev)
        for part in (out if len(shape) > 2 else (out,)):
            part.copy_(torch.randn(part.shape, generator=gen, device=dev) * sigma)
        return out

    x = normal(S_total, M, sigma=c["sigma_x"])
    Wg = normal(M, E, sigma=0.02, dtype=torch.float32)
    bias = _gate_bias(c, gen, dev)
    if c["kind"] == "route":
        S, C = S_total, api.moe_capacity(S_total, E, k, f)
        e = lambda *shape, dtype=torch.float32: torch.empty(*shape, dtype=dtype, device=dev)  # noqa: E731
        i32 = torch.int32
        ws = e(max(api.moe_gate_workspace_bytes(S, E, k), api.moe_gate_bwd_workspace_bytes(S, M, E), 256), dtype=torch.uint8)
        return {"c": c, "C": C, "x": x, "Wg": Wg, "bias": bias, "dy": normal(S, M), "Yret": normal(1, E, C, M),
                "dbuf": normal(1, E, C, M), "logits": e(S, E), "idx": e(S, k, dtype=i32), "slot": e(S, k, dtype=i32),
                "w": e(S, k), "inv": e(E, C, dtype=i32), "counts": e(E, dtype=i32), "buf": e(E, C, M, dtype=dt),
                "y": e(S, M, dtype=dt), "dYret": e(E, C, M, dtype=dt), "dw": e(S, k), "dlogits": e(S, E),
                "dWg": e(M, E), "dbias": e(E) if bias is not None else None, "dx": e(S, M, dtype=dt), "ws": ws}
    W1 = normal(E // c["n_ep"], M, H, sigma=c["sigma_w"])
    W2 = normal(E // c["n_ep"], H, M, sigma=c["sigma_w"])
    if c["kind"] == "infer":
        layer = MoERankLayer(S_total, M, H, E, k, f, dtype=dt, norm_topk=c["norm"], device=dev)
        return {"c": c, "layer": layer, "args": (x, Wg, bias, W1, W2)}
    rank = MoERankShape(S_total, M, H, E, k, f, dtype=dt, n_mp=c["n_mp"], mp_idx=c["mp_idx"], n_ep=c["n_ep"],
                        n_esp=c["n_esp"], esp_idx=c["esp_idx"], norm_topk=c["norm"], device=dev)
    rank.bind(x, Wg, bias, W1, W2, normal(rank.S, M))
    rank.dW1.zero_()     # a hidden shard writes its own columns / rows of the full gradient tensors
    rank.dW2.zero_()
    if not rank.closed:
        rank.fill_stand_ins()
    return {"c": c, "rank": rank}


def run(state):
    c = state["c"]
    if c["kind"] == "infer":
        L = state["layer"]
        y = (L.forward_fused_dispatch if c["fused"] else L.forward)(*state["args"])
        return {"y": y, "logits": L.logits, "idx": L.idx, "slot": L.slot, "w": L.w, "counts": L.counts}
    if c["kind"] == "route":
        s, S, M, E, k, C = state, c["S_total"], c["M"], c["E"], c["k"], state["C"]
        api.moe_gate_topk(s["x"], s["Wg"], s["bias"], S, M, E, k, C, 0, 1, c["norm"], s["logits"], s["idx"], s["slot"],
                          s["w"], s["inv"], s["counts"], s["ws"])
        api.moe_dispatch(s["x"], S, M, E, k, C, s["inv"], None, s["buf"])
        api.moe_combine_fwd(s["Yret"], 1, S, M, E, k, C, s["idx"], s["slot"], s["w"], s["y"])
        api.moe_combine_bwd(s["dy"], s["Yret"], 1, S, M, E, k, C, s["idx"], s["slot"], s["inv"], s["w"], s["dYret"], s["dw"])
        api.moe_combine_fwd(s["dbuf"], 1, S, M, E, k, C, s["idx"], s["slot"], None, s["dx"])
        api.moe_gate_bwd(s["dw"], s["w"], s["idx"], s["logits"], s["x"], s["Wg"], S, M, E, k, c["norm"], s["dlogits"],
                         s["dWg"], s["dbias"], s["dx"], 1, s["ws"])
        names = ("logits", "idx", "slot", "w", "inv", "counts", "buf", "y", "dYret", "dw", "dlogits", "dWg", "dbias", "dx")
        return {n: s[n] for n in names}
    L = state["rank"]
    L.step(c["fused"] and L.closed)
    out = {n: getattr(L, n) for n in ("logits", "idx", "slot", "w", "inv", "counts", "y", "dw", "dYret", "dlogits",
                                      "dWg", "dW1", "dW2", "dx")}
    if L.bias is not None:
        out["dbias"] = L.dbias
    if not L.closed:     # what goes back through the AlltoAlls
        out.update(buf=L.buf, Yout=L.Yout, dXout=L.dXout)
    return out


def _occupied(c):
    """Expected number of filled slots and of experts that any token asked for, from the routing distribution."""
    S, E, k = c["S_total"] // c["n_mp"], c["E"], c["k"]
    C = api.moe_capacity(S, E, k, c["f"])
    gen = torch.Generator()
    gen.manual_seed(1)
    n = 2048
    logits = torch.randn(n, E, generator=gen) * (0.02 * c["sigma_x"] * math.sqrt(c["M"]))
    if c["bias"] == "normal":
        logits += torch.randn(E, generator=gen)
    elif c["bias"] == "zipf":
        logits += -1.1 * torch.log1p(torch.randperm(E, generator=gen).float())
    demand = torch.bincount(logits.topk(k, dim=1).indices.reshape(-1), minlength=E).double() * (S / n)
    return float(demand.clamp(max=C).sum()), float((1 - torch.exp(-demand)).sum()), C


def work(case):
    c = dict(DEFAULTS, **case)
    S, M, E, k = c["S_total"] // c["n_mp"], c["M"], c["E"], c["k"]
    b = 4 if c["dtype"] == "f32" else 2
    valid, active, C = _occupied(c)
    train = c["kind"] != "infer"
    gate = {"bytes": S * M * b + M * E * 4 + S * E * 4 + 12 * S * k, "flops": 2.0 * S * M * E}
    if c["kind"] == "route" or c["n_ep"] * c["n_esp"] > 1:
        P = c["n_esp"]
        # [E, C, M] send buffers written whole, returned rows read where filled; token rows in and out
        nbytes = 2 * gate["bytes"] + b * M * (2 * E * C + 2 * valid * P + 3 * S)
    else:
        nbytes = gate["bytes"] + b * M * S * (4 if train else 1)   # y; dy, dx; x once more in backward
    flops = gate["flops"] * (3 if train else 1)
    if c["kind"] != "route":
        Hl = c["H"] // c["n_esp"]
        rows = valid * c["n_esp"]                 # the rank's experts receive as much as it sends
        experts = min(active, E) / c["n_ep"]      # experts whose weights are needed
        flops += (6 if train else 2) * 2.0 * rows * M * Hl
        nbytes += 2 * experts * M * Hl * b
        if train:
            nbytes += 2 * (E // c["n_ep"]) * M * Hl * b            # weight gradients of every local expert
        if c["n_ep"] * c["n_esp"] > 1:
            nbytes += b * M * (2 * rows + 2 * E * C * c["n_esp"])  # X, dY in; Y, dX out in the receive layout
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    # Against the same path in float64: bf16 outputs are off by 2e-3 to 4e-3 (rounding of Z, the activation, dZ and
    # the results), the bias gradient, a sum that cancels, by up to 9e-3; single values by up to 0.05 rms.
    # fp32 outputs (fp64 sums, rounded once per tensor) are off by 4e-8 to 1.5e-7, single values by up to 2e-6.
    return {"rel": 1e-6, "max": 1e-5} if case.get("dtype") == "f32" else {"rel": 2e-2, "max": 0.25}
