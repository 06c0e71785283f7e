"""The work that a server of MoE experts has this library do, as measurable cases.

A case is one call (one pass) through the public entry points: a batch of
tokens with expert ids and router scores goes in, the weighted sums of the
experts' outputs come back.  The shapes are the ones this repository names
(tiny, mixtral, qwen3 and dsv3, see paper_2509_17863_amd/synth.py) and generic
ones; the batches run from one token to a 16 384-token prefill.

Keys of a case:
  entry    forward   eaas_expert_forward on a caller's workspace
           noalloc   eaas_expert_forward_noalloc (library-owned scratch)
           modular   route_permute, expert_ffn_grouped, unpermute_combine
           segments  eaas_expert_forward_segments: `clients` requests of up to
                     `rows` tokens each, sizes read on the device
           server    eaas_server_step: `clients` slots of `rows` rows holding
                     requests for `layers` layers, some of them empty
  T        tokens (forward, noalloc, modular); clients * rows otherwise
  H, I, E, k   hidden size, expert intermediate size, resident experts, slots
  weights  bf16, fp8 (row-major), fp8_tiled, fp8_a8 (fp8 activations too)
  zipf     exponent of the experts' popularity, 0 for none
  servers  expert servers the router spreads its slots over: only 1/servers of
           the experts live here, ids of the others are skipped
  out      bf16 or fp32
"""
from __future__ import annotations

import math
import random

import torch

from paper_2509_17863_amd import eaas

_WDTYPE = {"bf16": eaas.EAAS_BF16, "fp8": eaas.EAAS_FP8_E4M3,
           "fp8_tiled": eaas.EAAS_FP8_E4M3_TILED, "fp8_a8": eaas.EAAS_FP8_E4M3_A8}

# hidden size, intermediate size, resident experts, slots per token
_TINY = (256, 128, 8, 2)
_MIXTRAL = (4096, 14336, 8, 2)
_QWEN3 = (2048, 768, 128, 8)
_DSV3 = (7168, 2048, 32, 8)


def _case(name, entry, shape, weights, T=0, out="bf16", zipf=0.0, servers=1, clients=0, rows=0,
          layers=1):
    H, I, E, k = shape
    c = dict(entry=entry, T=T or clients * rows, H=H, I=I, E=E, k=k, weights=weights, out=out,
             zipf=zipf, servers=servers, clients=clients, rows=rows, layers=layers)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a toy model's step: nothing but launches and latency
        _case("tiny_64", "forward", _TINY, "bf16", T=64, out="fp32"),
        # one user's decode step on a server that holds its tokens' experts
        _case("decode_1_fp8", "noalloc", _DSV3, "fp8_tiled", T=1),
        # a few users on a many-expert model in bf16
        _case("decode_4_bf16", "forward", _QWEN3, "bf16", T=4),
        # one of eight servers of a wide expert-parallel group: most slots of
        # a token are other servers' (fp8 activations)
        _case("decode_48_a8_ep8", "forward", _DSV3, "fp8_a8", T=48, servers=8),
        # the decode batch of this repository's benchmark
        _case("decode_256_fp8", "forward", _DSV3, "fp8_tiled", T=256),
        # a server turn over its clients' slots: two layers, ragged requests,
        # some slots empty
        _case("server_16x64_bf16", "server", _QWEN3, "bf16", clients=16, rows=64, layers=2),
        # continuous batching: ragged requests of several clients, fp8 weights
        _case("segments_12x160_fp8", "segments", _MIXTRAL, "fp8", clients=12, rows=160),
        # odd sizes through the separate entry points, half the experts elsewhere
        _case("modular_777_odd", "modular", (1920, 640, 24, 6), "bf16", T=777, out="fp32",
              servers=2),
        # prefill with many small, unevenly used experts
        _case("prefill_8192_qwen3", "forward", _QWEN3, "bf16", T=8192, zipf=1.1),
        # prefill with few large experts
        _case("prefill_4096_mixtral", "forward", _MIXTRAL, "bf16", T=4096),
        # a ragged prefill chunk with fp8 activations
        _case("prefill_6001_a8", "forward", _DSV3, "fp8_a8", T=6001, zipf=1.2),
        # the largest prefill of this repository's benchmark
        _case("prefill_16384_dsv3", "forward", _DSV3, "bf16", T=16384, zipf=1.2),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


_MAX_FLOPS = 6.0 * 16384 * 8 * 7168 * 2048   # the largest listed case
_MAX_WEIGHTS = 3.0e9                          # bytes of resident weights


def draw(rng):
    while True:
        weights = rng.choice(["bf16", "bf16", "fp8", "fp8_tiled", "fp8_a8"])
        if rng.random() < 0.6:
            H, I, E, k = rng.choice([_TINY, _MIXTRAL, _QWEN3, _DSV3])
        else:
            H, I = 128 * _log_int(rng, 2, 56), 128 * _log_int(rng, 1, 32)
            E, k = _log_int(rng, 2, 160), rng.randint(1, 8)
        servers = rng.choice([1, 1, 2, 8])
        zipf = rng.choice([0.0, 0.0, 1.1])
        out = rng.choice(["bf16", "bf16", "fp32"])
        entry = rng.choice(["forward"] * 5 + ["noalloc", "modular", "segments", "server"])
        clients = rows = T = 0
        layers = 1
        if entry in ("segments", "server"):
            clients, rows = rng.randint(2, 32), _log_int(rng, 1, 512)
            if entry == "server":
                layers, out = rng.randint(1, 2), "bf16"
        else:
            T = _log_int(rng, 1, 16384)
        if weights in ("fp8_tiled", "fp8_a8") and H % 256:
            continue
        c = _case(None, entry, (H, I, E, k), weights, T, out, zipf, servers, clients, rows, layers)
        if k > E * servers or layers * E > 1024 or c["T"] > 16384:
            continue
        if 6.0 * c["T"] * k * H * I > _MAX_FLOPS:
            continue
        if 3.0 * layers * E * H * I * (2 if weights == "bf16" else 1) > _MAX_WEIGHTS:
            continue
        if entry == "noalloc" and c["T"] * k * (4 * H + 2 * I) + 4 * c["T"] * H > 70e6:
            continue
        return c


# ------------------------------------------------------------------ inputs
def _batch_sizes(case):
    """Tokens of each client's request (part of the case, like its sizes):
    uneven, about a fifth of the clients without a request."""
    r = random.Random(case["clients"] * 1009 + case["rows"])
    return [0 if r.random() < 0.2 else r.randint(1, case["rows"]) for _ in range(case["clients"])]


def _quantize_blocks(w):
    """fp32 [N,K] -> e4m3 codes and one fp32 scale per 128x128 block."""
    n, kk = w.shape
    t = w.view(n // 128, 128, kk // 128, 128)
    amax = t.abs().amax(dim=(1, 3))
    s = torch.where(amax > 0, amax / 448.0, torch.ones_like(amax))
    q = (t / s[:, None, :, None]).clamp_(-448.0, 448.0).view(n, kk).to(torch.float8_e4m3fn)
    return q, s


def _matrices(case, gen, rows, cols):
    """[E, rows, cols] weights ~ N(0, 1/sqrt(fan_in)) and their scales."""
    E, bf16 = case["E"], case["weights"] == "bf16"
    w = torch.empty((E, rows, cols), device="cuda",
                    dtype=torch.bfloat16 if bf16 else torch.float8_e4m3fn)
    s = None if bf16 else torch.empty((E, rows // 128, cols // 128), device="cuda")
    for e in range(E):
        a = torch.randn((rows, cols), device="cuda", generator=gen).mul_(1.0 / math.sqrt(cols))
        if bf16:
            w[e] = a.to(torch.bfloat16)
        else:
            q, sc = _quantize_blocks(a)
            w[e].view(torch.uint8).copy_(q.view(torch.uint8))
            s[e] = sc
    return w, s


def _router(logits, case, gen):
    """Softmax, top-k, renormalised scores; ids past E live on other servers,
    and every token sent here has at least one expert that lives here."""
    k, E = case["k"], case["E"]
    val, ids = torch.topk(logits, k, dim=1)
    score = torch.softmax(val.float(), dim=1)
    lost = (ids >= E).all(dim=1)
    first = torch.randint(0, E, (ids.shape[0],), device=ids.device, generator=gen)
    ids[:, 0] = torch.where(lost, first, ids[:, 0])
    return ids.to(torch.int32).contiguous(), score.contiguous()


def _logits(case, T, gen, device):
    n = case["E"] * case["servers"]
    lg = torch.randn((T, n), device=device, generator=gen)
    if case["zipf"]:
        rank = torch.randperm(n, device=device, generator=gen).float() + 1.0
        lg = lg - case["zipf"] * torch.log(rank)
    return lg


def _inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed * 7919 + 13)
    T, H, I = case["T"], case["H"], case["I"]
    x = torch.randn((T, H), device="cuda", generator=gen).to(torch.bfloat16)
    ids, score = _router(_logits(case, T, gen, "cuda"), case, gen)
    layers = []
    for _ in range(case["layers"]):
        wgu, sgu = _matrices(case, gen, 2 * I, H)
        wd, sd = _matrices(case, gen, H, I)
        layers.append((wgu, sgu, wd, sd))
    return x, ids, score, layers


def _load(case, layer):
    """A layer's weights as the server keeps them."""
    wgu, sgu, wd, sd = layer
    if case["weights"] != "fp8_tiled":
        return layer
    H, I = case["H"], case["I"]
    tgu, td = torch.empty_like(wgu), torch.empty_like(wd)
    eaas.eaas_tile_weights_fp8(wgu, eaas.EAAS_GATE_UP, H, I, tgu)
    eaas.eaas_tile_weights_fp8(wd, eaas.EAAS_DOWN, H, I, td)
    return tgu, sgu, td, sd


def prepare(case, seed):
    T, H, I, E, k = (case[n] for n in ("T", "H", "I", "E", "k"))
    wdt = _WDTYPE[case["weights"]]
    x, ids, score, layers = _inputs(case, seed)
    layers = [_load(case, la) for la in layers]
    st = dict(case=case, x=x, ids=ids, score=score, layers=layers,
              mode=dict(act8=case["weights"] == "fp8_a8", tiled=case["weights"] == "fp8_tiled"))
    odt = torch.float32 if case["out"] == "fp32" else torch.bfloat16
    if case["entry"] in ("forward", "noalloc", "modular"):
        st["out"] = torch.empty((T, H), device="cuda", dtype=odt)
        if case["entry"] != "noalloc":
            st["ws"] = eaas.alloc_workspace(T, H, I, E, k, wdt)
        if case["entry"] == "modular":
            st["routing"] = eaas.alloc_routing(T, k, E)
            st["y"] = torch.zeros((T * k, H), device="cuda")
        return st
    n, rows = case["clients"], case["rows"]
    sizes = _batch_sizes(case)
    px, pi, pw = x.view(n, rows, H), _padded(ids, n, rows, k), _padded(score, n, rows, k)
    st["buffers"] = (pi, pw)
    if case["entry"] == "segments":
        st["out"] = torch.zeros((n, rows, H), device="cuda", dtype=odt)
        st["sizes"] = torch.tensor(sizes, dtype=torch.int32, device="cuda")
        st["table"] = eaas.segment_table([(px[i], pi[i], pw[i], st["out"][i]) for i in range(n)])
        st["ws"] = eaas.alloc_segments_workspace(T, H, I, E, k, wdt)
    else:
        st["payload"] = x.clone()
        flags = [eaas.EAAS_SLOT_READY if s else eaas.EAAS_SLOT_EMPTY for s in sizes]
        st["posted"] = torch.tensor(flags, dtype=torch.int32, device="cuda")
        st["flags"] = st["posted"].clone()
        st["headers"] = torch.tensor([[i % case["layers"], s] for i, s in enumerate(sizes)],
                                     dtype=torch.int32, device="cuda")
        py = st["payload"].view(n, rows, H)
        st["slots"] = eaas.slot_table([(st["flags"][i:i + 1], st["headers"][i], py[i], pi[i], pw[i])
                                       for i in range(n)])
        st["table"] = eaas.layer_table(layers)
        st["ws"] = eaas.alloc_server_workspace(T, H, I, E, k, case["layers"], wdt)
    return st


def _padded(t, n, rows, k):
    """[n*rows, k] -> n request arrays of [rows, k], each 16-byte aligned."""
    width = (rows * k + 3) // 4 * 4
    p = torch.zeros((n, width), dtype=t.dtype, device=t.device)
    p[:, : rows * k] = t.view(n, rows * k)
    return [p[i, : rows * k].view(rows, k) for i in range(n)]


def run(st):
    c = st["case"]
    if c["entry"] == "server":
        # the clients post their requests: payload first, then the flags
        st["payload"].copy_(st["x"])
        st["flags"].copy_(st["posted"])
        eaas.eaas_server_step(st["slots"], c["clients"], st["table"], c["layers"], c["T"], c["H"],
                              c["I"], c["E"], c["k"], st["ws"], _WDTYPE[c["weights"]])
        return {"payload": st["payload"], "flags": st["flags"]}
    wgu, sgu, wd, sd = st["layers"][0]
    scales = dict(w_gate_up_scale=sgu, w_down_scale=sd, **st["mode"])
    if c["entry"] == "segments":
        eaas.eaas_expert_forward_segments(
            st["table"], st["sizes"], c["clients"], c["T"], c["k"], wgu, wd, st["ws"],
            out_dtype=eaas.EAAS_FP32 if c["out"] == "fp32" else eaas.EAAS_BF16, **scales)
    elif c["entry"] == "modular":
        r = st["routing"]
        eaas.eaas_route_permute(st["ids"], c["E"], r, st["ws"], H=c["H"], I=c["I"])
        eaas.eaas_expert_ffn_grouped(st["x"], r, wgu, wd, st["y"], st["ws"], c["k"], **scales)
        eaas.eaas_unpermute_combine(st["y"], r, st["score"], st["out"], c["E"], I=c["I"])
        return {"out": st["out"], "y": st["y"], "counts": r["counts"], "offsets": r["offsets"],
                "perm": r["perm"], "inv": r["inv"], "active": r["active"]}
    elif c["entry"] == "noalloc":
        eaas.eaas_expert_forward_noalloc(st["x"], st["ids"], st["score"], wgu, wd, st["out"],
                                         **scales)
    else:
        eaas.eaas_expert_forward(st["x"], st["ids"], st["score"], wgu, wd, st["out"], st["ws"],
                                 **scales)
    return {"out": st["out"]}


# ------------------------------------------------------------------ measures
def work(case):
    """Weights of the experts that get a token, hidden states in and out, ids
    and scores; the three products of every slot that lives here."""
    gen = torch.Generator().manual_seed(1)
    H, I, E, k, layers = (case[n] for n in ("H", "I", "E", "k", "layers"))
    per_layer = [case["T"]]
    if case["clients"]:
        sizes = _batch_sizes(case)
        per_layer = [sum(sizes[i::layers]) for i in range(layers)]
    slots = active = 0.0
    for t in per_layer:
        if t == 0:
            continue
        ids, _ = _router(_logits(case, min(t, 4096), gen, "cpu"), case, gen)
        ids = ids[ids < E]
        slots += ids.numel() * t / min(t, 4096)
        active += ids.unique().numel()
    tokens = sum(per_layer)
    wb = 2.0 if case["weights"] == "bf16" else 1.0 + 4.0 / 16384
    ob = 4 if case["out"] == "fp32" else 2
    return {"bytes": active * 3.0 * H * I * wb + tokens * H * (2 + ob) + tokens * k * 8.0,
            "flops": 6.0 * slots * H * I}


def tolerance(case):
    """About four times the error against exact(): the rounding of a bf16
    output (1.7e-3), rare bf16 roundings of h next to the exact one (fp32
    outputs, up to 4.8e-5), and e4m3 codes of h moved by the fp8 products'
    own sums (fp8 activations, 1.6e-2)."""
    if case["weights"] == "fp8_a8":
        return {"rel": 3e-2, "max": 3e-1}
    if case["out"] == "fp32":
        return {"rel": 2e-4, "max": 8e-3}
    return {"rel": 7e-3, "max": 3e-2}


# ------------------------------------------------------------------ 64 bits
def _dequantized_rows(a):
    """The e4m3 values, times their scales, of bf16 rows [n, K] (one scale per
    row and 128 channels), in 64 bits."""
    n, kk = a.shape
    t = a.float().view(n, kk // 128, 128)
    amax = t.abs().amax(dim=2, keepdim=True)
    s = torch.where(amax > 0, amax / 448.0, torch.ones_like(amax))
    q = (t / s).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn)
    return (q.double() * s.double()).view(n, kk)


def _weight64(w, s):
    if s is None:
        return w.double()
    n, kk = w.shape
    t = w.to(torch.float64).view(n // 128, 128, kk // 128, 128) * s.double()[:, None, :, None]
    return t.view(n, kk)


def _ffn64(case, x, ids, score, layer, y=None, row0=0):
    """Weighted sums in 64 bits, with h rounded where the step defines it (to
    bf16; fp8 activations: x and h quantized per row and 128 channels).
    y: optional [R, H], the experts' rows grouped by expert."""
    wgu, sgu, wd, sd = layer
    a8 = case["weights"] == "fp8_a8"
    I = case["I"]
    out = torch.zeros((x.shape[0], case["H"]), dtype=torch.float64, device=x.device)
    x64 = _dequantized_rows(x) if a8 else x.double()
    for e in range(case["E"]):
        tok, slot = (ids == e).nonzero(as_tuple=True)
        if tok.numel() == 0:
            continue
        gu = x64[tok] @ _weight64(wgu[e], None if sgu is None else sgu[e]).t()
        g, u = gu[:, :I], gu[:, I:]
        h = (g / (1.0 + torch.exp(-g)) * u).float().to(torch.bfloat16)
        h = _dequantized_rows(h) if a8 else h.double()
        v = h @ _weight64(wd[e], None if sd is None else sd[e]).t()
        out.index_add_(0, tok, v * score[tok, slot].double()[:, None])
        if y is not None:
            y[row0: row0 + tok.numel()] = v
            row0 += tok.numel()
    return out


def exact(case, seed):
    x, ids, score, layers = _inputs(case, seed)
    if case["entry"] in ("forward", "noalloc"):
        return {"out": _ffn64(case, x, ids, score, layers[0])}
    if case["entry"] == "modular":
        y = torch.zeros((case["T"] * case["k"], case["H"]), dtype=torch.float64, device="cuda")
        out = _ffn64(case, x, ids, score, layers[0], y)
        return {"out": out, "y": y, "counts": None, "offsets": None, "perm": None, "inv": None,
                "active": None}
    n, rows = case["clients"], case["rows"]
    sizes = _batch_sizes(case)
    server = case["entry"] == "server"
    out = x.double().view(n, rows, -1).clone() if server else torch.zeros(
        (n, rows, case["H"]), dtype=torch.float64, device="cuda")
    for la in range(case["layers"]):
        rowsel = [i * rows + t for i, s in enumerate(sizes) if i % case["layers"] == la
                  for t in range(s)]
        if rowsel:
            sel = torch.tensor(rowsel, device="cuda")
            out.view(n * rows, -1)[sel] = _ffn64(case, x[sel], ids[sel], score[sel], layers[la])
    if server:
        return {"payload": out.view(n * rows, -1), "flags": None}
    return {"out": out}
