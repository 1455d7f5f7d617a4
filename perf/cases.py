"""Performance cases of the compression pass: what a serving program calls, over the range it calls it with.

The library's calls are measured the way a caller uses them:

* ``score``     nkv.score over the prompt's keys;
* ``compress``  nkv.budget + nkv.select_compact on scores that are there already (fixed scores, so that budgets, kept
                indices and packed rows can be compared bit for bit);
* ``pass``      the three calls through nkv.Compressor;
* ``decode``    one new token's attention over a compressed cache.

A case is a dict of plain values.  ``lens`` is the prompts' lengths separated by commas; ``layout`` says how the cache
tensors lie: "dense" ([L][H][T][d]), "layers" (one tensor per layer, as frameworks keep their caches) or "slab" (room
for ``room`` more tokens behind the prompt of every head, a cache allocated for the generation that follows).
Keys have the structure the method reacts to: a mean direction per head, an offset per 512-token segment, outliers, and
sink-like keys in front.
"""
from __future__ import annotations

import math

import torch

import paper_2605_26678_amd as nkv

DTYPES = {"fp32": (torch.float32, nkv.DTYPE_F32, 4), "bf16": (torch.bfloat16, nkv.DTYPE_BF16, 2),
          "fp16": (torch.float16, nkv.DTYPE_F16, 2), "fp8": (torch.float8_e4m3fn, nkv.DTYPE_F8_E4M3, 1)}
SEGMENT, N_SINK = 512, 4
RAGGED = "4096,8192,16384,32768,32768,16384,8192,4096"      # the batched serving shape of the benchmark


def listed():
    return [
        # the smallest call: one fp32 layer of two heads (the benchmark's tiny workload); launches and latency count
        dict(name="pass_tiny_fp32", path="pass", L=1, H=2, d=128, dtype="fp32", lens="4096", r=0.5, layout="dense"),
        # a few layers of a model with as many KV heads as query heads and a head dim that is no power of two, a ragged
        # batch of odd prompt lengths
        dict(name="score_mha_d96_ragged", path="score", L=4, H=32, d=96, dtype="fp16", lens="1531,4099,777,2050",
             layout="dense"),
        # a short prompt on a small model, after prefill, over the framework's list of per-layer cache tensors
        dict(name="score_llama1b_4k", path="score", L=16, H=8, d=64, dtype="bf16", lens="4096", layout="layers"),
        # layer by layer inside a long prefill (what streaming the compression costs), cache with room for decoding
        dict(name="score_layer_32k", path="score", L=1, H=8, d=128, dtype="bf16", lens="32768", layout="slab", room=1024),
        # the headline workload: 36 layers, a 32k-token prompt
        dict(name="score_qwen4b_32k", path="score", L=36, H=8, d=128, dtype="bf16", lens="32768", layout="dense"),
        # the batched serving shape
        dict(name="score_llama3b_ragged", path="score", L=28, H=8, d=128, dtype="bf16", lens=RAGGED, layout="dense"),
        # a group of layers of a very long prompt with an 8-bit cache
        dict(name="score_fp8_128k", path="score", L=8, H=8, d=128, dtype="fp8", lens="131072", layout="dense"),
        # the other two calls on the same three situations: one layer, the headline prompt, the ragged batch
        dict(name="compress_layer_32k", path="compress", L=1, H=8, d=128, dtype="bf16", lens="32768", r=0.75,
             layout="slab", room=1024),
        dict(name="compress_qwen4b_32k", path="compress", L=36, H=8, d=128, dtype="bf16", lens="32768", r=0.75,
             layout="dense"),
        dict(name="compress_llama3b_ragged", path="compress", L=28, H=8, d=128, dtype="bf16", lens=RAGGED, r=0.95,
             layout="dense"),
        # decoding over what is left of the headline prompt, all layers' attention in one call
        dict(name="decode_qwen4b_32k", path="decode", L=36, H=8, d=128, dtype="bf16", lens="32768", r=0.75, G=4),
        # decoding layer by layer, the ragged batch: the call a decode loop makes once per layer and token
        dict(name="decode_layer_ragged", path="decode", L=1, H=8, d=128, dtype="bf16", lens=RAGGED, r=0.95, G=3),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _lens(rng, longest):
    n = rng.choice([1, 1, 1, 2, 3, 5, 8])
    lens = [_log_int(rng, 512, longest) for _ in range(n)]
    if rng.random() < 0.3:
        lens = [max(512, x // 1024 * 1024) for x in lens]
    return lens


def draw(rng):
    path = rng.choice(["score", "score", "compress", "compress", "decode", "pass"])
    c = dict(path=path)
    if path == "pass":          # small calls, one layer
        c.update(L=1, H=rng.choice([1, 2, 4]), d=rng.choice([64, 128]), dtype=rng.choice(["fp32", "bf16", "fp16"]))
        lens, most = [_log_int(rng, 512, 8192)], 1 << 15
    elif path == "score":
        c.update(L=_log_int(rng, 1, 36), H=rng.choice([2, 4, 8, 8, 32]), d=rng.choice([64, 96, 128, 128]),
                 dtype=rng.choice(["bf16", "bf16", "fp16", "fp8"]))
        lens, most = _lens(rng, 131072), 1 << 20 if c["d"] == 96 else 8 << 20
    elif path == "compress":
        c.update(L=_log_int(rng, 1, 36), H=rng.choice([2, 4, 8, 8, 32]), d=rng.choice([64, 96, 128, 128]),
                 dtype=rng.choice(["bf16", "bf16", "fp16", "fp8"]))
        lens, most = _lens(rng, 131072), 8 << 20
    else:
        c.update(L=_log_int(rng, 1, 36), H=rng.choice([2, 4, 8, 8, 32]), d=rng.choice([64, 128, 128]),
                 dtype=rng.choice(["bf16", "fp16"]), G=rng.choice([1, 2, 3, 4, 8]))
        lens, most = _lens(rng, 65536), 8 << 20
    while c["L"] * c["H"] * sum(lens) > most:                          # (layer, head, token) triples
        if c["L"] > 1:
            c["L"] = max(1, c["L"] // 2)
        elif c["H"] > 8:
            c["H"] = 8
        else:
            lens = [max(512, x // 2) for x in lens]
    c["lens"] = ",".join(str(x) for x in lens)
    if path != "score":
        c["r"] = round(rng.uniform(0.3, 0.97), 3)
    if path != "decode":
        c["layout"] = rng.choice(["dense", "dense", "layers", "slab"]) if len(lens) == 1 else rng.choice(["dense", "layers"])
        if c["layout"] == "slab":
            c["room"] = 8 * rng.randint(1, 256)
    return c


def _generator(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + salt) & 0x7FFFFFFFFFFF)
    return g


def _unit(x):
    return x / x.norm(dim=-1, keepdim=True).clamp_min(1e-20)


def _keys(g, H, N, d):
    """fp32 keys [H, N, d] of one prompt and layer."""
    f = dict(device="cuda", generator=g)
    mean = _unit(torch.randn(H, d, **f))
    segments = (N + SEGMENT - 1) // SEGMENT
    offset = (0.5 + 1.5 * torch.rand(1, **f)) * _unit(torch.randn(H, segments, d, **f))
    k = torch.randn(H, N, d, **f)
    k += (3.0 * mean[:, None, :] + offset).repeat_interleave(SEGMENT, dim=1)[:, :N]
    n_out = min(128, (N - N_SINK) // 8)
    if n_out > 0:                                                      # one outlier in each of n_out stretches
        width = (N - N_SINK) // n_out
        at = N_SINK + torch.arange(n_out, device="cuda") * width + (torch.rand(H, n_out, **f) * width).long().clamp_(max=width - 1)
        away = torch.randn(H, n_out, d, **f)
        away -= (away * mean[:, None, :]).sum(-1, keepdim=True) * mean[:, None, :]
        k.scatter_(1, at[:, :, None].expand(H, n_out, d), 6.0 * _unit(away))
    k[:, :N_SINK] = 10.0 * mean[:, None, :]
    return k


def _scores(g, k):
    """Scores [H, N] of the kind the scoring call gives: a min-maxed anomaly per head with a token-wise spread, the sinks
    pinned."""
    kh = _unit(k)
    a = -(kh * _unit(kh.sum(dim=1, keepdim=True))).sum(-1)
    a += 0.05 * torch.randn(a.shape, device="cuda", generator=g)
    lo, hi = a.amin(dim=1, keepdim=True), a.amax(dim=1, keepdim=True)
    s = (a - lo) / (hi - lo)
    s[:, :N_SINK] = nkv.PIN
    return s


def _lens_of(case):
    return [int(x) for x in case["lens"].split(",")]


def _cache(case, N_all):
    """An empty cache in the case's layout: (per-layer views [H, T, d], the tensor to hand to a call, strides, layers)."""
    dt, L, H, d = DTYPES[case["dtype"]][0], case["L"], case["H"], case["d"]
    if case["layout"] == "layers":
        layers = [torch.empty(H, N_all, d, dtype=dt, device="cuda") for _ in range(L)]
        return layers, layers[0], None, layers
    room = case.get("room", 0)
    whole = torch.zeros(L, H, N_all + room, d, dtype=torch.uint8, device="cuda").to(dt) if room \
        else torch.empty(L, H, N_all, d, dtype=dt, device="cuda")
    views = [whole[l, :, :N_all] for l in range(L)]
    strides = (H * (N_all + room) * d, (N_all + room) * d, 0) if room else None
    return views, whole, strides, None


def prepare(case, seed):
    if case["path"] == "decode":
        return _prepare_decode(case, seed)
    lens, L, H, d = _lens_of(case), case["L"], case["H"], case["d"]
    dt, code, _ = DTYPES[case["dtype"]]
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    T = cu[-1]
    with_values = case["path"] != "score"
    k_views, keys, k_strides, k_layers = _cache(case, T)
    v_views, values, v_strides, v_layers = _cache(case, T) if with_values else (None,) * 4
    scores = torch.empty(L, H, T, dtype=torch.float32, device="cuda")
    g = _generator(seed, 1)
    for l in range(L):
        for p in range(len(lens)):
            k = _keys(g, H, lens[p], d)
            k_views[l][:, cu[p]:cu[p + 1]] = k.to(dt)
            if case["path"] == "compress":
                scores[l, :, cu[p]:cu[p + 1]] = _scores(g, k)
        if with_values:
            v_views[l].copy_(torch.randn(H, T, d, device="cuda", generator=g))
    shape = nkv.Shape(L, H, d, d, code, cu, key_strides=k_strides, value_strides=v_strides, key_layers=k_layers,
                      value_layers=v_layers)
    params = nkv.params_default()
    s = dict(path=case["path"], shape=shape, params=params, keys=keys, values=values, hold=(k_layers, v_layers))
    if case["path"] == "score":
        s["ws"] = torch.empty(nkv.workspace_bytes(shape, params), dtype=torch.uint8, device="cuda")
        s["scores"] = scores
        # the pinned and the routed scores apart: next to 3e38 no difference of a routed score would be seen
        s["out"] = [(scores[:, :, a:a + N_SINK], scores[:, :, a + N_SINK:b]) for a, b in zip(cu[:-1], cu[1:])]
        return s
    s["r"] = [case["r"]] * len(lens)
    s["c"] = c = nkv.Compressor(shape, s["r"], params)
    s["out"] = dict(k_per_head=c.k_per_head, head_off=c.head_off, kept_idx=c.kept_idx[:c.rows],
                    packed_k=c.packed_k[:c.rows], packed_v=c.packed_v[:c.rows], near=c.near)
    if case["path"] == "compress":
        s["scores"] = scores
    else:
        s["out"]["scores"] = [(c.scores[:, :, a:a + N_SINK], c.scores[:, :, a + N_SINK:b]) for a, b in zip(cu[:-1], cu[1:])]
    return s


def _head_rows(case, g):
    """Retained rows per (prompt, layer, head): a fifth of the average each, the rest dealt unevenly, as budgets are."""
    L, H = case["L"], case["H"]
    rows = []
    for N in _lens_of(case):
        n = int((1.0 - case["r"]) * N + 1e-9)
        share = torch.rand(L, H, generator=g) + 0.25
        part = (share / share.sum(-1, keepdim=True) * (H * (n - n // 5))).floor().long()
        part[:, 0] += H * (n - n // 5) - part.sum(-1)
        rows.append((n // 5 + part).clamp(max=N))
    return torch.stack(rows).reshape(-1)                               # [P * L * H]


def _prepare_decode(case, seed):
    lens, L, H, d, G = _lens_of(case), case["L"], case["H"], case["d"], case["G"]
    dt, code, _ = DTYPES[case["dtype"]]
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    shape, params, Hq = nkv.Shape(L, H, d, d, code, cu), nkv.params_default(), H * G
    # row counts are part of the case, not of the seed: buffers and outputs keep their sizes
    host = torch.Generator()
    host.manual_seed(20260)
    n_rows = _head_rows(case, host)
    head_off = torch.zeros(n_rows.numel() + 1, dtype=torch.int64)
    head_off[1:] = torch.cumsum(n_rows, 0)
    rows = int(head_off[-1])
    g = _generator(seed, 2)
    f = dict(device="cuda", generator=g)
    units = n_rows.numel()
    mean = _unit(torch.randn(units, d, **f))
    k = torch.randn(rows, d, **f) + (3.0 * mean).repeat_interleave(n_rows.cuda(), dim=0)
    # a query looks for one of its head's rows
    first, count = head_off[:-1].cuda()[:, None], n_rows.cuda()[:, None]
    at = first + (torch.rand(units, G, **f) * count).long().clamp(max=max(rows - 1, 0))
    q = torch.randn(units, G, d, **f) + 0.5 * k[at.clamp(max=rows - 1)]
    s = dict(path="decode", shape=shape, params=params, rows=rows, Hq=Hq, scale=1.0 / math.sqrt(d),
             q=q.reshape(len(lens), L, Hq, d).to(dt), head_off=head_off.cuda(), packed_k=k.to(dt),
             packed_v=torch.randn(rows, d, **f).to(dt))
    s["attn"] = torch.empty(len(lens), L, Hq, d, dtype=torch.float32, device="cuda")
    s["lse"] = torch.empty(len(lens), L, Hq, dtype=torch.float32, device="cuda")
    s["ws"] = torch.empty(max(256, nkv.decode_workspace_bytes(shape, Hq, rows)), dtype=torch.uint8, device="cuda")
    s["out"] = dict(attn=s["attn"], lse=s["lse"])
    return s


def run(s):
    if s["path"] == "score":
        nkv.score(s["keys"], s["shape"], s["params"], s["scores"], s["ws"])
    elif s["path"] == "compress":
        c = s["c"]
        nkv.budget(s["scores"], s["shape"], s["params"], s["r"], c.k_per_head, c.ws)
        nkv.select_compact(s["keys"], s["values"], s["scores"], c.k_per_head, s["shape"], s["params"], c.packed_k,
                           c.packed_v, c.kept_idx, c.head_off, c.rows, c.near, c.ws)
    elif s["path"] == "pass":
        s["c"].run(s["keys"], s["values"])
    else:
        nkv.decode_attention(s["q"], s["packed_k"], s["packed_v"], s["head_off"], s["rows"], s["shape"], s["params"],
                             s["Hq"], s["scale"], s["attn"], s["lse"], s["ws"])
    return s["out"]


def work(case):
    """Inputs read once and outputs written once.  Arithmetic: per key and dimension a square, a scaling, an addition to
    each of the two fixed anchors, an addition to and a subtraction from the window's, a square of the window's, and
    three dot products; decoding: two products per query head, row and dimension."""
    lens, L, H, d = _lens_of(case), case["L"], case["H"], case["d"]
    e = DTYPES[case["dtype"]][2]
    n = L * H * sum(lens)
    kept = 0 if case["path"] == "score" else L * H * sum(int((1.0 - case["r"]) * N + 1e-9) for N in lens)
    if case["path"] == "decode":
        q_rows = len(lens) * L * H * case["G"]
        return {"bytes": kept * 2 * d * e + q_rows * (d * e + 4 * d + 4), "flops": 4 * kept * case["G"] * d}
    score = {"bytes": n * (d * e + 4), "flops": n * d * 15}
    moved = kept * (4 * d * e + 4)
    if case["path"] == "score":
        return score
    if case["path"] == "compress":
        return {"bytes": 4 * n + moved, "flops": 0}
    return {"bytes": score["bytes"] + kept * (3 * d * e + 4), "flops": score["flops"]}   # kept keys have been read


def tolerance(case):
    if case["path"] == "compress":
        return "exact"
    if case["path"] == "decode":
        return {"rel": 1.5e-6, "max": 8e-6}           # against float64: 3.4e-7 and 1.8e-6
    return {"rel": 5e-7, "max": 4e-6}                # the library's scoring formulations among themselves: 1.2e-7 and 1.0e-6


def _exact_scores(k):
    """Scores [H, N] of fp64 keys [H, N, d]: every anchor a difference of running sums, every ranking a full sort."""
    H, n, d = k.shape
    eps, b = 1e-12, min(max(n // 32, 128), 256)
    kh = k / k.norm(dim=-1, keepdim=True).clamp_min(eps)
    run = torch.zeros(H, n + 1, d, dtype=torch.float64, device=k.device)
    torch.cumsum(kh, dim=1, out=run[:, 1:])
    i = torch.arange(n, device=k.device)
    first = i // b * b
    a = []
    for anchor in (run[:, -1:], run[:, (first + b).clamp_max(n)] - run[:, first], run[:, 1:] - run[:, (i - 63).clamp_min(0)]):
        x = -(kh * anchor).sum(-1) / (kh.norm(dim=-1).clamp_min(eps) * anchor.norm(dim=-1).clamp_min(eps))
        lo, hi = x.amin(-1, keepdim=True), x.amax(-1, keepdim=True)
        a.append(torch.where(hi - lo < 1e-6, torch.zeros_like(x), (x - lo) / (hi - lo)))
    a = torch.stack(a)                                                 # [3, H, n]
    m = max(1, int(0.1 * n + 1e-9))
    ranked = a.sort(dim=-1).values
    gap = ranked[..., n - m:].mean(-1) - ranked[..., :m].mean(-1)
    prior = torch.tensor([0.4, 0.4, 0.2], dtype=torch.float64, device=k.device)
    weight = torch.softmax(prior.log()[:, None] + 3.0 * gap, dim=0)
    s = a.std(dim=0, correction=0)
    lo, hi = s.amin(-1, keepdim=True), s.amax(-1, keepdim=True)
    s = torch.where(hi - lo < 1e-6, torch.zeros_like(s), (s - lo) / (hi - lo))
    s = (s - s.mean(-1, keepdim=True)).clamp_min(0.0)
    gate = torch.sigmoid(10.0 * (s - 0.6))
    out = (1.0 - gate) * (weight[..., None] * a).sum(0) + gate * a.amax(0)
    out[:, :N_SINK] = torch.tensor(nkv.PIN, dtype=torch.float32).double()
    return out


def _exact_decode(s):
    units, G = s["head_off"].numel() - 1, s["Hq"] // s["shape"].H
    q, off = s["q"].double().reshape(units, G, -1), s["head_off"].tolist()
    attn, lse = torch.zeros_like(q), torch.full((units, G), -math.inf, dtype=torch.float64, device="cuda")
    for u in range(units):
        if off[u + 1] > off[u]:
            z = s["scale"] * (q[u] @ s["packed_k"][off[u]:off[u + 1]].double().T)
            lse[u] = torch.logsumexp(z, dim=-1)
            attn[u] = torch.softmax(z, dim=-1) @ s["packed_v"][off[u]:off[u + 1]].double()
    return dict(attn=attn.reshape(s["attn"].shape), lse=lse.reshape(s["lse"].shape))


def exact(case, seed):
    """What run() returns for these inputs in 64 bits: scores, or the attention's output; budgets, indices and copied
    rows are whole values and have none."""
    if case["path"] == "compress":
        return None
    s = prepare(case, seed)
    if case["path"] == "decode":
        return _exact_decode(s)
    scores, at = [], 0
    for N in _lens_of(case):
        of_layers = []
        for l in range(case["L"]):
            k = (s["hold"][0][l] if s["hold"][0] else s["keys"][l])[:, at:at + N]
            of_layers.append(torch.cat([_exact_scores(x.double()) for x in k.split(8)]))
        of_prompt = torch.stack(of_layers)
        scores.append((of_prompt[:, :, :N_SINK], of_prompt[:, :, N_SINK:]))
        at += N
    if case["path"] == "score":
        return scores
    return {name: scores if name == "scores" else None for name in s["out"]}
