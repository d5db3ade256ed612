"""The calls whose speed is watched: one tensor-parallel rank's share of LLaMA2-shaped decoder blocks with the
Sync-Point-Drop wiring, through spd_block_forward() and spd_model_forward(), and the fp32 toy model with every rank
emulated.  Shapes are those of paper_2502_20727_amd/workloads.py; batch, tokens per sequence and context cover what a
serving program asks for: decode steps from one sequence to SPD_MAX_BATCH of them, short prompts, chunks of a prompt
behind an existing context, long prompts, and prompts of several sequences at once.

A case is a dict:
  model    "toy" | "7b" | "13b" | "70b"        tp       tensor-parallel degree (rank 0 runs; "toy": all ranks)
  entry    "block" (spd_block_forward) | "model" (spd_model_forward)
  mask     one character per layer: "1" SPD block, "0" TP block (attention sync point kept)
  batch, q_len   sequences and tokens per sequence of the call
  ctx      positions already in the cache of the longest sequence
  ragged   the sequences' contexts differ (spread over ctx/4 .. ctx)
  bias     the output projection has a bias
"""
from dataclasses import replace

import numpy as np
import torch

from paper_2502_20727_amd import binding as B
from paper_2502_20727_amd import workloads as W

MODELS = {"toy": W.TOY, "7b": W.LLAMA7B_DECODE, "13b": W.LLAMA13B_DECODE, "70b": W.LLAMA70B_DECODE}


def _case(name, model, mask, batch, q_len, ctx, entry="block", tp=8, ragged=False, bias=False):
    return {"name": name, "model": model, "tp": tp, "entry": entry, "mask": mask, "batch": batch, "q_len": q_len,
            "ctx": ctx, "ragged": ragged, "bias": bias}


def listed():
    return [
        # one decode step of the toy model, fp32, both ranks emulated: the smallest call there is
        _case("toy-f32-step", "toy", "10", 1, 1, 39, entry="model", tp=2),
        # the toy model's prompt of 32 tokens
        _case("toy-f32-prefill-32", "toy", "10", 1, 32, 0, entry="model", tp=2),
        # interactive decoding of one sequence, small model: launches and latencies
        _case("7b-decode-b1-ctx2048", "7b", "1", 1, 1, 2047),
        # decoding of a small batch, four layers of a model of which every fourth keeps its attention sync point;
        # multi-head attention over long caches
        _case("13b-decode-b8-ctx4096-4-layers", "13b", "1110", 8, 1, 4095, entry="model"),
        # the headline decode shape: a batch of 16 at context 4096, four layers of the model
        _case("70b-decode-b16-ctx4096-4-layers", "70b", "1101", 16, 1, 4095, entry="model"),
        # continuous batching: 48 sequences of different lengths, attention sync point kept
        _case("70b-decode-b48-ragged", "70b", "0", 48, 1, 3000, ragged=True),
        # a short prompt (the shape of the paper's latency breakdown)
        _case("70b-prefill-1x128", "70b", "1", 1, 128, 0),
        # an odd prompt length, block with bias, attention sync point kept
        _case("13b-prefill-1x333-bias", "13b", "0", 1, 333, 0, bias=True),
        # a chunk of 512 tokens of a long prompt: attends to the 1536 positions before it
        _case("70b-prefill-chunk-512", "70b", "1", 1, 512, 1536),
        # one prompt of a thousand tokens
        _case("70b-prefill-1x1000", "70b", "1", 1, 1000, 0),
        # one long prompt on a small model, attention sync point kept
        _case("7b-prefill-1x2048", "7b", "0", 1, 2048, 0),
        # four prompts of 2048 tokens, two layers, one of each kind: the headline prefill shape
        _case("70b-prefill-4x2048-2-layers", "70b", "10", 4, 2048, 0, entry="model"),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    """One more call of the same ranges."""
    kind = rng.choices(["toy", "decode", "short", "long", "batch"], [1, 4, 3, 2, 1])[0]
    model = rng.choice(["7b", "13b", "70b"])
    tp = 8 if model == "70b" else rng.choice([4, 8])
    flag = rng.choice("01")
    bias = rng.random() < 0.2
    if kind == "toy":
        q_len = _log_int(rng, 1, 40)
        c = _case("", "toy", rng.choice(["10", "11", "00"]), 1, q_len, rng.randrange(0, 64 - q_len), entry="model", tp=2)
    elif kind == "decode":
        batch = _log_int(rng, 1, 64)
        ctx = _log_int(rng, 32, max(64, min(16000, 65536 // batch)))
        c = _case("", model, flag, batch, 1, ctx, tp=tp, ragged=rng.random() < 0.5, bias=bias)
    elif kind == "short":
        q_len = _log_int(rng, 17, 512)
        batch = rng.randrange(1, max(1, min(4, 512 // q_len)) + 1)
        c = _case("", model, flag, batch, q_len, rng.choice([0, 0, _log_int(rng, 32, 6000)]), tp=tp, bias=bias)
    elif kind == "long":
        c = _case("", model, flag, 1, _log_int(rng, 513, 5000), rng.choice([0, 0, _log_int(rng, 32, 3000)]), tp=tp, bias=bias)
    else:
        batch = rng.randrange(2, 6)
        lo = 1024 // (batch // 2)
        c = _case("", model, rng.choice(["10", "11", "01"]), batch, _log_int(rng, lo, max(lo + 64, 8192 // batch)), 0,
                  entry="model", tp=tp)
    del c["name"]
    return c


# ------------------------------------------------------------------------------------------------ inputs

def _workload(case):
    w = MODELS[case["model"]]
    mask = tuple(int(m) for m in case["mask"])
    return replace(w, tp=case["tp"], n_layers=len(mask), mask=mask, batch=case["batch"], q_len=case["q_len"])


def _ranks(case):
    return list(range(case["tp"])) if case["model"] == "toy" else [0]


def _generator(seed, *key):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1000003 + sum((k + 1) * 7919 ** (i + 1) for i, k in enumerate(key))) % (2 ** 62))
    return g


def _positions(case, seed):
    b, ctx = case["batch"], case["ctx"]
    if not case["ragged"]:
        return [ctx] * b
    return [ctx] + [int(p) for p in np.random.RandomState(seed % (2 ** 31)).randint(ctx // 4, ctx + 1, size=b - 1)]


def _max_ctx(case):
    return (case["ctx"] + case["q_len"] + 31) // 32 * 32


def _weights(case, w, seed, layer, rank):
    """A rank's slices of one layer, fp32 on the GPU: linear weights N(0, 0.02), bf16 values for the bf16 models."""
    def mat(i, rows, cols):
        t = torch.randn(rows, cols, generator=_generator(seed, 1, layer, rank, i), device="cuda") * 0.02
        return t if w.dtype == W.F32 else t.bfloat16().float()

    h, d, q, kv, f = w.hidden, w.head_dim, w.q_per_rank, w.kv_per_rank, w.ffn_per_rank
    out = {"wq": mat(0, h, q * d), "wk": mat(1, h, kv * d), "wv": mat(2, h, kv * d), "wo": mat(3, q * d, h),
           "wg": mat(4, h, f), "wu": mat(5, h, f), "wd": mat(6, f, h)}
    for i, n in enumerate(("g1", "g2")):        # gains are replicated on every rank
        out[n] = 1.0 + 0.02 * torch.randn(h, generator=_generator(seed, 2, layer, i), device="cuda")
    if case["bias"]:
        out["bo"] = 0.02 * torch.randn(h, generator=_generator(seed, 3, layer), device="cuda")
    return out


def _cache(case, w, seed, layer, rank, positions):
    """Keys (already rotated) and values of the positions before the call: [batch, kv, ctx, d], N(0, 1)."""
    shape = (case["batch"], w.kv_per_rank, case["ctx"], w.head_dim)
    out = []
    for i in range(2):
        t = torch.randn(shape, generator=_generator(seed, 4, layer, rank, i), device="cuda")
        t = t if w.dtype == W.F32 else t.bfloat16().float()
        if case["ragged"]:
            live = torch.arange(case["ctx"], device="cuda")[None, :] < torch.tensor(positions, device="cuda")[:, None]
            t = t * live[:, None, :, None]
        out.append(t)
    return out


def _stream_inputs(case, w, seed):
    """Residual stream N(0, 1) and the partial sums met at the sync points (the peers' are inputs), 0.05 N(0, 1)."""
    tokens = case["batch"] * case["q_len"]
    x = torch.randn(tokens, w.hidden, generator=_generator(seed, 5), device="cuda")
    slots = torch.randn(w.tp, tokens, w.hidden, generator=_generator(seed, 6), device="cuda").mul_(0.05)
    return x, slots


class _State:
    pass


def prepare(case, seed):
    w, ranks, positions = _workload(case), _ranks(case), _positions(case, seed)
    tokens = case["batch"] * case["q_len"]
    s = _State()
    s.case, s.w, s.positions = case, w, positions
    s.shard = B.DeviceShard(w, ranks, torch.device("cuda"), max_ctx=_max_ctx(case), max_tokens=tokens,
                            max_batch=case["batch"], o_bias=int(case["bias"]))
    for l in range(w.n_layers):
        s.shard.load_layer(l, [{n: t.cpu().numpy() for n, t in _weights(case, w, seed, l, r).items()} for r in ranks])
        if case["ctx"]:
            s.shard.load_kv(l, [tuple(t.cpu().numpy() for t in _cache(case, w, seed, l, r, positions)) for r in ranks])
    s.x, s.slots = _stream_inputs(case, w, seed)
    s.out = torch.empty_like(s.x)
    s.kv = [t.view(torch.float32 if w.dtype == W.F32 else torch.bfloat16) for t in s.shard.kv]
    return s


def run(s):
    c, sh = s.case, s.shard
    if c["entry"] == "model":
        B.spd_model_forward(sh.ctx, s.w.mask, sh.rank_arg(), sh.weights, sh.kv, s.positions, c["batch"], c["q_len"], s.x,
                            s.slots, s.out, sh.workspace)
    else:
        B.spd_block_forward(sh.ctx, 0, s.w.mask[0], sh.rank_arg(), sh.weights[0], sh.kv[0], s.positions, c["batch"],
                            c["q_len"], s.x, s.slots, s.out, sh.workspace)
    # the block output, the partial sums this process wrote, and the caches with the appended keys and values
    return {"x": s.out, "slots": s.slots if c["model"] == "toy" else s.slots[0], "kv": s.kv}


# ------------------------------------------------------------------------------------------------ cost and reference

def work(case):
    w = _workload(case)
    nr, L, M = len(_ranks(case)), w.n_layers, case["batch"] * case["q_len"]
    es = 4 if w.dtype == W.F32 else 2
    h, d, q, kv, f = w.hidden, w.head_dim, w.q_per_rank, w.kv_per_rank, w.ffn_per_rank
    n_weights = h * (q + 2 * kv) * d + q * d * h + 3 * h * f
    contexts = _positions(case, 0)
    kv_bytes = sum(2 * kv * d * es * (p + case["q_len"]) for p in contexts)      # context read, new positions written
    keys = sum(case["q_len"] * p + case["q_len"] * (case["q_len"] + 1) // 2 for p in contexts)
    # the residual stream in and out once; per layer the peers' partial sums in and the own ones out
    stream = 2 * M * h * 4 + L * M * h * 4 * w.tp
    return {"bytes": nr * L * (n_weights * es + kv_bytes) + stream,
            "flops": nr * L * (2 * M * n_weights + 4 * q * d * keys)}


def tolerance(case):
    # about four times the largest distance from exact() measured over the listed cases and some drawn ones
    if case["model"] == "toy":
        return {"rel": 2e-6, "max": 1e-5}        # fp32 throughout: 5e-7, 2.2e-6
    # fp16 projection operands, bf16 cache, fp32 sums: 5.5e-4 for one layer, 1.1e-3 for two layers of a prefill; single
    # elements 9e-3 (and 2^-7 where the last place of a bf16 key or value differs)
    return {"rel": 2.2e-3 if len(case["mask"]) == 1 else 4.5e-3, "max": 4e-2}


def _rotate(t, positions, w):
    """Rotary embedding, rotate-half, of t [batch, q_len, heads, d] (float64)."""
    d = w.head_dim
    theta = w.rope_base ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device="cuda") / d)
    pos = torch.tensor(positions, dtype=torch.float64, device="cuda")[:, None] + torch.arange(t.shape[1], device="cuda")
    a = pos[:, :, None, None] * theta
    lo, hi = t[..., :d // 2], t[..., d // 2:]
    return torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], dim=-1)


def _norm(t, g, eps):
    return t / torch.sqrt((t * t).mean(dim=-1, keepdim=True) + eps) * g


def _stored(t, w):
    return t if w.dtype == W.F32 else t.to(torch.bfloat16).double()     # the cache holds bf16 values


def _layout(k, v, w):
    """[batch, kv, max_ctx, d] float64 -> the cache as the library lays it out, flat."""
    if w.dtype == W.F32:
        return torch.cat([k.reshape(-1), v.reshape(-1)])
    b, n, c, d = k.shape
    # keys: blocks of 16 positions, d / 32 fragments of (4 groups of 8 features, 16 positions, 8 features)
    kp = k.reshape(b, n, c // 16, 16, d // 32, 4, 8).permute(0, 1, 2, 4, 5, 3, 6)
    # values: blocks of 32 positions (half, group, place), d / 16 fragments of (4 groups, 16 features, half, place)
    vp = v.reshape(b, n, c // 32, 2, 4, 4, d // 16, 16).permute(0, 1, 2, 6, 4, 7, 3, 5)
    return torch.cat([kp.reshape(-1), vp.reshape(-1)])


def _attention_partial(case, w, wt, kc, vc, x, positions):
    """Appends to the caches (in place) and returns Y_r [tokens, h]."""
    b, n, d, q, kv = case["batch"], case["q_len"], w.head_dim, w.q_per_rank, w.kv_per_rank
    xn = _norm(x, wt["g1"], w.rms_eps)
    qs = _rotate((xn @ wt["wq"]).view(b, n, q, d), positions, w)
    ks = _stored(_rotate((xn @ wt["wk"]).view(b, n, kv, d), positions, w), w)
    vs = _stored((xn @ wt["wv"]).view(b, n, kv, d), w)
    out = torch.empty(b, n, q, d, dtype=torch.float64, device="cuda")
    for i, p in enumerate(positions):
        kc[i, :, p:p + n] = ks[i].transpose(0, 1)
        vc[i, :, p:p + n] = vs[i].transpose(0, 1)
        hide = torch.arange(p + n, device="cuda")[None, :] > p + torch.arange(n, device="cuda")[:, None]
        for j in range(q):
            g = j // (q // kv)
            sc = (qs[i, :, j] @ kc[i, g, :p + n].t()) / d ** 0.5
            out[i, :, j] = torch.softmax(sc.masked_fill_(hide, float("-inf")), dim=-1) @ vc[i, g, :p + n]
    return out.view(b * n, q * d) @ wt["wo"]


def _mlp_partial(w, wt, r):
    m = _norm(r, wt["g2"], w.rms_eps)
    g = m @ wt["wg"]
    return (g * torch.sigmoid(g) * (m @ wt["wu"])) @ wt["wd"]


def exact(case, seed):
    w, ranks, positions = _workload(case), _ranks(case), _positions(case, seed)
    x32, slots32 = _stream_inputs(case, w, seed)
    x = x32.double()
    own = [slots32[r].double() for r in ranks]
    peers = torch.zeros_like(x)                  # the partial sums of the ranks that do not run here never change
    for r in range(w.tp):
        if r not in ranks:
            peers += slots32[r]
    del x32, slots32
    caches = []
    for l, flag in enumerate(w.mask):
        wts = [{k: t.double() for k, t in _weights(case, w, seed, l, r).items()} for r in ranks]
        bias = wts[0]["bo"] if case["bias"] else 0.0
        layer = []
        for r in ranks:
            kc, vc = (torch.zeros(case["batch"], w.kv_per_rank, _max_ctx(case), w.head_dim, dtype=torch.float64,
                                  device="cuda") for _ in range(2))
            k, v = _cache(case, w, seed, l, r, positions)
            kc[:, :, :case["ctx"]] = k
            vc[:, :, :case["ctx"]] = v
            layer.append((kc, vc))
        ys = [_attention_partial(case, w, wt, kc, vc, x, positions) for wt, (kc, vc) in zip(wts, layer)]
        if flag:
            own = [y + _mlp_partial(w, wt, x + y + bias) for wt, y in zip(wts, ys)]
            x = x + (peers + sum(own)) + bias
        else:
            r = x + (peers + sum(ys)) + bias
            own = [_mlp_partial(w, wt, r) for wt in wts]
            x = r + (peers + sum(own))
        caches.append(torch.cat([_layout(k, v, w) for k, v in layer]))
    return {"x": x, "slots": torch.stack(own) if case["model"] == "toy" else own[0], "kv": caches}
