"""The decode-step work that a user of this library has it do, as measurable cases.

Four kinds of pass, each over one or more layers of a model (every layer has
weights and KV caches of its own, as in a model, so that what one layer reads
has left the caches by the time the next pass comes to it):

* ``attention``: paged decode attention of the step's query tokens, through
  ``paged_decode_attention`` or, with several query tokens or a sliding
  window, ``paged_decode_attention_ext``;
* ``prelude``: QKV projection, Q/K RMSNorm and rotation, with the new token's
  k and v appended to the paged cache or returned;
* ``oproj``: output projection, residual add and RMSNorm;
* ``block``: a layer's whole attention block, the three in turn.

A case fixes the set of context lengths; the seed decides which sequence has
which, where the pages lie in the pool, and every value.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2606_07665_amd import binding as pda

THETA = 5.0e5
EPS_QK = 1e-6
EPS_OUT = 1e-5
#: Layers of a pass read at least this much together, more than the last-level cache holds.
COLD_BYTES = 400_000_000
MAX_LAYERS = 16


def _attention(**kw):
    return dict(dict(kind="attention", batch=1, hq=32, hkv=8, d=128, page=16, lengths="fixed:4096",
                     capacity=0, queries=1, window=0, layers=1), **kw)


def _prelude(**kw):
    return dict(dict(kind="prelude", batch=1, hidden=4096, hq=32, hkv=8, d=128, page=16, lengths="fixed:1024",
                     append=False, qk_norm=False, bias=False, rotary=128, interleaved=False, layers=1), **kw)


def _oproj(**kw):
    return dict(dict(kind="oproj", batch=1, features=4096, hidden=4096, layers=1), **kw)


def _block(**kw):
    return dict(dict(kind="block", batch=1, hidden=4096, hq=32, hkv=8, d=128, page=16, lengths="fixed:4096",
                     capacity=0, qk_norm=False, bias=False, rotary=128, interleaved=False, layers=1), **kw)


def listed():
    return [
        # one interactive request on an 8B model, half-way through its 8192-token table: latency
        _attention(name="attn_single_8b", lengths="fixed:4096", capacity=8192, layers=16),
        # continuous batching on an 8B model: ordinary serving
        _attention(name="attn_batched_8b", batch=64, lengths="uniform:128:8192"),
        # a few very long documents on a 70B model
        _attention(name="attn_long_70b", batch=4, hq=64, lengths="fixed:131072"),
        # a large batch with a heavy-tailed length mix, 40 query heads, 32-token pages: the largest
        _attention(name="attn_ragged_256", batch=256, hq=40, page=32, lengths="zipf:1.2:16:32768"),
        # verification of four drafted tokens under a sliding window
        _attention(name="attn_draft4_window", batch=64, lengths="uniform:1024:16384", queries=4, window=4096),
        # head size 256, three query heads per kv head, a small batch of mixed lengths
        _attention(name="attn_d256_b16", batch=16, hq=12, hkv=4, d=256, lengths="uniform:16:32768"),
        # one request's prelude on a 4B model with Q/K norm, appended to the cache
        _prelude(name="prelude_b1_4b", hidden=2560, lengths="fixed:4096", append=True, qk_norm=True, layers=13),
        # a serving batch's prelude on an 8B model
        _prelude(name="prelude_b64_8b", batch=64, lengths="uniform:128:8192", layers=8),
        # the largest batch's prelude, 40 query heads
        _prelude(name="prelude_b256_40h", batch=256, hidden=5120, hq=40, lengths="uniform:16:32768", layers=6),
        # output projection of a 70B model at a small batch
        _oproj(name="oproj_b4_70b", batch=4, features=8192, hidden=8192, layers=4),
        # output projection at an odd batch, as continuous batching leaves it
        _oproj(name="oproj_b100_40h", batch=100, features=5120, hidden=5120, layers=8),
        # a whole attention block per layer, four layers of an 8B model at a moderate batch
        _block(name="block_b16_8b", batch=16, lengths="uniform:128:8192", layers=4),
    ]


# (hidden, query heads, kv heads, head size, options): the model shapes of the repository's workloads
_MODELS = (
    (2560, 32, 8, 128, dict(qk_norm=True)),
    (4096, 32, 8, 128, {}),
    (8192, 64, 8, 128, {}),
    (4096, 32, 2, 128, dict(bias=True, rotary=64, interleaved=True)),
    (3072, 12, 4, 256, dict(rotary=256)),
    (5120, 40, 8, 128, {}),
)


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def _layers_for(bytes_per_layer):
    return max(1, min(MAX_LAYERS, -(-COLD_BYTES // max(1, int(bytes_per_layer)))))


def _draw_lengths(rng, batch, mean):
    mean = max(16, min(131072, int(mean)))
    form = rng.choice(("fixed", "uniform", "uniform", "zipf"))
    if batch == 1 or form == "fixed":
        return "fixed:%d" % mean
    if form == "zipf" and batch >= 16:
        return "zipf:1.2:16:%d" % min(32768, 2 * mean + 16)
    return "uniform:%d:%d" % (max(16, mean // 8), 2 * mean - max(16, mean // 8) if mean > 32 else mean + 16)


def draw(rng):
    kind = rng.choice(("attention",) * 6 + ("prelude",) * 5 + ("oproj",) * 4 + ("block",) * 3)
    hidden, hq, hkv, d, opts = rng.choice(_MODELS)
    batch = _log_int(rng, 1, 256)
    if kind == "oproj":
        c = _oproj(batch=batch, features=hq * d, hidden=hidden)
        c["layers"] = _layers_for(2 * hidden * hq * d)
        return c
    if kind == "prelude":
        append = rng.random() < 0.5
        c = _prelude(batch=batch, hidden=hidden, hq=hq, hkv=hkv, d=d, append=append, page=rng.choice((16, 16, 32, 64)),
                     lengths=_draw_lengths(rng, batch, _log_int(rng, 16, 512) if append else _log_int(rng, 16, 65536)),
                     **opts)
        c["layers"] = min(6 if append else MAX_LAYERS, _layers_for(2 * hidden * (hq + 2 * hkv) * d))
        return c
    page = rng.choice((1, 16, 16, 16, 32, 64))
    token = 4 * hkv * d  # bytes of K and V per token
    if kind == "block":
        c = _block(batch=batch, hidden=hidden, hq=hq, hkv=hkv, d=d, page=max(16, page), **opts)
        weights = 2 * hidden * (2 * hq + 2 * hkv) * d
        kv = math.exp(rng.uniform(math.log(4e6), math.log(4e8)))
        c["lengths"] = _draw_lengths(rng, batch, kv / (batch * token))
        c["layers"] = min(4, _layers_for(weights + kv))
        return c
    c = _attention(batch=batch, hq=hq, hkv=hkv, d=d, page=page)
    group = hq // hkv
    if rng.random() < 0.3:
        c["queries"] = rng.randint(1, max(1, min(8, 16 // group)))
    if rng.random() < 0.25:
        c["window"] = rng.choice((512, 1024, 4096))
    c["lengths"] = _draw_lengths(rng, batch, math.exp(rng.uniform(math.log(4e6), math.log(2.5e9))) / (batch * token))
    lens = _lens(c)
    if batch <= 8:
        c["capacity"] = int(max(lens)) * rng.choice((1, 1, 2))
    c["layers"] = _layers_for(_attention_bytes(c))
    return c


# ------------------------------------------------------------------ inputs
def _lens(case):
    """The case's context lengths, the new tokens included (ascending order not implied)."""
    b = case["batch"]
    kind, *args = case["lengths"].split(":")
    if kind == "fixed":
        lens = np.full(b, int(args[0]), dtype=np.int64)
    elif kind == "uniform":
        lo, hi = int(args[0]), int(args[1])
        lens = (lo + (hi - lo) * (np.arange(b) + 0.5) / b).astype(np.int64)
    else:
        s, lo, hi = float(args[0]), int(args[1]), int(args[2])
        lens = np.clip(np.random.default_rng([b, hi]).zipf(s, size=b).astype(np.int64), lo, hi)
    return np.maximum(lens, case.get("queries", 1))


def _table(case, seed):
    """(block table, lengths, pages in the pool): pages of a shuffled pool with a tenth of it unused."""
    rng = np.random.default_rng([seed, 7])
    lens = rng.permutation(_lens(case))
    page = case["page"]
    pages = (lens + page - 1) // page
    pool = int(pages.sum()) + int(pages.sum()) // 10 + 1
    width = max(int(pages.max()), -(-case.get("capacity", 0) // page))
    ids = rng.permutation(pool)
    table = np.full((case["batch"], width), -1, dtype=np.int32)
    at = 0
    for i, n in enumerate(pages):
        table[i, :n] = ids[at:at + n]
        at += int(n)
    return torch.from_numpy(table).cuda(), torch.from_numpy(lens.astype(np.int32)).cuda(), pool


class _Values:
    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(1_000_003 * (seed + 1))

    def normal(self, *shape, std=1.0, mean=0.0):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(mean, std, generator=self.gen)


def _weights(case, v):
    """Prelude weights of one layer: plain, for exact(), and packed, as a program keeps them."""
    rows = (case["hq"] + 2 * case["hkv"]) * case["d"]
    w = v.normal(rows, case["hidden"], std=case["hidden"] ** -0.5)
    return dict(w=w, bias=v.normal(rows, std=0.1) if case["bias"] else None,
                q_norm=v.normal(case["d"], std=0.1, mean=1.0) if case["qk_norm"] else None,
                k_norm=v.normal(case["d"], std=0.1, mean=1.0) if case["qk_norm"] else None)


def _inputs(case, seed):
    """Everything the seed decides, layer by layer."""
    v = _Values(seed)
    kind, b = case["kind"], case["batch"]
    state = dict(case=case)
    if kind != "oproj":
        state["table"], state["lens"], pool = _table(case, seed)
    layers = []
    for _ in range(case["layers"]):
        s = {}
        if kind == "attention":
            shape = (b, case["hq"], case["d"])
            if case["queries"] > 1 or case["window"]:
                shape = (b, case["queries"], case["hq"], case["d"])
            s["q"] = v.normal(*shape)
        if kind in ("prelude", "block"):
            s.update(_weights(case, v))
            s["x"] = v.normal(b, case["hidden"])
        if kind in ("oproj", "block"):
            features = case["features"] if kind == "oproj" else case["hq"] * case["d"]
            s["w_o"] = v.normal(case["hidden"], features, std=features ** -0.5)
            s["residual"] = v.normal(b, case["hidden"])
            s["norm_w"] = v.normal(case["hidden"], std=0.1, mean=1.0)
            if kind == "oproj":
                s["attn"] = v.normal(b, features)
        if kind in ("attention", "block") or case.get("append"):
            s["k"] = v.normal(pool, case["page"], case["hkv"], case["d"])
            s["v"] = v.normal(pool, case["page"], case["hkv"], case["d"])
        layers.append(s)
    state["layers"] = layers
    return state


def prepare(case, seed):
    state = _inputs(case, seed)
    kind, b = case["kind"], case["batch"]
    for s in state["layers"]:
        if "w" in s:
            s["w"] = pda.pack_weights(s["w"])
            s["q"] = torch.empty((b, case["hq"], case["d"]), dtype=torch.bfloat16, device="cuda")
            if kind == "prelude" and not case["append"]:
                s["k_out"], s["v_out"] = (torch.empty((b, case["hkv"], case["d"]), dtype=torch.bfloat16, device="cuda")
                                          for _ in range(2))
        if kind in ("attention", "block"):
            s["out"] = torch.empty_like(s["q"])
        if "w_o" in s:
            s["w_o"] = pda.pack_weights(s["w_o"])
            s["z"], s["h"] = torch.empty_like(s["residual"]), torch.empty_like(s["residual"])
    if kind != "oproj":
        state["scale"] = case["d"] ** -0.5
        state["shape"] = dict(num_q_heads=case["hq"], num_kv_heads=case["hkv"], head_dim=case["d"])
    if kind in ("prelude", "block"):
        state["shape"].update(rope_theta=THETA, rotary_dim=case["rotary"], interleaved=case["interleaved"], eps=EPS_QK)
    return state


# -------------------------------------------------------------------- pass
def _run_prelude_append(state, s):
    pda.attention_prelude_append(s["x"], s["w"], state["lens"], s["q"], s["k"], s["v"], state["table"],
                                 bias=s["bias"], q_norm=s["q_norm"], k_norm=s["k_norm"], **state["shape"])


def run(state):
    case = state["case"]
    kind = case["kind"]
    outs = []
    for s in state["layers"]:
        if kind == "attention":
            if case["queries"] > 1 or case["window"]:
                pda.paged_decode_attention_ext(s["q"], s["k"], s["v"], state["table"], state["lens"], s["out"],
                                               state["scale"], window=case["window"])
            else:
                pda.paged_decode_attention(s["q"], s["k"], s["v"], state["table"], state["lens"], s["out"],
                                           state["scale"])
            outs.append(s["out"])
        elif kind == "prelude":
            if case["append"]:
                _run_prelude_append(state, s)
                outs.append((s["q"], s["k"], s["v"]))
            else:
                pda.attention_prelude(s["x"], s["w"], state["lens"], s["q"], s["k_out"], s["v_out"], bias=s["bias"],
                                      q_norm=s["q_norm"], k_norm=s["k_norm"], **state["shape"])
                outs.append((s["q"], s["k_out"], s["v_out"]))
        elif kind == "oproj":
            pda.o_proj_residual_norm(s["attn"], s["w_o"], s["residual"], s["norm_w"], s["z"], s["h"], eps=EPS_OUT)
            outs.append((s["z"], s["h"]))
        else:
            _run_prelude_append(state, s)
            pda.paged_decode_attention(s["q"], s["k"], s["v"], state["table"], state["lens"], s["out"],
                                       state["scale"])
            pda.o_proj_residual_norm(s["out"].view(case["batch"], -1), s["w_o"], s["residual"], s["norm_w"], s["z"],
                                     s["h"], eps=EPS_OUT)
            outs.append((s["k"], s["v"], s["z"], s["h"]))
    return outs


# ---------------------------------------------------------- what it cannot do without
def _live_tokens(case):
    lens = _lens(case)
    if not case.get("window"):
        return int(lens.sum())
    start = np.maximum(0, lens - case["queries"] + 1 - case["window"])
    return int((lens - start).sum())


def _attention_bytes(case):
    """K and V of every visible token once, q in, out out, the page ids and lengths (one layer)."""
    b, tokens = case["batch"], _live_tokens(case)
    q = 2 * b * case.get("queries", 1) * case["hq"] * case["d"]
    return 4 * case["hkv"] * case["d"] * tokens + 2 * q + 4 * (tokens // case["page"] + b) + 4 * b


def work(case):
    kind, b = case["kind"], case["batch"]
    nbytes = flops = 0
    if kind in ("attention", "block"):
        nbytes += _attention_bytes(case)
        flops += 4 * case.get("queries", 1) * case["hq"] * case["d"] * _live_tokens(case)
    if kind in ("prelude", "block"):
        rows = (case["hq"] + 2 * case["hkv"]) * case["d"]
        nbytes += 2 * rows * case["hidden"] + 2 * b * (case["hidden"] + rows) + (2 * rows if case["bias"] else 0)
        flops += 2 * b * rows * case["hidden"]
    if kind in ("oproj", "block"):
        hidden, features = case["hidden"], case["features"] if kind == "oproj" else case["hq"] * case["d"]
        nbytes += 2 * hidden * features + 2 * b * features + 6 * b * hidden + 2 * hidden
        flops += 2 * b * hidden * features
    return {"bytes": nbytes * case["layers"], "flops": flops * case["layers"]}


def tolerance(case):
    # Measured against exact(): outputs rounded once to bf16 from 32-bit sums are 1.7e-3 off (2-norm) and at
    # most half a bf16 spacing, 3.9e-3 of the value; in a block the rounding of q, k, v and of the attention
    # output between its steps stays below that of z and h themselves.  Four times what is seen.
    return {"rel": 7e-3, "max": 1.6e-2}


# ------------------------------------------------------------ the same in 64 bits
def _f32(x):
    """The value the entry points take: they hold scalars in 32 bits."""
    return float(np.float32(x))


def _exact_attention(case, q, k, v, table, lens):
    """softmax(scale q K^T) V over each sequence's pages; q [B, Tq, Hq, D] in any type."""
    b, tq, hq, d = q.shape
    hkv, page = case["hkv"], case["page"]
    scale, group = _f32(d ** -0.5), hq // hkv
    out = torch.zeros((b, tq, hq, d), dtype=torch.float64, device=q.device)
    for i, n in enumerate(lens.tolist()):
        ids = table[i, : -(-n // page)].long()
        first = max(0, n - tq + 1 - case["window"]) // page if case.get("window") else 0
        t0 = first * page
        qi = q[i].double().reshape(tq, hkv, group, d).permute(1, 0, 2, 3).reshape(hkv, tq * group, d).contiguous()
        ki = k[ids[first:]].reshape(-1, hkv, d)[: n - t0].double().permute(1, 2, 0).contiguous()
        s = torch.bmm(qi, ki).mul_(scale).view(hkv, tq, group, n - t0)
        del ki
        pos = torch.arange(t0, n, device=q.device)
        last = torch.arange(n - tq, n, device=q.device)[:, None]
        hide = pos[None] > last
        if case.get("window"):
            hide |= pos[None] <= last - case["window"]
        s.masked_fill_(hide[None, :, None], -math.inf)
        p = torch.softmax(s, dim=-1).view(hkv, tq * group, n - t0)
        vi = v[ids[first:]].reshape(-1, hkv, d)[: n - t0].double().permute(1, 0, 2).contiguous()
        o = torch.bmm(p, vi)
        out[i] = o.view(hkv, tq, group, d).permute(1, 0, 2, 3).reshape(tq, hq, d)
    return out


def _exact_prelude(case, s, lens):
    b, hq, hkv, d, r = case["batch"], case["hq"], case["hkv"], case["d"], case["rotary"]
    y = s["x"].double() @ s["w"].double().t().contiguous()
    if s["bias"] is not None:
        y = y + s["bias"].double()
    y = y.view(b, hq + 2 * hkv, d)
    q, k, v = y[:, :hq], y[:, hq: hq + hkv], y[:, hq + hkv:]
    i = torch.arange(r // 2, dtype=torch.float64, device=y.device)
    angle = (lens.double() - 1)[:, None] * _f32(THETA) ** (-2.0 * i / r)
    sin, cos = angle.sin()[:, None], angle.cos()[:, None]

    def turned(t, weight):
        if weight is not None:
            t = t * torch.rsqrt(t.square().mean(-1, keepdim=True) + _f32(EPS_QK)) * weight.double()
        out = t.clone()
        lo, hi = (slice(0, r, 2), slice(1, r, 2)) if case["interleaved"] else (slice(0, r // 2), slice(r // 2, r))
        out[..., lo] = t[..., lo] * cos - t[..., hi] * sin
        out[..., hi] = t[..., hi] * cos + t[..., lo] * sin
        return out

    return turned(q, s["q_norm"]), turned(k, s["k_norm"]), v


def _exact_append(case, s, k_new, v_new, table, lens):
    at = lens.long() - 1
    pages = table.gather(1, (at // case["page"])[:, None]).squeeze(1).long()
    k, v = s["k"].double(), s["v"].double()
    k[pages, at % case["page"]] = k_new
    v[pages, at % case["page"]] = v_new
    return k, v


def _exact_oproj(attn, s):
    z = attn.double() @ s["w_o"].double().t().contiguous() + s["residual"].double()
    return z, z * torch.rsqrt(z.square().mean(-1, keepdim=True) + _f32(EPS_OUT)) * s["norm_w"].double()


def exact(case, seed):
    state = _inputs(case, seed)
    kind, table, lens = case["kind"], state.get("table"), state.get("lens")
    outs = []
    for s in state["layers"]:
        if kind == "attention":
            q = s["q"] if s["q"].dim() == 4 else s["q"].unsqueeze(1)
            outs.append(_exact_attention(case, q, s["k"], s["v"], table, lens).view(s["q"].shape))
        elif kind == "oproj":
            outs.append(_exact_oproj(s["attn"], s))
        else:
            q, k_new, v_new = _exact_prelude(case, s, lens)
            if kind == "prelude" and not case["append"]:
                outs.append((q, k_new, v_new))
                continue
            k, v = _exact_append(case, s, k_new, v_new, table, lens)
            if kind == "prelude":
                outs.append((q, k, v))
                continue
            attn = _exact_attention(case, q.unsqueeze(1), k, v, table, lens).view(case["batch"], -1)
            outs.append((k, v, *_exact_oproj(attn, s)))
        s.clear()
    return outs
