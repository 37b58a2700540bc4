"""What a generation or label-building program has this library do, as measurable cases.

Every case is a plain dict; `kind` says which calls of the library make one pass:

  cycle    the whole protocol at a small size: the L steps between two eviction events, then fk_score_kv, fk_select_keep
           and fk_compact (back to the budget, so that a pass can follow a pass)
  step     sequential decoding of one layer: one fk_decode_step call per generated token
  window   the steps between two events on tokens that are known beforehand (replay of a trace, log-probabilities of
           a rollout): one fk_decode_window call
  stack    one generated token through a stack of layers: one fk_decode_step per layer, every layer its own cache
  ragged   one generated token for a batch of sequences of very different lengths: one fk_decode_step
  score    the scorer of an eviction event or of a one-shot compression: fk_score_kv
  event    selection and compaction of an eviction event: fk_select_keep, fk_compact
  oneshot  selection and compaction of a long prompt before decoding starts: fk_select_keep_ws, fk_compact
  feat     a chunk of steps with the scorer's attention features, and the scores at its end: fk_score_kv_feat
  sampled  the sampled eviction policy with attention features: fk_select_keep_sampled, fk_compact_feat
  golden   the label builder on the attention of one full trace: fk_golden_scores, fk_golden_trace

cycle and feat come in two forms: `known` tokens (a replayed trace: one fk_decode_window / fk_decode_window_feat call) or
generated ones (one fk_decode_step / fk_decode_step_feat call per token).  Calls made per token are marshalled once with
fk.prepare, as a decoding loop does.

The listed sizes are the workloads of bench.py and synth_inputs.py plus one small head_dim 64 model; draw() spreads
them over the ranges a user meets: batch 1 to 64, 1 to 8 KV heads, group sizes 1 to 8, head_dim 64 and 128, rows of
a hundred to 131072 pairs, any length.  Selection gets its scores as an input except in `cycle` and `golden`: a pair
that sits at the cut to within rounding may fall on either side of it, and everything behind it moves by one slot.
Keys, values and queries are normal, one key in a hundred three times as long (sparse heavy keys).
"""
from __future__ import annotations

import math

import torch

import paper_2602_03203_amd as fk

PLANES = 6      # attention features per (pair, query head)
DECAY = 0.9     # of the carried feature sum, per chunk


def listed():
    return [
        # the tiny fp32 workload: launches and latency
        dict(name="cycle_tiny_f32", kind="cycle", dtype="f32", batch=1, hkv=2, g=4, d=64, budget=128, interval=32, hidden=64, known=False),
        # Qwen3-4B layer shape at the steady state of the protocol, token by token (the benchmark's headline shape)
        dict(name="step_b16", kind="step", dtype="bf16", batch=16, hkv=8, g=4, d=128, n=2112, steps=8),
        # a small model's layer, two sequences
        dict(name="step_small_d64", kind="step", dtype="bf16", batch=2, hkv=4, g=4, d=64, n=1500, steps=16),
        # the same layer shape as step_b16, the whole window between two events at once
        dict(name="window_b16", kind="window", dtype="bf16", batch=16, hkv=8, g=4, d=128, n=2048, steps=128),
        # one token through the 28-layer GQA-7 stack, caches in HBM
        dict(name="stack_gqa7", kind="stack", dtype="bf16", layers=28, batch=16, hkv=4, g=7, d=128, n=4128),
        # the ragged batch: initial lengths uniform in [1024, 32768]
        dict(name="ragged_b64", kind="ragged", dtype="bf16", batch=64, hkv=8, g=4, d=128, lo=1024, hi=32768),
        # an eviction event of the Qwen3-4B layer shape: score, then selection and compaction
        dict(name="score_event", kind="score", dtype="bf16", batch=16, hkv=8, g=4, d=128, n=2176, hidden=256),
        dict(name="event_topk", kind="event", dtype="bf16", batch=16, hkv=8, g=4, d=128, n=2176, budget=2048, recent=128, ties=False),
        # one-shot compression of a 131072-token prompt to 2048 pairs
        dict(name="oneshot_128k", kind="oneshot", dtype="bf16", batch=4, hkv=8, g=4, d=128, n=131072, budget=2048, recent=128, ties=False),
        # the paper's configuration, a chunk of a replayed trace: attention features, scorer of width 16; sampled eviction
        dict(name="feat_b16", kind="feat", dtype="bf16", batch=16, hkv=8, g=4, d=128, n=2048, steps=128, hidden=16, known=True),
        dict(name="sampled_b16", kind="sampled", dtype="bf16", batch=16, hkv=8, g=4, d=128, n=2176, budget=2048, recent=128, ties=False),
        # labels from one 8192-token trace of a 32-head layer
        dict(name="golden_8k", kind="golden", dtype="bf16", heads=32, hkv=8, tokens=8192, budget=2048, interval=128),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["cycle", "step", "window", "stack", "ragged", "score", "event", "oneshot", "feat", "sampled", "golden"])
    d = rng.choice([64, 128, 128])
    c = dict(kind=kind, dtype="bf16", batch=_log(rng, 1, 32), hkv=rng.choice([1, 2, 4, 8]), g=rng.choice([1, 2, 4, 4, 5, 7, 8]), d=d)
    rows = c["batch"] * c["hkv"]

    def length(lo, hi, pairs):   # a row length: spread over [lo, hi], the whole cache bounded
        return _log(rng, lo, max(lo, min(hi, pairs // rows)))
    if kind == "cycle":
        c.update(dtype=rng.choice(["f32", "bf16"]), batch=rng.randint(1, 4), hkv=rng.choice([1, 2, 4]), budget=_log(rng, 64, 512),
                 interval=rng.choice([8, 16, 32, 64]), hidden=rng.choice([16, 32, 64, 128]), known=rng.random() < 0.5)
    elif kind == "step":
        c.update(n=length(200, 16384, 1 << 20), steps=rng.choice([4, 8, 16]))
    elif kind == "window":
        c.update(n=length(100, 8192, 1 << 18), steps=rng.choice([16, 32, 64, 128]))
    elif kind == "stack":
        c.update(layers=rng.randint(8, 36), hkv=rng.choice([2, 4, 8]), batch=rng.choice([1, 2, 4, 8, 16]))
        rows = c["batch"] * c["hkv"]
        c.update(n=length(500, 16384, 1 << 18))
    elif kind == "ragged":
        c.update(batch=rng.randint(8, 64), lo=_log(rng, 1, 2000))
        c.update(hi=c["lo"] + _log(rng, 2000, 30000))
    elif kind == "score":
        c.update(n=length(300, 131072, 1 << 19), hidden=8 * _log(rng, 2, 32))
    elif kind == "event":
        b = length(200, 8192, 1 << 18)
        r = rng.choice([16, 64, 128])
        c.update(n=b + r + rng.choice([0, 0, _log(rng, 1, 200)]), budget=b, recent=r, ties=rng.random() < 0.5)
    elif kind == "oneshot":
        c.update(batch=rng.choice([1, 2, 4, 8]), hkv=rng.choice([2, 4, 8]))
        rows = c["batch"] * c["hkv"]
        c.update(n=length(16384, 131072, 1 << 22), budget=_log(rng, 500, 4000), recent=rng.choice([32, 128]), ties=rng.random() < 0.5)
    elif kind == "feat":
        c.update(n=length(100, 8192, 1 << 18), steps=rng.choice([16, 32, 64, 128]), hidden=rng.choice([16, 16, 64, 128]), known=rng.random() < 0.5)
    elif kind == "sampled":
        b = length(200, 8192, 1 << 18)
        r = rng.choice([16, 64, 128])
        c.update(n=b + r, budget=b, recent=r, ties=rng.random() < 0.5)
    else:
        c = dict(kind=kind, dtype=rng.choice(["bf16", "bf16", "f32"]), hkv=rng.choice([2, 4, 8]), tokens=_log(rng, 1500, 6000))
        c.update(heads=c["hkv"] * rng.choice([1, 2, 4]), budget=_log(rng, 256, min(2048, c["tokens"] // 2)), interval=rng.choice([32, 64, 128]))
    return c


# ---- inputs -------------------------------------------------------------------------------------------------------

def _dtype(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _randn(gen, shape, dtype):
    return torch.randn(shape, generator=gen, device="cuda", dtype=dtype)


def _cache(c, gen, batch, capacity):
    """K, V [batch][hkv][capacity][d] and ascending positions."""
    shape = (batch, c["hkv"], capacity, c["d"])
    K, V = _randn(gen, shape, _dtype(c)), _randn(gen, shape, _dtype(c))
    K *= 1.0 + 2.0 * (torch.rand((batch, 1, capacity, 1), generator=gen, device="cuda") < 0.01).to(K.dtype)
    pos = torch.arange(capacity, dtype=torch.int32, device="cuda").expand(batch, c["hkv"], capacity).contiguous()
    return K, V, pos


def _lens(c, values):
    return torch.tensor(values, dtype=torch.int32, device="cuda").reshape(-1, 1).repeat(1, c["hkv"]).contiguous()


def _tokens(c, gen, steps, batch):
    """q, k, v of `steps` generated tokens."""
    return (_randn(gen, (steps, batch, c["hkv"] * c["g"], c["d"]), _dtype(c)), _randn(gen, (steps, batch, c["hkv"], c["d"]), _dtype(c)),
            _randn(gen, (steps, batch, c["hkv"], c["d"]), _dtype(c)))


def _scorer(c, gen, features=0):
    F, H, S = 2 * c["d"], c["hidden"], c["hkv"]
    w1 = _randn(gen, (S, F, H), torch.float32) / math.sqrt(F)
    if features:
        w1 = torch.cat([w1, _randn(gen, (S, features, H), torch.float32) * (8.0 / math.sqrt(features))], dim=1)
    return (w1.to(_dtype(c)).contiguous(), _randn(gen, (S, H), torch.float32) / math.sqrt(F), _randn(gen, (S, H), torch.float32) / math.sqrt(H),
            _randn(gen, (S,), torch.float32) / math.sqrt(H))


def _scores(c, gen, shape, ties):
    s = torch.randn(shape, generator=gen, device="cuda")
    return torch.round(s * 64) / 64 if ties else s


def _desc(c, batch, capacity, cold=False):
    return fk.CacheDesc(batch, c["hkv"] * c["g"], c["hkv"], c["d"], capacity, c["dtype"], cold=cold)


def _capacity(n):
    return (n + 63) // 64 * 64


def prepare(c, seed):
    gen, kind = _gen(seed), c["kind"]
    s = dict(kind=kind)
    if kind == "golden":
        T = c["tokens"]
        ld = (T + 7) // 8 * 8
        A = torch.zeros((c["heads"], T, ld), dtype=_dtype(c), device="cuda")
        above = torch.ones((T, T), dtype=torch.bool, device="cuda").triu_(1)
        for h in range(c["heads"]):
            z = 1.5 * torch.randn((T, T), generator=gen, device="cuda")
            z += 3.0 * (torch.rand((T,), generator=gen, device="cuda") < 0.02).float()
            z[:, :4] += 4.0
            A[h, :, :T] = torch.softmax(z.masked_fill_(above, float("-inf")), dim=1).to(A.dtype)
        M = fk.fk_golden_steps(T, c["budget"], c["interval"])
        s.update(A=A, hkv=c["hkv"], T=T, budget=c["budget"], interval=c["interval"],
                 block=torch.empty((c["hkv"], M, T), dtype=torch.float32, device="cuda"),
                 alpha=torch.empty((c["hkv"], M, T), dtype=torch.float32, device="cuda"),
                 kept=torch.empty((c["hkv"], M, c["budget"]), dtype=torch.int32, device="cuda"))
        return s
    scale = 1.0 / math.sqrt(c["d"])
    if kind == "stack":
        n, L = c["n"], c["layers"]
        desc = _desc(c, c["batch"], _capacity(n + 1), cold=True)
        ws = fk.new_attn_workspace(desc)
        len0 = _lens(c, [n] * c["batch"]).expand(L, c["batch"], c["hkv"]).contiguous()
        ln, pn = len0.clone(), torch.full((c["batch"],), n, dtype=torch.int32, device="cuda")
        q, k, v = _tokens(c, gen, L, c["batch"])
        out = torch.empty_like(q)
        caches = [_cache(c, gen, c["batch"], desc.capacity) for _ in range(L)]
        calls = [fk.prepare(fk.fk_decode_step, desc, q[l], *caches[l], ln[l], k[l], v[l], pn, n + 1, scale, out[l], ws) for l in range(L)]
        s.update(len0=len0, len=ln, calls=calls, outputs=dict(out=out, len=ln, K=[x[0] for x in caches], V=[x[1] for x in caches]),
                 keep_alive=(q, k, v, pn, ws, caches))
        return s
    if kind == "ragged":
        lens = (c["lo"] + torch.randint(0, c["hi"] - c["lo"] + 1, (c["batch"],), generator=gen, device="cuda")).tolist()
        s["lens"] = [int(x) for x in lens]
        ml = max(s["lens"]) + 1
        n = _capacity(c["hi"] + 1)
    else:
        s["lens"] = [c["budget"] if kind == "cycle" else c["n"]] * c["batch"]
        n = _capacity(s["lens"][0] + (c["interval"] if kind == "cycle" else c.get("steps", 0)))
        ml = s["lens"][0] + 1
    desc = _desc(c, c["batch"], n)
    K, V, pos = _cache(c, gen, c["batch"], n)
    len0 = _lens(c, s["lens"])
    s.update(desc=desc, K=K, V=V, pos=pos, len0=len0, len=len0.clone(), max_len=ml, scale=scale)
    if kind in ("cycle", "step", "window", "ragged", "feat"):
        T = c["interval"] if kind == "cycle" else c.get("steps", 1)
        s["q"], s["k"], s["v"] = _tokens(c, gen, T, c["batch"])
        s["pos_new"] = (torch.tensor(s["lens"], dtype=torch.int32, device="cuda")[None, :] + torch.arange(T, dtype=torch.int32, device="cuda")[:, None]).contiguous()
        s["out"], s["T"] = torch.empty_like(s["q"]), T
        s["ws"] = fk.new_feat_workspace(desc) if kind == "feat" else fk.new_attn_workspace(desc)
    if kind in ("cycle", "score", "feat"):
        s["scorer"] = _scorer(c, gen, PLANES * c["g"] if kind == "feat" else 0)
        s["scores"] = torch.zeros((c["batch"], c["hkv"], n), dtype=torch.float32, device="cuda")
    if kind in ("feat", "sampled"):   # carried sums of the earlier chunks; the planes of this chunk are empty (feat) or full (sampled)
        s["feat"] = fk.new_feat(desc)
        first = 4 if kind == "feat" else 0
        u = torch.rand((c["batch"], c["hkv"], PLANES - first, n, s["feat"].shape[-1]), generator=gen, device="cuda") * 0.05
        u[..., c["g"]:] = 0
        s["feat"][:, :, first:] = u
    if kind in ("cycle", "step", "window", "ragged", "feat"):
        state = (K, V, pos, s["len"])
        if c.get("known", kind == "window"):
            more = (s["T"], ml, scale, s["feat"], 0, s["T"], s["out"], s["ws"]) if kind == "feat" else (s["T"], ml, scale, s["out"], s["ws"])
            s["calls"] = [fk.prepare(fk.fk_decode_window_feat if kind == "feat" else fk.fk_decode_window, desc, s["q"], *state, s["k"], s["v"],
                                     s["pos_new"], *more)]
        else:
            s["calls"] = []
            for t in range(s["T"]):
                more = (ml + t, scale, s["feat"], t, s["T"], s["out"][t], s["ws"]) if kind == "feat" else (ml + t, scale, s["out"][t], s["ws"])
                s["calls"].append(fk.prepare(fk.fk_decode_step_feat if kind == "feat" else fk.fk_decode_step, desc, s["q"][t], *state, s["k"][t],
                                             s["v"][t], s["pos_new"][t], *more))
        s["outputs"] = dict(out=s["out"], K=K, V=V, pos=pos, len=s["len"])
    if kind in ("event", "oneshot", "sampled"):
        shape = (c["batch"], c["hkv"], n)
        s["scores"] = _scores(c, gen, shape, c["ties"])
        if kind == "sampled":
            s["noise"] = -torch.log(-torch.log(torch.rand(shape, generator=gen, device="cuda").clamp_(1e-7, 1 - 1e-7)))
        if kind == "oneshot":
            need = fk.fk_select_keep_workspace(desc, c["n"], c["budget"], c["recent"])
            s["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
    if kind in ("cycle", "event", "oneshot", "sampled"):
        s["budget"], s["recent"] = c["budget"], c["interval"] if kind == "cycle" else c["recent"]
        s["keep"] = torch.zeros((c["batch"], c["hkv"], c["budget"]), dtype=torch.int32, device="cuda")
    return s


# ---- one pass -----------------------------------------------------------------------------------------------------

def run(s):
    kind = s["kind"]
    if kind == "golden":
        fk.fk_golden_scores(s["A"], s["hkv"], s["T"], s["budget"], s["interval"], s["block"], s["alpha"])
        fk.fk_golden_trace(s["alpha"], s["T"], s["budget"], s["interval"], s["kept"])
        return dict(block=s["block"], alpha=s["alpha"], kept=s["kept"])
    if kind != "cycle" and kind != "score":   # every pass starts from the same cache lengths
        s["len"].copy_(s["len0"])
    if kind == "feat":
        s["feat"][:, :, :4] = 0   # a chunk starts with empty planes
    for call in s.get("calls", ()):
        call()
    if kind in ("step", "window", "ragged", "stack"):
        return s["outputs"]
    desc, K, V, pos, ln = s["desc"], s["K"], s["V"], s["pos"], s["len"]
    if kind == "score":
        fk.fk_score_kv(desc, K, V, ln, s["max_len"] - 1, *s["scorer"], s["scores"])
        return dict(scores=s["scores"])
    if kind == "feat":
        fk.fk_score_kv_feat(desc, K, V, s["feat"], ln, s["max_len"] + s["T"] - 1, *s["scorer"], s["scores"])
        return dict(s["outputs"], feat=s["feat"], scores=s["scores"])
    if kind == "cycle":
        n = s["max_len"] + s["T"] - 1
        fk.fk_score_kv(desc, K, V, ln, n, *s["scorer"], s["scores"], skip_len=s["budget"])
        fk.fk_select_keep(desc, s["scores"], pos, ln, n, s["budget"], s["recent"], s["keep"])
        fk.fk_compact(desc, K, V, pos, ln, s["keep"], s["budget"])
        s["pos_new"].add_(s["T"])   # the next chunk's positions
        return dict(s["outputs"], scores=s["scores"], keep=s["keep"])
    n = s["max_len"] - 1
    if kind == "event":
        fk.fk_select_keep(desc, s["scores"], pos, ln, n, s["budget"], s["recent"], s["keep"])
        fk.fk_compact(desc, K, V, pos, ln, s["keep"], s["budget"])
        return dict(keep=s["keep"], K=K, V=V, pos=pos, len=ln)
    if kind == "oneshot":
        fk.fk_select_keep_ws(desc, s["scores"], pos, ln, n, s["budget"], s["recent"], s["keep"], s["ws"])
        fk.fk_compact(desc, K, V, pos, ln, s["keep"], s["budget"])
        return dict(keep=s["keep"], K=K, V=V, pos=pos, len=ln)
    fk.fk_select_keep_sampled(desc, s["scores"], s["noise"], pos, ln, n, s["budget"], s["recent"], 2 * (n - s["budget"]), s["keep"])
    fk.fk_compact_feat(desc, K, V, pos, s["feat"], ln, s["keep"], s["budget"])
    return dict(keep=s["keep"], feat=s["feat"], K=K, V=V, pos=pos, len=ln)


# ---- the least a pass has to do -------------------------------------------------------------------------------------

def work(c):
    e, kind = (4 if c["dtype"] == "f32" else 2), c["kind"]
    if kind == "golden":
        T, B, L = c["tokens"], c["budget"], c["interval"]
        M = max(0, -(-(T - B) // L) - 1)
        entries = c["heads"] * sum(q + 1 for q in range(B + L, T))
        return dict(bytes=entries * e + c["hkv"] * M * (2 * T + B) * 4, flops=entries)
    rows, d, g = c["batch"] * c["hkv"], c["d"], c["g"]
    pair = 2 * d * e                                    # K and V of one pair
    token = rows * (pair + 2 * g * d * e)               # new pair, queries and output of one step
    attn = lambda n: 4.0 * rows * g * d * n             # noqa: E731  flops of one step over n pairs
    mlp = lambda n, f, h: rows * n * (2.0 * f * h + 4 * h)  # noqa: E731
    if kind == "ragged":
        n = (c["lo"] + c["hi"]) / 2 + 1
        return dict(bytes=rows * n * pair + token, flops=attn(n))
    if kind == "step":
        return dict(bytes=sum(rows * (c["n"] + t + 1) * pair + token for t in range(c["steps"])), flops=sum(attn(c["n"] + t + 1) for t in range(c["steps"])))
    if kind == "stack":
        return dict(bytes=c["layers"] * (rows * (c["n"] + 1) * pair + token), flops=c["layers"] * attn(c["n"] + 1))
    if kind == "score":
        return dict(bytes=rows * c["n"] * (pair + 4) + c["hkv"] * 2 * d * c["hidden"] * e, flops=mlp(c["n"], 2 * d, c["hidden"]))
    n = c["budget"] + c["interval"] if kind == "cycle" else c["n"]
    move = rows * c.get("budget", 0) * (2 * (pair + 4) + 4) + rows * n * 4     # kept pairs read and written, keep list, scores
    if kind in ("event", "oneshot"):
        return dict(bytes=move, flops=rows * n)
    if kind == "sampled":
        gp = 4 if g <= 4 else 8
        return dict(bytes=move + rows * n * 4 + rows * gp * 4 * (3 * n + 2 * c["budget"] + 4 * n), flops=rows * n)
    if kind == "window":
        T = c["steps"]
        return dict(bytes=rows * n * pair + 2 * T * token, flops=sum(attn(n + t + 1) for t in range(T)))
    T = c["interval"] if kind == "cycle" else c["steps"]
    # known tokens need the cache once; generated ones once per step
    cached = rows * pair * (n if c["known"] else sum((c["budget"] if kind == "cycle" else n) + t for t in range(T)))
    if kind == "feat":
        gp = 4 if g <= 4 else 8
        planes = 10 if c["known"] else 2 * T + 10
        return dict(bytes=cached + 2 * T * token + rows * (n + T) * (gp * 4 * planes + 4),
                    flops=sum(attn(n + t + 1) for t in range(T)) + mlp(n + T, 2 * d + PLANES * g, c["hidden"]))
    return dict(bytes=cached + 2 * T * token + move, flops=sum(attn(c["budget"] + t + 1) for t in range(T)) + mlp(n, 2 * d, c["hidden"]))


def tolerance(c):
    kind = c["kind"]
    if kind in ("event", "oneshot"):
        return "exact"                     # copies and whole numbers
    if kind == "sampled":
        return dict(rel=1e-6, max=1e-5)    # feature sums: one fp32 addition or fma
    if kind == "score":
        return dict(rel=4e-6, max=4e-5)    # fp32 sums of 256 terms and a gelu good to 6e-7
    if kind == "golden":
        return dict(rel=2e-6, max=2e-5, differ=0.01)   # fp32 means; pairs at the cut to within rounding
    if kind == "cycle" and c["dtype"] == "f32":
        return dict(rel=1e-5, max=1e-4)
    return dict(rel=1e-2, max=6e-2)        # bf16 outputs, bf16 softmax weights


# ---- the same in 64 bits ------------------------------------------------------------------------------------------

def _attention(q, K, V, k, v, lens, scale, weights=False):
    """q [T][B][Hq][d], K, V [B][H][cap][d] before the steps, k, v [T][B][H][d] -> out [T][B][Hq][d]; with weights also the
    attention weights of one (sequence, head) after another through a generator."""
    T, Bt, Hq, d = q.shape
    H = K.shape[1]
    g = Hq // H
    out = torch.empty((T, Bt, Hq, d), dtype=torch.float64, device=q.device)
    kept = []
    for b in range(Bt):
        n = lens[b]
        live = torch.arange(n + T, device=q.device)[None, :] <= n + torch.arange(T, device=q.device)[:, None]
        for h in range(H):
            kk = torch.cat([K[b, h, :n], k[:, b, h]]).double()
            vv = torch.cat([V[b, h, :n], v[:, b, h]]).double()
            z = (q[:, b, h * g:(h + 1) * g].double().reshape(T * g, d) @ kk.T).reshape(T, g, n + T) * scale
            p = torch.softmax(z.masked_fill_(~live[:, None, :], float("-inf")), dim=2)
            out[:, b, h * g:(h + 1) * g] = (p.reshape(T * g, n + T) @ vv).reshape(T, g, d)
            if weights:
                kept.append(_chunk_sums(p))
    return (out, kept) if weights else out


def _chunk_sums(p):
    """Attention weights p [T][g][n] of a chunk -> sums over its last 8, 16, 32 and all queries, [4][n][g]."""
    T = p.shape[0]
    return torch.stack([p[max(0, T - w):].sum(0).T for w in (8, 16, 32, T)])


def _mlp(x, scorer, heads):
    """x [B][H][n][F] one (sequence, head) at a time from a callable -> scores [B][H][n]"""
    w1, b1, w2, b2 = (t.double() for t in scorer)
    return [torch.nn.functional.gelu(x(i) @ w1[i % heads] + b1[i % heads]) @ w2[i % heads] + b2[i % heads] for i in range(len(x))]


class _Rows:
    """The scorer's inputs, one row after the other."""

    def __init__(self, K, V, n, extra=None):
        self.K, self.V, self.n, self.extra = K.flatten(0, 1), V.flatten(0, 1), n, extra

    def __len__(self):
        return self.K.shape[0]

    def __call__(self, i):
        x = [self.K[i, :self.n].double(), self.V[i, :self.n].double()]
        return torch.cat(x + ([self.extra[i]] if self.extra is not None else []), dim=1)


def _rolled(s, c):
    """The feature state after the sampled selection and the compaction that closes the chunk."""
    n, budget, cut = c["n"], c["budget"], c["n"] - c["recent"]
    evict = n - budget
    feat = s["feat"].double()
    for b in range(c["batch"]):
        for h in range(c["hkv"]):
            sc, nz = s["scores"][b, h, :cut], s["noise"][b, h, :cut]
            low = sc.sort(descending=True, stable=True).indices[cut - min(max(2 * evict, evict), cut):].sort().values   # the candidates
            gone = low[(sc[low] - nz[low]).sort(descending=True, stable=True).indices[low.numel() - evict:]]
            stay = torch.ones(n, dtype=torch.bool, device="cuda")
            stay[gone] = False
            keep = stay.nonzero()[:, 0]
            f = feat[b, h]
            wl, cum, dec = f[3, keep], f[4, keep], f[5, keep]
            f[:4, :n] = 0
            f[4, :budget], f[5, :budget] = cum + wl, DECAY * dec + wl
    return feat


def _extended(X, x, n):
    """The cache X with the new rows x [T][B][H][d] from slot n on."""
    Y = X.clone()
    Y[:, :, n:n + x.shape[0]] = x.permute(1, 2, 0, 3)
    return Y


def exact(c, seed):
    kind = c["kind"]
    if kind in ("event", "oneshot"):
        return None
    s = prepare(c, seed)
    if kind == "golden":
        T, B, L, g = c["tokens"], c["budget"], c["interval"], c["heads"] // c["hkv"]
        M = s["block"].shape[1]
        block = torch.zeros((c["hkv"], M, T), dtype=torch.float64, device="cuda")
        for h in range(c["heads"]):
            for t in range(M):
                block[h // g, t] += s["A"][h, B + (t + 1) * L:min(B + (t + 2) * L, T), :T].double().sum(0)
        block /= g * L
        return dict(block=block, alpha=block.flip(1).cummax(1).values.flip(1), kept=None)
    if kind == "stack":
        q, k, v, _, _, caches = s["keep_alive"]
        out = torch.cat([_attention(q[l:l + 1], caches[l][0], caches[l][1], k[l:l + 1], v[l:l + 1], [c["n"]] * c["batch"], 1 / math.sqrt(c["d"]))
                         for l in range(c["layers"])])
        return dict(out=out, len=None, K=None, V=None)
    if kind == "sampled":
        return dict(keep=None, feat=_rolled(s, c), K=None, V=None, pos=None, len=None)
    if kind == "score":
        out = torch.zeros(s["scores"].shape, dtype=torch.float64, device="cuda")
        out[:, :, :c["n"]] = torch.stack(_mlp(_Rows(s["K"], s["V"], c["n"]), s["scorer"], c["hkv"])).reshape(c["batch"], c["hkv"], c["n"])
        return dict(scores=out)
    want = kind == "feat"
    got = _attention(s["q"], s["K"], s["V"], s["k"], s["v"], s["lens"], s["scale"], want)
    if kind in ("step", "ragged", "window"):
        return dict(out=got, K=None, V=None, pos=None, len=None)
    n, T = s["lens"][0], s["T"]
    K, V = _extended(s["K"], s["k"], n), _extended(s["V"], s["v"], n)
    scores = torch.zeros(s["scores"].shape, dtype=torch.float64, device="cuda")
    if kind == "cycle":
        scores[:, :, :n + T] = torch.stack(_mlp(_Rows(K, V, n + T), s["scorer"], c["hkv"])).reshape(c["batch"], c["hkv"], n + T)
        return dict(out=got, scores=scores, keep=None, K=None, V=None, pos=None, len=None)
    out, sums = got
    feat, extra, g = s["feat"].double(), [], c["g"]
    feat[:, :, 4:, n:n + T] = 0    # a new pair starts from zero
    for i, w in enumerate(sums):
        f = feat[i // c["hkv"], i % c["hkv"]]
        f[:4] = 0
        f[:4, :n + T, :g] = w
        a = f[:, :n + T, :g].clone()
        a[4] += a[3]
        a[5] = DECAY * a[5] + a[3]
        extra.append(a.permute(1, 2, 0).reshape(n + T, g * PLANES))
    scores[:, :, :n + T] = torch.stack(_mlp(_Rows(K, V, n + T, extra), s["scorer"], c["hkv"])).reshape(c["batch"], c["hkv"], n + T)
    return dict(out=out, feat=feat, scores=scores, K=None, V=None, pos=None, len=None)
