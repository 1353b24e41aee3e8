"""Measured cases of the rollout engine, through its public entry points.

A rollout worker does three things with the engine: it prefills prompts (at the
start of a round, or again when a preempted sequence resumes with a long
history), it decodes one token for every live row, step after step, while the
batch shrinks from hundreds of rows to the one longest response, and it scores
given responses (prefill, then teacher-forced decode).  The cases cover the
Qwen2.5 shapes of the repository's workloads (0.5B, 7B, 32B and the small fp32
decoder), from one row to several hundred and from tens of tokens of context to
more than ten thousand.

The 0.5B model runs whole.  The 7B and 32B models run a seventh or a
thirty-second of themselves: 4 of 28 layers (2 of 64) with the vocabulary cut
in the same proportion, so that the layers, the LM head and the sampling keep
the shares they have in the whole model, every product keeps its K and the
layers keep all of their shapes.

Kinds of case:
  decode   the rows stand prefilled; a pass is one teacher-forced decode step of
           all rows (the sampled step with its logits returned).  The rows of one
           prompt are its responses.  Every pass appends a token, as in a rollout;
           rows that reach their length are replaced by fresh ones.
  prefill  a pass admits the prompts, which prefills them and samples their first
           token, returns the last logits of each, and drops the sequences again.
  score    a pass admits the prompts, forces `steps - 1` response tokens through
           decode steps, returns the logits of every position, and drops them.
"""
from __future__ import annotations

import random
import types

import numpy as np
import torch

from paper_2509_21009_amd import rollpack

# layers, hidden, q heads, KV heads, head dim, intermediate, vocabulary, tied embeddings, type
_MODELS = {
    "tiny": (2, 256, 4, 2, 64, 688, 2048, False, "f32"),
    "0.5b": (24, 896, 14, 2, 64, 4864, 151936, True, "bf16"),
    "7b": (4, 3584, 28, 4, 128, 18944, 21760, False, "bf16"),      # 4 of 28 layers, 1/7 of the vocabulary
    "32b": (2, 5120, 40, 8, 128, 27648, 4864, False, "bf16"),      # 2 of 64 layers, 1/32 of the vocabulary
}
_EPS, _THETA = 1e-6, 1e6
_PAGE = 64
_CHUNK = 16384      # prefill chunk, the benchmark's (the engine's limit, whatever a case admits)
_ROOM = 4096        # decode steps a row has ahead of it


def _shape(model):
    n, h, q, kv, hd, i, v, tied, dt = _MODELS[model]
    return types.SimpleNamespace(layers=n, hidden=h, n_q=q, n_kv=kv, head_dim=hd, inter=i, vocab=v, tied=tied,
                                 dtype=dt, eps=_EPS, theta=_THETA)


def listed():
    return [
        # The fp32 decoder of the parity tests: a whole small round, greedy; launch latency counts.
        dict(name="tiny-f32-score", kind="score", model="tiny", prompts=8, responses=1, lo=32, hi=32, steps=9),
        # The smallest serving call: a handful of rows of the 0.5B model.
        dict(name="0.5b-decode-4", kind="decode", model="0.5b", prompts=4, responses=1, lo=65, hi=500, steps=1),
        # The 0.5B round at its full batch, 32 prompts x 8 responses.
        dict(name="0.5b-decode-256", kind="decode", model="0.5b", prompts=32, responses=8, lo=130, hi=1300, steps=1),
        # Admission of 0.5B prompts, four responses each.
        dict(name="0.5b-prefill-32", kind="prefill", model="0.5b", prompts=8, responses=4, lo=64, hi=512, steps=1),
        # The end of a long round: the longest response decodes alone.
        dict(name="7b-decode-1", kind="decode", model="7b", prompts=1, responses=1, lo=12001, hi=12001, steps=1),
        # Most of a long round's steps: a dozen rows at long contexts.
        dict(name="7b-decode-12", kind="decode", model="7b", prompts=12, responses=1, lo=1500, hi=7000, steps=1),
        # The full long round: 64 rows, ragged contexts.
        dict(name="7b-decode-64", kind="decode", model="7b", prompts=16, responses=4, lo=600, hi=4500, steps=1),
        # A short round at its full width.
        dict(name="7b-decode-330", kind="decode", model="7b", prompts=66, responses=5, lo=200, hi=1700, steps=1),
        # One prompt arrives: time to first token.
        dict(name="7b-prefill-1", kind="prefill", model="7b", prompts=1, responses=1, lo=397, hi=397, steps=1),
        # Admission of a round's prompts, U[128, 1024].
        dict(name="7b-prefill-20", kind="prefill", model="7b", prompts=20, responses=1, lo=128, hi=1024, steps=1),
        # A preempted long response resumes: its whole history is prefilled again.
        dict(name="7b-prefill-long", kind="prefill", model="7b", prompts=1, responses=1, lo=14500, hi=14500, steps=1),
        # A 32B round with half of its rows left.
        dict(name="32b-decode-45", kind="decode", model="32b", prompts=15, responses=3, lo=300, hi=3000, steps=1),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "prefill", "prefill", "score"])
    if kind == "decode":
        model = rng.choice(["0.5b", "7b", "7b", "32b"])
        rows = _log(rng, 1, {"0.5b": 256, "7b": 330, "32b": 96}[model])
        responses = rng.choice([1, 1, 2, 3, 4, 8])
        prompts = max(1, rows // responses)
        # as many tokens in all as a listed case of the model at most
        most = min(12000, {"0.5b": 160000, "7b": 300000, "32b": 70000}[model] // (prompts * responses))
        hi = _log(rng, 60, max(61, most))
        return dict(kind=kind, model=model, prompts=prompts, responses=responses, lo=max(1, hi // rng.choice([1, 2, 8])),
                    hi=hi, steps=1)
    if kind == "prefill":
        model = rng.choice(["0.5b", "7b"])
        prompts = _log(rng, 1, 24)
        hi = _log(rng, 20, min(14000, {"0.5b": 9000, "7b": 14000}[model] // prompts))
        return dict(kind=kind, model=model, prompts=prompts, responses=1, lo=max(1, hi // rng.choice([1, 2, 8])), hi=hi,
                    steps=1)
    model = rng.choice(["tiny", "0.5b"])
    prompts = rng.randint(1, 12)
    hi = rng.randint(4, 100)
    return dict(kind=kind, model=model, prompts=prompts, responses=1, lo=max(1, hi // 2), hi=hi, steps=rng.randint(2, 12))


def _lengths(case):
    """Prompt lengths, spread evenly over [lo, hi] in an order of the case's own (the same for every seed)."""
    n, lo, hi = case["prompts"], case["lo"], case["hi"]
    out = [hi if n == 1 else lo + (hi - lo) * i // (n - 1) for i in range(n)]
    random.Random(n * 1000003 + hi).shuffle(out)
    return out


def _randn(dims, dtype, gen):
    return torch.randn(dims, generator=gen, device="cuda", dtype=torch.float32).mul_(0.02).to(dtype)


def _inputs(case, seed):
    """Weights on the GPU (N(0, 0.02); norm gains around one), prompts and forced tokens on the host."""
    s = _shape(case["model"])
    dt = torch.float32 if s.dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 7919 + 1)
    h, i, qd, kd = s.hidden, s.inter, s.n_q * s.head_dim, s.n_kv * s.head_dim

    def gain():
        return (1 + torch.randn(h, generator=gen, device="cuda") * 0.1).to(dt)

    w = {"embed": _randn((s.vocab, h), dt, gen), "final_norm": gain(), "layers": []}
    for _ in range(s.layers):
        w["layers"].append({
            "attn_norm": gain(), "mlp_norm": gain(),
            "wq": _randn((qd, h), dt, gen), "bq": _randn((qd,), dt, gen),
            "wk": _randn((kd, h), dt, gen), "bk": _randn((kd,), dt, gen),
            "wv": _randn((kd, h), dt, gen), "bv": _randn((kd,), dt, gen),
            "wo": _randn((h, qd), dt, gen), "w_gate": _randn((i, h), dt, gen), "w_up": _randn((i, h), dt, gen),
            "w_down": _randn((h, i), dt, gen)})
    w["lm_head"] = None if s.tied else _randn((s.vocab, h), dt, gen)
    rng = np.random.default_rng([int(seed), 17])
    prompts = [rng.integers(0, s.vocab, size=n).astype(np.int32) for n in _lengths(case)]
    rows = case["prompts"] * case["responses"]
    forced = rng.integers(0, s.vocab, size=(max(1, case["steps"] - 1), rows)).astype(np.int32)
    return s, w, prompts, forced


def prepare(case, seed):
    """The engine with its weights, the prompts, and for a decode case the rows prefilled."""
    s, w, prompts, forced = _inputs(case, seed)
    r = case["responses"]
    rows = case["prompts"] * r
    per_row = [p for p in prompts for _ in range(r)]
    room = _ROOM if case["kind"] == "decode" else case["steps"]
    lens = [len(p) for p in per_row]
    st = types.SimpleNamespace()
    st.case, st.forced = case, forced
    st.ids = np.arange(1000, 1000 + rows, dtype=np.int64)
    st.tokens = np.concatenate(per_row)
    st.offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    st.max_new = np.full(rows, room, np.int32)
    st.sample_seed = int(seed) & 0xFFFF
    st.temperature = 0.0 if s.dtype == "f32" else 1.0
    pages = sum(-(-(n + room - 1) // _PAGE) for n in lens)
    st.engine = rollpack.Engine(s, w, max_seqs=rows, max_prefill_tokens=_CHUNK, max_context=max(lens) + room,
                                kv_pages=pages)
    st.left = 0
    if case["kind"] == "decode":
        _admit(st)
    return st


def _admit(st, logits=False):
    out, _ = st.engine.prefill(st.ids, st.tokens, st.offsets, st.max_new, st.sample_seed, st.temperature, logits=logits)
    st.left = int(st.max_new[0]) - 1
    return out


def run(st):
    if st.case["kind"] == "decode":
        if st.left == 0:  # every row has reached its length: the next batch takes its place
            st.engine.free_finished()
            _admit(st)
        st.left -= 1
        return st.engine.decode_step(st.forced[0], logits=True)[2]
    out = [_admit(st, logits=True)]
    for j in range(st.case["steps"] - 1):
        out.append(st.engine.decode_step(st.forced[j], logits=True)[2])
    st.engine.abort(st.ids)
    return out


def work(case):
    """Weights and K/V read once, logits written once, and the products of every token."""
    s = _shape(case["model"])
    e = 4 if s.dtype == "f32" else 2
    h, i, qd, kd = s.hidden, s.inter, s.n_q * s.head_dim, s.n_kv * s.head_dim
    layer = h * (qd + 2 * kd) + qd * h + 3 * h * i
    r = case["responses"]
    lens = [n for n in _lengths(case) for _ in range(r)]
    rows = len(lens)
    kv_token = s.layers * 2 * kd * e
    weights = (s.layers * layer + s.vocab * h) * e

    def step(ctx):  # one decode step at these contexts (the row's own token among them)
        b = weights + sum(ctx) * kv_token + rows * (s.vocab * 4 + h * e)
        f = 2 * rows * (s.layers * layer + s.vocab * h) + s.layers * 4 * qd * sum(ctx)
        return b, f

    if case["kind"] == "decode":
        b, f = step([n + 1 for n in lens])
        return {"bytes": b, "flops": f}
    tokens = sum(lens)
    b = weights + tokens * (kv_token + h * e) + rows * s.vocab * 4
    f = (2 * tokens * s.layers * layer + 2 * rows * s.vocab * h
         + s.layers * 4 * qd * sum(n * (n + 1) // 2 for n in lens))
    for j in range(1, case["steps"]):
        db, df = step([n + j for n in lens])
        b, f = b + db, f + df
    return {"bytes": b, "flops": f}


def tolerance(case):
    """bf16: the same path with its sums in another order (prefill in chunks of 700 tokens, so that other tiles and K
    splits run) differs by up to 0.007 and 0.054 (max); both are 0.007-0.015 from the 64-bit result.  f32: sums of up to
    688 products, 7e-7 from it."""
    if _MODELS[case["model"]][8] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 0.02, "max": 0.2}


# ---- the same in 64 bits -------------------------------------------------------------

def _norm(x, g):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + _EPS) * g.double()


def _rope(u, pos, hd):
    d = torch.arange(hd // 2, device="cuda", dtype=torch.float64)
    ang = pos.double()[:, None] * _THETA ** (-2.0 * d / hd)
    c, sn = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
    u1, u2 = u[..., :hd // 2], u[..., hd // 2:]
    return torch.cat([u1 * c - u2 * sn, u2 * c + u1 * sn], -1)


def _qkv(s, L, x, pos):
    hn = _norm(x, L["attn_norm"])
    q = (hn @ L["wq"].double().t() + L["bq"].double()).view(-1, s.n_q, s.head_dim)
    k = (hn @ L["wk"].double().t() + L["bk"].double()).view(-1, s.n_kv, s.head_dim)
    v = (hn @ L["wv"].double().t() + L["bv"].double()).view(-1, s.n_kv, s.head_dim)
    return _rope(q, pos, s.head_dim), _rope(k, pos, s.head_dim), v


def _causal(s, q, k, v):
    """Attention of a whole prompt, 512 queries at a time: q [n, n_q, hd], k and v [n, n_kv, hd]."""
    n, g = q.shape[0], s.n_q // s.n_kv
    out = torch.empty_like(q)
    at = torch.arange(n, device="cuda")
    for o in range(0, n, 512):
        m = min(o + 512, n)
        mask = at[None, :m] > at[o:m, None]
        for kh in range(s.n_kv):
            for hh in range(kh * g, kh * g + g):
                sc = q[o:m, hh] @ k[:m, kh].t().contiguous() / s.head_dim ** 0.5
                out[o:m, hh] = torch.softmax(sc.masked_fill(mask, -float("inf")), -1) @ v[:m, kh]
    return out


def _mlp(L, x):
    hn = _norm(x, L["mlp_norm"])
    g = hn @ L["w_gate"].double().t()
    return (g * torch.sigmoid(g) * (hn @ L["w_up"].double().t())) @ L["w_down"].double().t()


def exact(case, seed):
    s, w, prompts, forced = _inputs(case, seed)
    flops = work(dict(case, kind="prefill", responses=1))["flops"]
    if flops > 3.0e14:  # over 20 s in 64 bits
        return None
    r = case["responses"]
    lens = [len(p) for p in prompts]
    pos = torch.cat([torch.arange(n, device="cuda") for n in lens])
    x = w["embed"][torch.from_numpy(np.concatenate(prompts)).cuda().long()].double()
    offs = np.concatenate([[0], np.cumsum(lens)])
    caches = []  # per layer, per row: K and V
    for L in w["layers"]:
        a = torch.empty((x.shape[0], s.n_q * s.head_dim), device="cuda", dtype=torch.float64)
        cache = []
        for j in range(len(lens)):
            sl = slice(int(offs[j]), int(offs[j + 1]))
            q, k, v = _qkv(s, L, x[sl], pos[sl])
            a[sl] = _causal(s, q, k, v).reshape(a[sl].shape)
            cache += [(k, v)] * r
        x = x + a @ L["wo"].double().t()
        for o in range(0, x.shape[0], 8192):
            x[o:o + 8192] += _mlp(L, x[o:o + 8192])
        caches.append(cache)
    lm = (w["embed"] if s.tied else w["lm_head"])

    def head(y):
        hn = _norm(y, w["final_norm"])
        return torch.cat([hn @ lm[o:o + 16384].double().t() for o in range(0, s.vocab, 16384)], -1)

    last = torch.from_numpy(offs[1:] - 1).cuda().repeat_interleave(r)
    out = [] if case["kind"] == "decode" else [head(x[last])]
    steps = 1 if case["kind"] == "decode" else case["steps"] - 1
    at = torch.tensor([n for n in lens for _ in range(r)], device="cuda")
    grp = s.n_q // s.n_kv
    for j in range(steps):
        y = w["embed"][torch.from_numpy(forced[j]).cuda().long()].double()
        for li, L in enumerate(w["layers"]):
            q, k, v = _qkv(s, L, y, at + j)
            a = torch.empty_like(q)
            for b in range(y.shape[0]):
                ck, cv = caches[li][b]
                ck, cv = torch.cat([ck, k[b:b + 1]]), torch.cat([cv, v[b:b + 1]])
                caches[li][b] = (ck, cv) if steps > 1 else None
                for kh in range(s.n_kv):
                    qs = slice(kh * grp, kh * grp + grp)
                    p = torch.softmax(q[b, qs] @ ck[:, kh].t().contiguous() / s.head_dim ** 0.5, -1)
                    a[b, qs] = p @ cv[:, kh]
            y = y + a.reshape(y.shape[0], -1) @ L["wo"].double().t()
            y = y + _mlp(L, y)
        out.append(head(y))
    return out[0] if case["kind"] == "decode" else out
