"""Workloads by which this library is timed: what each call is in use, its inputs, its bytes and flops, its error.

A case is a dict of plain values.  `listed()` holds the ones that are always looked at, `draw()` makes others of the
same ranges, `prepare()` builds what a serving program has in hand before the call (models, contexts with prefilled
caches, candidates, uniforms), `run()` is one pass through the public entry points and `exact()` the same numbers in
64-bit torch.  Models have random weights of the repository's shapes; most target cases carry one or two layers of
the real widths (a block of the model behind the real entry point), one is the whole 32-layer target.

A pass that commits tokens makes its sequences grow, as in service: small-batch cases keep several conversations open
and advance them in turn, every few passes the lengths are read back (`Context.sync`, as a server does to deliver
tokens), and conversations that could outgrow their capacity start over from their prompt.
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

from paper_2505_08600_amd import api
from paper_2505_08600_amd import datagen as dg

# Next-token distributions as trained models have them on predictable text at T = 1: after a token one successor takes
# nearly all the mass, and what is left is peaked too.  The draft and the target of one seed know the same successors.
TAIL_STD, SUCCESSOR = 5.0, 50.0


def listed():
    return [
        # one conversation's acceptance decision on logits the caller holds: the smallest call, two dependent launches
        {"name": "accept_b1", "kind": "accept", "n": 1, "gamma": 5, "vocab": 32000, "temp": 1.0},
        # the same rule for a full batch over a large vocabulary (300 MB of logits)
        {"name": "accept_b64_v128k", "kind": "accept", "n": 64, "gamma": 8, "vocab": 128000, "temp": 0.7},
        # routing the 400 prompts of a classifier test set to their drafts
        {"name": "classify_400", "kind": "classify", "n": 400, "max_len": 128},
        # a whole step of the tiny fp32 pair (the 32-bit data type): draft, verify, commit
        {"name": "step_tiny_fp32", "kind": "step", "b": 1, "open": 16, "lo": 32, "hi": 32, "gamma": 4, "temp": 1.0},
        # draft phase of one conversation with the 68M-shape draft: some seventy small launches in a row
        {"name": "draft_b1", "kind": "draft", "shape": "draft_a", "b": 1, "open": 8, "lo": 512, "hi": 512, "gamma": 5,
         "temp": 1.0, "adapters": 0},
        # one routed group of a batch on the deepest draft
        {"name": "draft_b9", "kind": "draft", "shape": "draft_c", "b": 9, "open": 9, "lo": 128, "hi": 1024, "gamma": 5,
         "temp": 0.7, "adapters": 0},
        # a batch whose routed drafts are low-rank adapters of one base model
        {"name": "draft_b32_lora", "kind": "draft", "shape": "draft_a", "b": 32, "open": 32, "lo": 128, "hi": 1024,
         "gamma": 3, "temp": 1.0, "adapters": 4},
        # the whole 7B-shape target verifying one conversation's candidates: the headline call
        {"name": "verify_7b_b1", "kind": "verify", "shape": "t7b", "layers": 32, "b": 1, "open": 4, "lo": 512, "hi": 512,
         "gamma": 5, "temp": 1.0},
        # a few conversations at once (24 rows)
        {"name": "verify_b4", "kind": "verify", "shape": "t7b", "layers": 2, "b": 4, "open": 4, "lo": 301, "hi": 1500,
         "gamma": 5, "temp": 1.0},
        # the ordinary serving batch: 32 prompts of 128 to 1024 tokens (192 rows)
        {"name": "verify_b32", "kind": "verify", "shape": "t7b", "layers": 2, "b": 32, "open": 32, "lo": 128, "hi": 1024,
         "gamma": 5, "temp": 0.7},
        # large batch with long, ragged contexts (576 rows, up to 8192 tokens each)
        {"name": "verify_b64_long", "kind": "verify", "shape": "t7b", "layers": 2, "b": 64, "open": 64, "lo": 1024,
         "hi": 8192, "gamma": 8, "temp": 1.0},
        # a new conversation with a long prompt: tokens in, prefill, first verify pass
        {"name": "prefill_8k", "kind": "prefill", "shape": "t7b", "layers": 2, "b": 1, "lo": 8192, "hi": 8192,
         "rows": 1024, "gamma": 5, "temp": 1.0},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["accept", "classify", "step", "draft", "draft", "verify", "verify", "verify", "prefill"])
    temp = rng.choice([0.0, 0.7, 1.0, 1.0])
    if kind == "accept":
        gamma, vocab = rng.randint(0, 12), 4 * _log(rng, 250, 65536)
        most = max(1, min(64, 64 * 9 * 128000 // ((gamma + 1) * vocab)))
        return {"kind": kind, "n": _log(rng, 1, most), "gamma": gamma, "vocab": vocab, "temp": temp}
    if kind == "classify":
        return {"kind": kind, "n": _log(rng, 1, 1600), "max_len": rng.randint(24, 200)}
    if kind == "step":
        b, lo = _log(rng, 1, 8), rng.randint(4, 100)
        return {"kind": kind, "b": b, "open": 16 // b * b, "lo": lo, "hi": lo + rng.randint(0, 100), "gamma": rng.randint(1, 6),
                "temp": temp}
    if kind == "draft":
        b, lo, lora = _log(rng, 1, 32), rng.randint(16, 512), rng.random() < 0.3
        return {"kind": kind, "shape": "draft_a" if lora else rng.choice(["draft_a", "draft_b", "draft_c", "draft_d"]),
                "b": b, "open": b * max(1, 8 // b), "lo": lo, "hi": lo + rng.randint(0, 700), "gamma": rng.randint(1, 6),
                "temp": rng.choice([0.7, 1.0]), "adapters": 4 if lora else 0}
    shape = rng.choice(["t7b", "t7b", "t13b"])
    if kind == "verify":
        b = _log(rng, 1, 64)
        lo = _log(rng, 16, 4000 if b <= 32 else 2000)
        return {"kind": kind, "shape": shape, "layers": 1 if shape == "t13b" else 2, "b": b, "open": b * max(1, 4 // b), "lo": lo,
                "hi": min(8000, lo + rng.randint(0, 2000)), "gamma": rng.randint(0, 8), "temp": temp}
    b, lo = rng.choice([1, 1, 2, 3]), _log(rng, 24, 2400)
    return {"kind": kind, "shape": shape, "layers": 1 if shape == "t13b" else 2, "b": b, "lo": lo,
            "hi": lo + rng.randint(0, 300), "rows": rng.choice([192, 576, 1024, 2048]), "gamma": rng.randint(0, 5),
            "temp": temp}


# ---------------------------------------------------------------- inputs

def _gen(seed, stream):
    return torch.Generator(device="cuda").manual_seed((int(seed) * 1000003 + stream) & 0x7FFFFFFF)


def _successor(seed, vocab):
    return torch.randperm(vocab, generator=torch.Generator().manual_seed(int(seed) * 104729 + 3))


def _weights(shape, seed, stream):
    """Random weights on the device: unit-variance activations (residual projections scaled by the depth), an LM head
    that points from each token's embedding to its successor, gains around 1."""
    g, d, f, v, L = _gen(seed, stream), shape.d_model, shape.d_ffn, shape.vocab, shape.n_layers
    dt = torch.bfloat16 if shape.dtype == dg.BF16 else torch.float32

    def mat(n, k, std):
        return torch.empty((n, k), dtype=dt, device="cuda").normal_(0.0, std, generator=g)

    def gain():
        return torch.empty(d, dtype=torch.float32, device="cuda").normal_(1.0, 0.02, generator=g)

    w = {"embed": mat(v, d, 1.0), "lm_head": mat(v, d, TAIL_STD / math.sqrt(d)), "final_norm": gain()}
    w["lm_head"][_successor(seed, v).cuda()] += (SUCCESSOR / d) * w["embed"]
    out = (2.0 * L) ** -0.5
    for name, n, k, scale in (("wq", d, d, 1.0), ("wk", d, d, 1.0), ("wv", d, d, 1.0), ("wo", d, d, out), ("wgate", f, d, 1.0),
                              ("wup", f, d, 1.0), ("wdown", d, f, out)):
        w[name] = [mat(n, k, scale / math.sqrt(k)) for _ in range(L)]
    for name in ("norm_attn", "norm_ffn"):
        w[name] = [gain() for _ in range(L)]
    return w


def _model(shape, w, max_rows, max_pos):
    """sd_load_model on weights that are on the device already (the C ABI takes device pointers; the binding's
    constructor uploads host arrays)."""
    torch.cuda.synchronize()
    m = api.Model.__new__(api.Model)
    m.shape, m.device, m.max_rows = shape, "cuda", max_rows
    cw, keep = api._Weights(), []
    cw.embed, cw.lm_head, cw.final_norm = (w[n].data_ptr() for n in ("embed", "lm_head", "final_norm"))
    for n in ("wq", "wk", "wv", "wo", "wgate", "wup", "wdown", "norm_attn", "norm_ffn"):
        arr = (ctypes.c_void_p * shape.n_layers)(*[t.data_ptr() for t in w[n]])
        keep.append(arr)
        setattr(cw, n, ctypes.cast(arr, ctypes.POINTER(ctypes.c_void_p)))
    cfg = api._Config(shape.n_layers, shape.d_model, shape.n_heads, shape.head_dim, shape.d_ffn, shape.vocab,
                      shape.dtype, shape.rope_base, shape.rms_eps, max_rows, max_pos)
    h = ctypes.c_void_p()
    rc = api.lib().sd_load_model(ctypes.byref(cfg), ctypes.byref(cw), ctypes.byref(h))
    if rc != api.SD_OK:
        raise api.SdError(rc, api.lib().sd_last_error().decode())
    m.h = h
    return m


def _shape(case):
    if case["kind"] == "step":
        return dg.SHAPES["tiny_target"]
    return dg.with_layers(dg.SHAPES[case["shape"]], case["layers"]) if "layers" in case else dg.SHAPES[case["shape"]]


def _prompts(case, seed, vocab):
    n = case.get("open", case["b"])
    g = torch.Generator().manual_seed(int(seed) * 7919 + 1)
    lens = torch.randint(case["lo"], case["hi"] + 1, (n,), generator=g).tolist()
    return [torch.randint(0, vocab, (l,), dtype=torch.int32, generator=g).numpy() for l in lens]


def _uniforms(seed, stream, *shape):
    return torch.randint(0, 1 << 24, shape, device="cuda", generator=_gen(seed, stream)).float() * 2.0 ** -24


def _candidates(seed, b, gamma, vocab, last):
    """Candidates of a good draft and the distribution they came with: the successor chain of each sequence's last token,
    every fourth link replaced by some other token, 0.9 of q's mass on the candidate."""
    succ, g = _successor(seed, vocab), torch.Generator().manual_seed(int(seed) * 15485863 + 2)
    chain, t = [], torch.as_tensor(last, dtype=torch.int64)
    for _ in range(gamma):
        t = torch.where(torch.rand(b, generator=g) < 0.25, torch.randint(0, vocab, (b,), generator=g), succ[t])
        chain.append(t)
    cand = torch.stack(chain, 1).int().cuda() if gamma else torch.zeros((b, 0), dtype=torch.int32, device="cuda")
    q = 0.1 * torch.softmax(TAIL_STD * torch.randn((b, gamma, vocab), device="cuda", generator=_gen(seed, 31)), dim=-1)
    q.scatter_add_(2, cand.long()[..., None], torch.full((b, gamma, 1), 0.9, device="cuda"))
    return cand.contiguous(), q.contiguous()


def _lora(shape, seed, n, rank):
    g = _gen(seed, 41)

    def fac(*dims):
        return torch.empty(dims, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=g)

    w = {"n_adapters": n, "rank": rank}
    for p in ("q", "k", "v", "o"):
        w["a_" + p] = [fac(n, rank, shape.d_model) for _ in range(shape.n_layers)]
        w["b_" + p] = [fac(n, shape.d_model, rank) for _ in range(shape.n_layers)]
    return w


LORA_RANK, LORA_SCALE = 8, 2.0
SLACK = 1024  # tokens a conversation may grow by before it starts over
SYNC_EVERY = 32  # passes between two reads of the lengths


def _accept_inputs(case, seed):
    n, gamma, v = case["n"], case["gamma"], case["vocab"]
    logits = TAIL_STD * torch.randn((n, gamma + 1, v), device="cuda", generator=_gen(seed, 3))
    last = torch.randint(0, v, (n,), generator=torch.Generator().manual_seed(int(seed)))
    cand, q = _candidates(seed, n, gamma, v, last)
    succ = _successor(seed, v)[torch.cat([last[:, None], cand.cpu().long()], 1)]  # the target's own choice at each row
    logits.scatter_(2, succ.cuda()[..., None], 0.9 * SUCCESSOR)
    return logits, cand, q, _uniforms(seed, 4, n, gamma + 1)


def _classifier_inputs(case, seed):
    shape = dg.ClassifierShape()
    tokens, lens = dg.make_classifier_prompts(seed, case["n"], shape.vocab, case["max_len"])
    return shape, dg.make_classifier(shape, seed), tokens, lens


def prepare(case, seed):
    kind = case["kind"]
    dev = dict(device="cuda")
    st = {"case": case, "passes": 0}
    if kind == "accept":
        logits, cand, q, u = _accept_inputs(case, seed)
        n, gamma = case["n"], case["gamma"]
        st.update(logits=logits, cand=cand, q=q, u=u, ws=torch.zeros(3 * n * (gamma + 1), **dev))
    elif kind == "classify":
        shape, w, tokens, lens = _classifier_inputs(case, seed)
        st.update(cls=api.Classifier(shape, w), tokens=torch.from_numpy(tokens).cuda(), lens=torch.from_numpy(lens).cuda(),
                  logits=torch.zeros((case["n"], shape.n_classes), **dev))
        n = case["n"]
    else:
        shape, b, gamma = _shape(case), case["b"], case["gamma"]
        v = shape.vocab
        n = b
        prompts = _prompts(case, seed, v)
        longest = max(len(p) for p in prompts)
        slack = SLACK if kind != "prefill" else 4 * (gamma + 1)
        rows = max(case.get("rows", 1024), b * (gamma + 1), 2 * b)
        w = _weights(shape, seed, 11)
        m = _model(shape, w, rows, longest + slack + 64)
        del w
        st.update(m=m, prompts=prompts, slack=slack, models=[m])
        if kind == "step":
            ds = dg.SHAPES["tiny_draft"]
            st["draft"] = _model(ds, _weights(ds, seed, 12), rows, longest + slack + 64)
            st["models"].append(st["draft"])
        if case.get("adapters"):
            lw = _lora(shape, seed, case["adapters"], LORA_RANK)
            host = {k: [t.view(torch.int16).cpu().numpy().view(np.uint16) for t in x] if isinstance(x, list) else x for k, x in lw.items()}
            m.set_lora(host, LORA_SCALE)
        ctx = api.Context([len(p) + slack for p in prompts])
        for x in st["models"]:
            ctx.attach(x)
        if case.get("adapters"):
            ctx.set_adapters(m, [j % (case["adapters"] + 1) - 1 for j in range(len(prompts))])
        st["ctx"] = ctx
        if kind != "prefill":
            _begin(st)
        turns = len(prompts) // b  # groups of conversations that are advanced in turn
        st["ids"] = [torch.arange(t * b, (t + 1) * b, dtype=torch.int32, **dev) for t in range(turns)]
        st["u_draft"], st["u"] = _uniforms(seed, 5, b, max(1, gamma)), _uniforms(seed, 4, b, gamma + 1)
        if kind in ("draft", "step"):
            st["cand"] = torch.zeros((b, gamma), dtype=torch.int32, **dev)
            st["q"] = torch.zeros((b, gamma, v), **dev)
        else:
            st["cand"], st["q"] = _candidates(seed, b, gamma, v, [int(p[-1]) for p in prompts[:b]])
        if kind == "draft":  # what the verification elsewhere decided: nothing accepted, this token instead
            st["rejected"] = torch.zeros(b, dtype=torch.int32, **dev)
            st["instead"] = torch.randint(0, v, (b,), dtype=torch.int32, generator=_gen(seed, 6), **dev)
    st["na"], st["nx"] = (torch.zeros(n, dtype=torch.int32, **dev) for _ in range(2))
    return st


def _begin(st):
    """New conversations: prompts into the context, caches of every model prefilled."""
    ctx, prompts = st["ctx"], st["prompts"]
    ctx.set_tokens(prompts)
    for m in st["models"]:
        per = max(1, m.max_rows // 512)
        for s in range(0, len(prompts), per):
            part = prompts[s:s + per]
            ids = torch.arange(s, s + len(part), dtype=torch.int32, device="cuda")
            api.sd_prefill(m, ctx, ids, len(part), max(len(p) for p in part) - 1)
            torch.cuda.synchronize()
    st["grown"] = 0


# ---------------------------------------------------------------- one pass

def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "accept":
        api.sd_accept(st["logits"], case["gamma"], case["temp"], st["cand"], st["q"], st["u"], st["na"], st["nx"], st["ws"])
        return {"n_accepted": st["na"], "next": st["nx"]}
    if kind == "classify":
        st["cls"].route(st["tokens"], st["lens"], st["na"], st["logits"])
        return {"logits": st["logits"], "draft_id": st["na"]}
    ctx, m, b, gamma, temp = st["ctx"], st["m"], case["b"], case["gamma"], case["temp"]
    if kind == "prefill":
        ctx.set_tokens(st["prompts"])
        api.sd_prefill(m, ctx, None, b, max(len(p) for p in st["prompts"]) - 1)
        api.sd_verify(m, ctx, None, b, gamma, temp, st["cand"], st["q"], st["u"], st["na"], st["nx"], commit=False)
        return {"logits": m.last_logits(), "n_accepted": st["na"], "next": st["nx"]}
    turn = st["passes"] % len(st["ids"])
    if st["passes"] and st["passes"] % SYNC_EVERY == 0:
        ctx.sync()
    if turn == 0 and st["grown"] + gamma + 1 > st["slack"] - 16:
        _begin(st)
    if turn == 0:
        st["grown"] += 1 if kind == "draft" else gamma + 1
    st["passes"] += 1
    ids = st["ids"][turn]
    if kind == "draft":
        api.sd_draft(m, ctx, ids, b, gamma, temp, st["u_draft"], st["cand"], st["q"])
        api.sd_commit(ctx, ids, b, gamma, st["cand"], st["rejected"], st["instead"])
        return {"cand": st["cand"], "q": st["q"], "logits": m.last_logits()}  # (of the last candidate's row)
    if kind == "step":
        api.sd_draft(st["draft"], ctx, ids, b, gamma, temp, st["u_draft"], st["cand"], st["q"])
    api.sd_verify(m, ctx, ids, b, gamma, temp, st["cand"], st["q"], st["u"], st["na"], st["nx"], commit=True)
    out = {"logits": m.last_logits(), "n_accepted": st["na"], "next": st["nx"]}
    if kind == "step":
        out.update(cand=st["cand"], q=st["q"])
    return out


# ---------------------------------------------------------------- what a pass cannot do without

def _forward_work(shape, rows, lm_rows, keys):
    """Bytes and flops of one forward over `rows` rows: weights once, the cache once (`keys` cached tokens in all),
    embedding rows, new cache rows, logits; 2 flops per weight and row, 4 per (row, visible token, width)."""
    esz = 2 if shape.dtype == dg.BF16 else 4
    d, f, v, L = shape.d_model, shape.d_ffn, shape.vocab, shape.n_layers
    lin = L * (4 * d * d + 3 * d * f)
    byt = (lin + (v * d if lm_rows else 0)) * esz + (keys + rows) * 2 * L * d * esz + rows * d * esz + lm_rows * v * 4
    flop = 2.0 * rows * lin + 2.0 * lm_rows * v * d
    return byt, flop


def work(case):
    kind = case["kind"]
    if kind == "accept":
        n, g, v = case["n"], case["gamma"], case["vocab"]
        return {"bytes": 4.0 * n * v * (g + 1) + (4.0 * n * v if g and case["temp"] > 0 else 0), "flops": 4.0 * n * (g + 1) * v}
    if kind == "classify":
        tokens = case["n"] * min(28.0, case["max_len"])  # mean length of the prompts
        di, j, ds, dm = 192, 38, 16, 96
        return {"bytes": tokens * (2 * di * 4 + 4) + 4e5, "flops": tokens * di * (2 * j + 2 * 6 + 6 * ds + 20) + case["n"] * 2.0 * di * dm}
    shape, b, gamma = _shape(case), case["b"], case["gamma"]
    mean = 0.5 * (case["lo"] + case["hi"])
    att = 4.0 * shape.n_layers * shape.d_model
    if kind == "prefill":
        tok = b * mean
        byt, flop = _forward_work(shape, tok, b * (gamma + 1), 0)
        return {"bytes": byt, "flops": flop + att * b * mean * mean / 2}
    if kind == "draft":
        byt = flop = 0.0
        for i in range(gamma):
            x, y = _forward_work(shape, b, b, b * (mean + i))
            byt, flop = byt + x + 4.0 * b * shape.vocab, flop + y + att * b * (mean + i)
        return {"bytes": byt, "flops": flop}
    rows = b * (gamma + 1)
    byt, flop = _forward_work(shape, rows, rows, b * mean)
    q = 4.0 * b * shape.vocab if gamma and case["temp"] > 0 else 0.0
    byt, flop = byt + q, flop + att * rows * mean
    if kind == "step":
        ds = dg.SHAPES["tiny_draft"]
        for i in range(gamma):
            x, y = _forward_work(ds, b, b, b * (mean + i))
            byt, flop = byt + x, flop + y
    return {"bytes": byt, "flops": flop}


def tolerance(case):
    """Four times what the same path shows with its sums in another order (K splits, block shapes, attention splits) and
    against exact(), over three seeds: a bf16 cache row that rounds the other way moves logits by about 1e-5."""
    kind = case["kind"]
    if kind == "accept":
        return {"rel": 0.0, "differ": 0.01}
    if kind == "classify":
        return {"rel": 4e-6, "max": 4e-5, "differ": 0.01}
    if kind == "step":
        return {"rel": 4e-6, "max": 2e-5, "differ": 0.01}
    if kind == "draft":
        return {"rel": 1.2e-4, "max": 1e-3, "differ": 0.01}
    return {"rel": 1.2e-4, "max": 6e-4, "differ": 0.01}


# ---------------------------------------------------------------- the same numbers in 64 bits

class _Exact:
    """A decoder in float64 on the weights of _weights(); the cache rows of a bf16 model are rounded to bf16, the type
    they are kept in."""

    def __init__(self, shape, w, lora=None):
        self.s, self.w, self.lora = shape, w, lora

    def norm(self, x, g):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + self.s.rms_eps) * g.double()

    def rope(self, x, pos):
        half = self.s.head_dim // 2
        inv = self.s.rope_base ** (-2.0 * torch.arange(half, device="cuda", dtype=torch.float64) / self.s.head_dim)
        a = pos.double()[:, None] * inv[None]
        c, s = torch.cos(a)[:, None], torch.sin(a)[:, None]
        x0, x1 = x[..., :half], x[..., half:]
        return torch.cat([x0 * c - x1 * s, x1 * c + x0 * s], -1)

    def stored(self, x):
        return x.float().to(torch.bfloat16).double() if self.s.dtype == dg.BF16 else x

    def delta(self, p, l, x, a):
        if self.lora is None or a < 0:
            return 0.0
        return LORA_SCALE * ((x @ self.lora["a_" + p][l][a].double().t().contiguous()) @ self.lora["b_" + p][l][a].double().t().contiguous())

    def logits(self, seqs, last, adapter=None):
        """Logits of the last `last` positions of each token sequence: [len(seqs)][last][vocab]."""
        s, w = self.s, self.w
        H, hd, d = s.n_heads, s.head_dim, s.d_model
        xs = [w["embed"][torch.as_tensor(t, device="cuda").long()].double() for t in seqs]
        for l in range(s.n_layers):
            mats = {n: w[n][l].double().t().contiguous() for n in ("wq", "wk", "wv", "wo", "wgate", "wup", "wdown")}
            for j, x in enumerate(xs):
                a = -1 if adapter is None else adapter[j]
                n = x.shape[0]
                keep = last if l == s.n_layers - 1 else n  # rows this layer still has to produce
                h = self.norm(x, w["norm_attn"][l])
                hq = h[n - keep:]
                pos = torch.arange(n, device="cuda")
                q = self.rope((hq @ mats["wq"] + self.delta("q", l, hq, a)).view(keep, H, hd), pos[n - keep:])
                k = self.stored(self.rope((h @ mats["wk"] + self.delta("k", l, h, a)).view(n, H, hd), pos))
                v = self.stored((h @ mats["wv"] + self.delta("v", l, h, a)).view(n, H, hd))
                kt, vt = k.permute(1, 2, 0).contiguous(), v.permute(1, 0, 2).contiguous()
                o = torch.empty((keep, H, hd), device="cuda", dtype=torch.float64)
                step = max(16, min(keep, int(2e8 / (n * H))))
                for r in range(0, keep, step):
                    e = min(keep, r + step)
                    sc = torch.matmul(q[r:e].permute(1, 0, 2).contiguous(), kt) / math.sqrt(hd)
                    sc.masked_fill_(pos[None, None, :] > pos[n - keep + r:n - keep + e][None, :, None], -math.inf)
                    o[r:e] = torch.matmul(torch.softmax(sc, -1), vt).permute(1, 0, 2)
                o = o.reshape(keep, d)
                x = x[n - keep:] + o @ mats["wo"] + self.delta("o", l, o, a)
                h = self.norm(x, w["norm_ffn"][l])
                xs[j] = x + (torch.nn.functional.silu(h @ mats["wgate"]) * (h @ mats["wup"])) @ mats["wdown"]
        head = w["lm_head"].double().t().contiguous()
        return torch.stack([self.norm(x[-last:], w["final_norm"]) @ head for x in xs])


def _exact_draft(model, prompts, gamma, temp, u, adapter=None):
    seqs, qs, cands = [list(p) for p in prompts], [], []
    for i in range(gamma):
        lg = model.logits(seqs, 1, adapter)[:, 0]
        if temp > 0:
            q = torch.softmax(lg / temp, -1)
            cum = torch.cumsum(q, -1)
            pick = (cum > u[:, i:i + 1].double() * cum[:, -1:]).int().argmax(-1)
            qs.append(q)
        else:
            pick = lg.argmax(-1)
            qs.append(torch.zeros_like(lg))
        cands.append(pick)
        for s, c in zip(seqs, pick.tolist()):
            s.append(c)
    return torch.stack(cands, 1), torch.stack(qs, 1), lg


def exact(case, seed):
    kind = case["kind"]
    if kind == "accept":
        return None  # whole numbers only
    if kind == "classify":
        return {"logits": _exact_classifier(case, seed), "draft_id": None}
    shape, b, gamma, temp = _shape(case), case["b"], case["gamma"], case["temp"]
    prompts = _prompts(case, seed, shape.vocab)[:b]
    lora = _lora(shape, seed, case["adapters"], LORA_RANK) if case.get("adapters") else None
    model = _Exact(shape, _weights(shape, seed, 11), lora)
    u = _uniforms(seed, 5, b, max(1, gamma))
    if kind == "draft":
        adapter = [j % (case["adapters"] + 1) - 1 for j in range(b)] if lora else None
        _, q, lg = _exact_draft(model, prompts, gamma, temp, u, adapter)
        return {"cand": None, "q": q, "logits": lg}
    out = {}
    if kind == "step":
        ds = dg.SHAPES["tiny_draft"]
        cand, q, _ = _exact_draft(_Exact(ds, _weights(ds, seed, 12)), prompts, gamma, temp, u)
        out.update(cand=None, q=q)
    else:
        cand, _ = _candidates(seed, b, gamma, shape.vocab, [int(p[-1]) for p in prompts])
    lg = model.logits([list(p) + c for p, c in zip(prompts, cand.tolist())], gamma + 1)
    return {"logits": lg.reshape(b * (gamma + 1), -1), "n_accepted": None, "next": None, **out}


def _exact_classifier(case, seed):
    shape, w, tokens, lens = _classifier_inputs(case, seed)
    t = {k: torch.from_numpy(x).cuda().double() for k, x in w.items()}
    ids, n_tok = torch.from_numpy(tokens).cuda().long(), torch.from_numpy(lens).cuda()
    n, L, di, ds, dr = ids.shape[0], ids.shape[1], shape.d_inner, shape.d_state, shape.dt_rank
    xz = t["emb"][ids] @ t["w_in"]
    x, z = xz[..., :di], xz[..., di:]
    xp = torch.cat([torch.zeros((n, shape.d_conv - 1, di), device="cuda", dtype=torch.float64), x], 1)
    x = torch.nn.functional.silu(t["conv_b"] + sum(t["conv_w"][:, j] * xp[:, j:j + L] for j in range(shape.d_conv)))
    r = x @ t["w_x"]
    delta = torch.nn.functional.softplus(r[..., :dr] @ t["w_dt"] + t["b_dt"], threshold=100.0)
    A, h = -torch.exp(t["a_log"]), torch.zeros((n, di, ds), device="cuda", dtype=torch.float64)
    pooled = torch.zeros((n, di), device="cuda", dtype=torch.float64)
    for s in range(L):
        dl = delta[:, s, :, None]
        h = torch.exp(dl * A) * h + dl * x[:, s, :, None] * r[:, s, None, dr:dr + ds]
        y = ((h * r[:, s, None, dr + ds:]).sum(-1) + t["d"] * x[:, s]) * torch.nn.functional.silu(z[:, s])
        pooled += torch.where((s < n_tok)[:, None], y, 0.0)
    pooled = pooled / n_tok.clamp(min=1)[:, None]
    return (pooled @ t["w_out"]) @ t["w_fc"].t().contiguous() + t["b_fc"]
