"""Performance cases of the speculative-decoding step: what a serving program has
the engine do, through its public entry points (SDEngine, Batch, accept_resample
and HIP graphs over them), at the sizes of the repository's workloads.

A case is a dict of plain values with a "kind":

  accept   acceptance / resampling of a batch on given p, q and uniforms
  draft    the draft calls of one step of a batch (gamma calls)
  verify   the target's verification pass of a batch
  step     draft calls, verification and acceptance of one step
  request  new tasks arrive: prefill, `steps` whole decoding steps, release

Models are layer cuts ("layers") of the repository's model pairs with their full
width and vocabulary: every layer of a pass is the same work, so a cut measures the
layer.  Weights are N(0, 0.02^2) (norm gains around 1); they belong to the engine a
program keeps, and do not depend on the seed.  Prompts, draft tokens, uniforms and
distributions come from the seed.

Tokens that are sampled or arg-maxed from 16-bit logits flip with any change of
rounding, and what follows a flipped token is another computation.  So the draft
tokens that a pass consumes are fixed by the seed: verification passes get them
written into the batch, chains of draft calls run greedy with every token forced
(sd_force_draft at alpha = 1), and the outputs are logits and distributions.
"""
from __future__ import annotations

import gc
import math
import zlib
from collections import OrderedDict

import numpy as np
import torch

import synth
from paper_2510_11331_amd import SDEngine
from paper_2510_11331_amd.engine import Batch, accept_resample

DEVICE = "cuda"

PAIRS = {
    "tiny": ("tiny_target", "tiny_draft"),
    "small": ("small_target", "small_draft"),
    "7b": ("7b_target", "7b_draft"),
    "13b": ("13b_target", "13b_draft"),
}


def listed():
    return [
        # a short prompt on the fp32 pair, four decoding steps, eager: the smallest
        # request, where launches and latency count
        dict(name="tiny_request", kind="request", pair="tiny", layers=2, batch=2, gamma=4, lo=32, hi=32, steps=4,
             rows=256),
        # acceptance of a decoding batch on its own (no engine needed)
        dict(name="accept_b8", kind="accept", batch=8, gamma=4, vocab=32000, greedy=False),
        # one sampled draft call at the headline batch
        dict(name="draft_7b_b8", kind="draft", pair="7b", layers=1, batch=8, gamma=1, lo=1024, hi=1024, greedy=False),
        # the draft chain of a large greedy batch
        dict(name="draft_13b_b64", kind="draft", pair="13b", layers=1, batch=64, gamma=4, lo=512, hi=512, greedy=True),
        # verification: a single user
        dict(name="verify_7b_b1", kind="verify", pair="7b", layers=2, batch=1, gamma=4, lo=1024, hi=1024, graph=True),
        # verification: the headline batch
        dict(name="verify_7b_b8", kind="verify", pair="7b", layers=2, batch=8, gamma=4, lo=1024, hi=1024, graph=True),
        # verification: ragged paged prompts, eager as in the two-stream pipeline
        dict(name="verify_7b_b32", kind="verify", pair="7b", layers=2, batch=32, gamma=4, lo=128, hi=2048, graph=False),
        # verification: a large batch of the widest model
        dict(name="verify_13b_b64", kind="verify", pair="13b", layers=2, batch=64, gamma=4, lo=512, hi=512, graph=True),
        # a whole step of a whole model (grouped KV heads, head dimension 64)
        dict(name="step_small_b8", kind="step", pair="small", layers=16, batch=8, gamma=4, lo=512, hi=512),
        # long contexts, long speculation, few tasks
        dict(name="verify_long_b2", kind="verify", pair="small", layers=4, batch=2, gamma=8, lo=15000, hi=16000,
             graph=True),
        # time to the first verified tokens of one prompt
        dict(name="request_7b_b1", kind="request", pair="7b", layers=4, batch=1, gamma=4, lo=1024, hi=1024, steps=1,
             rows=1024),
        # a batch of ragged prompts arrives
        dict(name="request_7b_b8", kind="request", pair="7b", layers=4, batch=8, gamma=4, lo=128, hi=2048, steps=1,
             rows=2048),
    ]


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    kind = rng.choice(["accept", "draft", "verify", "verify", "verify", "step", "request", "request"])
    if kind == "accept":
        return dict(kind=kind, batch=_log_uniform(rng, 1, 64), gamma=rng.randint(1, 8),
                    vocab=4 * _log_uniform(rng, 64, 8000), greedy=rng.random() < 0.25)
    pair = rng.choice(["small", "7b", "7b", "13b"])
    if kind == "request":
        # up to 6000 prompt tokens in all
        batch = _log_uniform(rng, 1, 16)
        hi = min(_log_uniform(rng, 64, 3000), 6000 // batch)
        lo = rng.randint(max(1, hi // 8), hi)
        return dict(kind=kind, pair=pair, layers=rng.randint(2, 3), batch=batch, gamma=rng.randint(1, 8), lo=lo, hi=hi,
                    steps=1, rows=rng.choice([256, 1024, 2048]))
    batch = _log_uniform(rng, 1, 64)
    hi = min(_log_uniform(rng, 128, 8192), 32768 // batch)
    lo = rng.randint(hi // 8, hi)
    case = dict(kind=kind, pair=pair, layers=rng.randint(1, 2), batch=batch, gamma=rng.randint(1, 8), lo=lo, hi=hi)
    if kind == "draft":
        case["greedy"] = rng.random() < 0.5
        if not case["greedy"]:
            case["gamma"] = 1
    if kind == "verify":
        case["graph"] = rng.random() < 0.7
    return case


# --------------------------------------------------------------------------
# models and engines


def _shapes(case):
    t, d = (synth.MODELS[n] for n in PAIRS[case["pair"]])
    return t.replace(n_layers=case["layers"]), d


def _weight(shape, role, name):
    """One weight tensor on the GPU, in the model's dtype; the same for every seed."""
    dims = synth.weight_shapes(shape)[name]
    g = torch.Generator(device=DEVICE)
    g.manual_seed(zlib.crc32(f"{role}.{name}.{shape.d_model}".encode()))
    w = torch.randn(dims, generator=g, device=DEVICE, dtype=torch.float32)
    w = 1.0 + 0.1 * w if name.endswith("norm") else 0.02 * w
    return w.to(torch.bfloat16) if shape.dtype == "bf16" else w


def _host(shape, role):
    def get(name):
        w = _weight(shape, role, name)
        if shape.dtype == "bf16":
            return w.view(torch.int16).cpu().numpy().view(np.uint16)
        return w.cpu().numpy()
    return get


GROUPS = 4            # states of one case that may be alive together
_ENGINES: "OrderedDict" = OrderedDict()


class Serving:
    """The engine of one case, as a serving program keeps it, with GROUPS sets of
    slots to hand out."""

    def __init__(self, case):
        t, d = _shapes(case)
        B = case["batch"]
        steps = case.get("steps", 1)
        self.greedy = case["kind"] in ("step", "request") or bool(case.get("greedy"))
        self.max_new = (steps + 1) * (case["gamma"] + 1)
        self.eng = SDEngine(t, d, _host(t, "target"), _host(d, "draft"), max_slots=GROUPS * B, max_batch=B,
                            gamma_max=case["gamma"], max_ctx=case["hi"] + self.max_new + case["gamma"] + 16,
                            prefill_rows=case.get("rows", 2048), temperature=1.0, greedy=self.greedy)
        self.free = list(range(GROUPS))

    def take(self):
        if not self.free:
            gc.collect()
        return self.free.pop(0)


def _serving(case):
    key = tuple(sorted((k, v) for k, v in case.items() if k not in ("name", "graph")))
    s = _ENGINES.pop(key, None)
    if s is None:
        s = Serving(case)
    _ENGINES[key] = s
    while len(_ENGINES) > 12:
        _ENGINES.popitem(last=False)
    return s


# --------------------------------------------------------------------------
# inputs


def _lengths(case):
    return [int(n) for n in synth.ragged_lengths(case["batch"], case["lo"], case["hi"])]


def _inputs(case, seed):
    """Prompts, draft tokens [B, gamma], forced continuations [B, max_ctx] and uniforms of a seed."""
    r = np.random.default_rng([seed, 17])
    V = synth.MODELS[PAIRS[case["pair"]][0]].vocab
    B, g = case["batch"], case["gamma"]
    prompts = [r.integers(0, V, size=n).astype(np.int32) for n in _lengths(case)]
    cont = r.integers(0, V, size=(B, case["hi"] + (case.get("steps", 1) + 2) * (g + 1))).astype(np.int32)
    # token i of the step after a prompt of n tokens sits at position n + i
    drafts = np.stack([cont[k, len(p):len(p) + g] for k, p in enumerate(prompts)])
    u = r.integers(0, 2 ** 32, size=(case.get("steps", 1), B, 2 * g + 1), dtype=np.uint64).astype(np.uint32)
    return prompts, drafts, cont, u


class State:
    def __init__(self, case, seed):
        self.case = case
        self.serving = _serving(case)
        eng = self.eng = self.serving.eng
        B, g = case["batch"], case["gamma"]
        self.group = self.serving.take()
        self.slots = list(range(self.group * B, (self.group + 1) * B))
        self.prompts, drafts, cont, u = _inputs(case, seed)
        self.max_new = [self.serving.max_new] * B
        self.u = torch.from_numpy(u.view(np.int32)).to(DEVICE)
        self.b = eng.batch(self.slots, g)
        self.z = None
        self.graph = None
        self.prefilled = False
        if self.serving.greedy:
            self.b.set_force(cont, 1.0)
        if case["kind"] == "request":
            self.z = [torch.empty(B, g + 1, eng.vocab, dtype=torch.float32, device=DEVICE)
                      for _ in range(case["steps"])]
            return
        eng.prefill(self.slots, self.prompts, self.max_new)
        self.prefilled = True
        if case["kind"] == "verify":
            for i in range(g):
                eng.draft_step(self.b, i, self.u[0])
            self.b.draft_tok.copy_(torch.from_numpy(drafts))
        self.call()
        torch.cuda.synchronize()
        if case.get("graph", True):
            self.graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(self.graph):
                self.call()

    def call(self):
        """The pass of a decoding case: it rewrites the same uncommitted positions, so it can be repeated."""
        eng, b, kind = self.eng, self.b, self.case["kind"]
        if kind in ("draft", "step"):
            for i in range(b.gamma):
                eng.draft_step(b, i, self.u[0])
        if kind in ("verify", "step"):
            eng.verify(b)
        if kind == "step":
            eng.accept(b, self.u[0])

    def request(self):
        eng, b = self.eng, self.b
        eng.prefill(self.slots, self.prompts, self.max_new)
        for n in range(self.case["steps"]):
            eng.step(b, self.u[n], logits=self.z[n])
        torch.cuda.current_stream().synchronize()      # the slots may be given to other tasks now
        for s in self.slots:
            eng.release(s)

    def __del__(self):
        try:
            if self.prefilled:
                torch.cuda.synchronize()
                for s in self.slots:
                    self.eng.release(s)
            self.serving.free.append(self.group)
        except Exception:
            pass


class AcceptState:
    """p and q as a draft model of middling quality gives them: softmax rows of
    correlated logits with a spread of 3, draft tokens drawn from q (arg-maxes of
    q's logits in greedy mode, where p and q hold logits)."""

    def __init__(self, case, seed):
        self.case = case
        B, g, V = case["batch"], case["gamma"], case["vocab"]
        r = torch.Generator(device=DEVICE)
        r.manual_seed(seed)
        zp = 3.0 * torch.randn(B, g + 1, V, generator=r, device=DEVICE)
        zq = 0.95 * zp[:, :g] + 0.9 * torch.randn(B, g, V, generator=r, device=DEVICE)
        if case["greedy"]:
            self.p, self.q = zp, zq.contiguous()
            self.draft_tok = zq.argmax(-1).to(torch.int32)
        else:
            self.p, self.q = torch.softmax(zp, -1), torch.softmax(zq, -1).contiguous()
            self.draft_tok = torch.multinomial(self.q.view(B * g, V), 1, generator=r).view(B, g).to(torch.int32)
        self.u = torch.randint(-2 ** 31, 2 ** 31, (B, 2 * g + 1), generator=r, device=DEVICE, dtype=torch.int64
                               ).to(torch.int32)
        self.n_acc = torch.zeros(B, dtype=torch.int32, device=DEVICE)
        self.out_tok = torch.zeros(B, g + 1, dtype=torch.int32, device=DEVICE)


def prepare(case, seed):
    return AcceptState(case, seed) if case["kind"] == "accept" else State(case, seed)


def run(state):
    case = state.case
    kind = case["kind"]
    if kind == "accept":
        accept_resample(case["batch"], case["gamma"], case["vocab"], case["greedy"], state.draft_tok, state.q, state.p,
                        state.u, state.n_acc, state.out_tok)
        return {"n_acc": state.n_acc, "out_tok": state.out_tok}
    if kind == "request":
        state.request()
        return {"logits": state.z, "q": state.b.q}
    if state.graph is not None:
        state.graph.replay()
    else:
        state.call()
    b = state.b
    if kind == "draft":
        return {"q": b.q}
    if kind == "verify":
        return {"p": b.p}
    return {"q": b.q, "p": b.p, "n_acc": b.n_acc}


# --------------------------------------------------------------------------
# what a pass cannot do without


def _layer_params(m):
    hd = m.d_model // m.n_heads
    return m.d_model * (m.n_heads + 2 * m.n_kv_heads) * hd + m.n_heads * hd * m.d_model + 3 * m.d_model * m.d_ffn


def _kv_row(m):
    return 2 * m.n_kv_heads * (m.d_model // m.n_heads)       # K and V entries of a token in one layer


def _pass(m, rows, ctx_sum, new_rows, lm_rows):
    """One decoding pass: every weight, the cached K/V of every task and the new rows' K/V once, lm_rows rows of
    logits out.  ctx_sum: cached tokens of all tasks; rows: rows computed (each attends ctx_sum / tasks tokens)."""
    e = 2 if m.dtype == "bf16" else 4
    P = m.n_layers * _layer_params(m) + m.vocab * m.d_model
    by = P * e + m.n_layers * (ctx_sum + new_rows) * _kv_row(m) * e + lm_rows * m.vocab * 4 + rows * m.d_model * e
    return by, 2.0 * m.n_layers * _layer_params(m) * rows + 2.0 * m.vocab * m.d_model * lm_rows


def work(case):
    B, g = case["batch"], case["gamma"]
    if case["kind"] == "accept":
        V = case["vocab"]
        # greedy: a row of p per tested position, at least one; sampling: a row of p and one of q
        return dict(bytes=float(B * V * 4 * (1 if case["greedy"] else 2) + B * (5 * g + 3) * 4), flops=float(4 * B * V))
    t, d = _shapes(case)
    n = _lengths(case)
    ctx = sum(n)
    by = fl = 0.0

    def attn(m, k, rows_per_task):
        return 4.0 * m.n_layers * m.d_model * rows_per_task * (ctx + B * k)

    if case["kind"] in ("draft", "step", "request"):
        for i in range(g):
            x, y = _pass(d, B, ctx + B * i, B, B)
            by, fl = by + x, fl + y + attn(d, i, 1)
    if case["kind"] in ("verify", "step", "request"):
        x, y = _pass(t, B * (g + 1), ctx, B * (g + 1), B * (g + 1))
        by, fl = by + x, fl + y + attn(t, g, g + 1)
    if case["kind"] == "request":
        by, fl = by * case["steps"], fl * case["steps"]
        for m in (t, d):
            # of the last layer, prompt rows need the keys and values only
            e = 2 if m.dtype == "bf16" else 4
            kv = m.d_model * _kv_row(m)
            by += ((m.n_layers - 1) * _layer_params(m) + kv) * e + ctx * (m.d_model + m.n_layers * _kv_row(m)) * e
            fl += 2.0 * ctx * ((m.n_layers - 1) * _layer_params(m) + kv)
            fl += 2.0 * (m.n_layers - 1) * m.d_model * sum(float(k) * k for k in n)
    return dict(bytes=float(by), flops=float(fl))


def tolerance(case):
    """About four times the distance to the float64 model: fp32 logits 3.9e-7; 16-bit operands 4e-4 (a draft's q) to
    2.1e-3 (the 13B width's p)."""
    if case["kind"] == "accept":
        return "exact"
    if case["pair"] == "tiny":
        return {"rel": 2e-6}
    return {"rel": 8e-3}


# --------------------------------------------------------------------------
# 64-bit reference


class Ref:
    """Decoder-only model in float64: RMSNorm, rotate-half rotary embedding, causal attention with grouped KV heads,
    SwiGLU, untied head; the weights as they are given and nothing else rounded."""

    def __init__(self, shape, role):
        self.m, self.role = shape, role

    def w(self, name):
        return _weight(self.m, self.role, name).double()

    def norm(self, x, name):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + self.m.rms_eps) * self.w(name)

    def rope(self, x, pos):
        hd = x.shape[-1]
        inv = self.m.rope_theta ** (-2.0 * torch.arange(hd // 2, dtype=torch.float64, device=DEVICE) / hd)
        a = pos.double()[:, None, None] * inv
        x0, x1 = x[..., :hd // 2], x[..., hd // 2:]
        return torch.cat([x0 * a.cos() - x1 * a.sin(), x0 * a.sin() + x1 * a.cos()], -1)

    def attend(self, q, k, v):
        """q [n, H, hd], k and v [n, KV, hd] of one sequence -> [n, H hd]."""
        n, H, hd = q.shape
        G = H // k.shape[1]
        out = torch.empty_like(q)
        idx = torch.arange(n, device=DEVICE)
        for h in range(k.shape[1]):
            kh, vh = k[:, h], v[:, h]
            for c in range(0, n, 2048):
                e = min(n, c + 2048)
                qh = q[c:e, h * G:(h + 1) * G].reshape(-1, hd)
                s = (qh @ kh[:e].t()) / math.sqrt(hd)
                s = s.view(e - c, G, e).masked_fill((idx[None, :e] > idx[c:e, None])[:, None], -math.inf)
                out[c:e, h * G:(h + 1) * G] = (torch.softmax(s, -1).view(-1, e) @ vh[:e]).view(e - c, G, hd)
        return out.reshape(n, H * hd)

    def logits(self, seqs, last):
        """Logits of the last `last` positions of every sequence, [len(seqs), last, V]."""
        m = self.m
        hd, H, KV = m.d_model // m.n_heads, m.n_heads, m.n_kv_heads
        lens = [len(s) for s in seqs]
        tok = torch.from_numpy(np.concatenate(seqs).astype(np.int64)).to(DEVICE)
        pos = torch.cat([torch.arange(n, device=DEVICE) for n in lens])
        x = self.w("embed")[tok]
        for l in range(m.n_layers):
            p = f"l{l}."
            y = self.norm(x, p + "attn_norm")
            q = self.rope((y @ self.w(p + "wq").t()).view(-1, H, hd), pos).split(lens)
            k = self.rope((y @ self.w(p + "wk").t()).view(-1, KV, hd), pos).split(lens)
            v = (y @ self.w(p + "wv").t()).view(-1, KV, hd).split(lens)
            o = torch.cat([self.attend(*a) for a in zip(q, k, v)])
            x = x + o @ self.w(p + "wo").t()
            y = self.norm(x, p + "ffn_norm")
            gate = y @ self.w(p + "w_gate").t()
            x = x + (gate * torch.sigmoid(gate) * (y @ self.w(p + "w_up").t())) @ self.w(p + "w_down").t()
        x = torch.stack([s[-last:] for s in x.split(lens)])
        return self.norm(x, "final_norm") @ self.w("lm_head").t()


def exact(case, seed):
    if case["kind"] == "accept":
        return None                    # whole numbers
    t, d = _shapes(case)
    g = case["gamma"]
    prompts, drafts, cont, _ = _inputs(case, seed)
    seqs = [list(p) for p in prompts]
    tgt, dft = Ref(t, "target"), Ref(d, "draft")
    if case["kind"] == "draft":
        q = dft.logits([np.array(s + list(c[:g - 1])) for s, c in zip(seqs, drafts)], g)
        return {"q": q if case["greedy"] else torch.softmax(q, -1)}
    zs, q, n_acc = [], None, None
    for _ in range(case.get("steps", 1)):
        dr = [cont[k, len(s):len(s) + g] for k, s in enumerate(seqs)]
        z = tgt.logits([np.array(s + list(c)) for s, c in zip(seqs, dr)], g + 1)
        if case["kind"] != "verify":
            q = dft.logits([np.array(s + list(c[:g - 1])) for s, c in zip(seqs, dr)], g)
        zs.append(z)
        am = z.argmax(-1).cpu().numpy()
        n_acc = []
        for k, s in enumerate(seqs):
            a = 0
            while a < g and dr[k][a] == am[k, a]:
                a += 1
            n_acc.append(a)
            s += [int(x) for x in dr[k][:a]] + [int(am[k, a])]
    if case["kind"] == "verify":
        return {"p": torch.softmax(zs[0], -1)}
    if case["kind"] == "step":
        return {"q": q, "p": zs[0], "n_acc": None}
    return {"logits": zs, "q": q}
