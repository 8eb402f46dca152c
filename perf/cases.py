"""Performance cases of the verification library: what a program that serves or trains with it calls.

A case is a dict of plain values.  `call` names the entry point:

  step     sj_verify_step      one verification cycle of a draft block (the serving loop of the target model)
  draft    sj_draft_block      gamma single-token decodes (the serving loop of the draft model)
  prefill  sj_prefill          a prompt into an empty cache, then sj_score_block of a short continuation
  score    sj_score_block      teacher-forced log-probabilities and a judge feature (building the judge's training set)
  head     sj_verify_head      the verification tail alone on given hidden states
  train    sj_judge_train      training of the judge over a grid of C

Model shapes are those of the repository's workloads, with fewer layers where a whole stack would only repeat the
same launches.  A model's weights belong to its shape and are kept between states, as a program keeps them; caches,
prompts, drafts and uniforms come from the seed.  The LM head is scaled so that next-token distributions are as peaked
as a language model's (a few tokens carry most of the mass): in a flat one, the token that a uniform draws changes with
the last bits of the logits, and with it everything that is decoded after it.
"""
from __future__ import annotations

import math
import random
import zlib
from collections import OrderedDict

import numpy as np
import torch

import paper_2510_02329_amd as sj

# d_model, query heads, kv heads, head dim, FFN width, vocabulary, dtype, rotary base
MODELS = {
    "tiny": (256, 4, 4, 64, 768, 4096, "fp32", 10000.0),
    "small": (512, 8, 2, 128, 1408, 4992, "bf16", 500000.0),
    "1b": (2048, 32, 8, 64, 8192, 128256, "bf16", 500000.0),
    "8b": (4096, 32, 8, 128, 14336, 128256, "bf16", 500000.0),
    "70b": (8192, 64, 8, 128, 28672, 128256, "bf16", 500000.0),
}
EPS = 1e-5
C_GRID = [float(c) for c in np.logspace(-3, 2, 10)]     # the paper's grid
THETA = 0.5
DEV = "cuda:0"


def _case(name, call, model, layers, batch, n, ctx_lo=0, ctx_hi=0, temperature=1.0, mode=0):
    """n: draft length (step, draft, head), rows per sequence (score), prompt length (prefill)."""
    case = {"call": call, "model": model, "layers": layers, "batch": batch, "n": n, "ctx_lo": ctx_lo, "ctx_hi": ctx_hi,
            "temperature": temperature, "mode": mode}
    return {"name": name, **case} if name else case


def listed():
    return [
        # the smallest model: launches and gaps are all there is
        _case("step tiny fp32", "step", "tiny", 2, 1, 4, 128, 128),
        # interactive serving, the benchmark's workload: one user, the whole 32-layer target
        _case("step 8b b1", "step", "8b", 32, 1, 5, 1024, 1024),
        # a few users at odd lengths, greedy (the paper's evaluation setting): 20 rows
        _case("step 8b b5 greedy", "step", "8b", 4, 5, 3, 77, 1900, 0.0),
        # batched serving, ragged contexts: 144 rows
        _case("step 8b b16", "step", "8b", 4, 16, 8, 512, 4096),
        # the large target at its batch: 24 rows
        _case("step 70b b4", "step", "70b", 2, 4, 5, 2048, 2048),
        # the draft model beside it, one user and a batch
        _case("draft 1b b1", "draft", "1b", 16, 1, 5, 1024, 1024),
        _case("draft 1b b12", "draft", "1b", 16, 12, 4, 100, 1500),
        # admission of a request: a prompt into an engine whose blocks are gamma + 1 = 6 rows
        _case("prefill 8b", "prefill", "8b", 4, 1, 509),
        # labels of the judge's training set: N + 1 = 21 rows at several mismatch positions
        _case("score 8b b6", "score", "8b", 4, 6, 21, 60, 700),
        # the tail alone: a handful of rows, and the large batch where it is a dense product
        _case("head b2", "head", "8b", 0, 2, 5),
        _case("head b64", "head", "8b", 0, 64, 8),
        # training of the judge, a quarter of the paper's set: n = training rows of d_model features
        _case("train judge 8b", "train", "8b", 0, 1, 17358),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng: random.Random):
    call = rng.choice(["step", "step", "step", "draft", "prefill", "score", "head", "train"])
    if call == "train":
        return _case(None, "train", rng.choice(["small", "1b", "8b"]), 0, 1, _log(rng, 700, 17000))
    if call == "head":
        return _case(None, "head", rng.choice(["1b", "8b"]), 0, _log(rng, 1, 64), rng.randint(1, 8), 0, 0, 1.0, rng.choice([0, 1, 2]))
    if call == "draft":
        hi = _log(rng, 40, 2000)
        return _case(None, "draft", rng.choice(["1b", "1b", "small"]), rng.randint(2, 16), _log(rng, 1, 16), rng.randint(1, 7),
                     _log(rng, 20, hi), hi)
    model = rng.choice(["tiny", "small", "1b", "8b", "8b"])
    layers = rng.randint(1, 4)
    if call == "prefill":
        return _case(None, "prefill", model, layers, 1, _log(rng, 10, 500))
    hi = _log(rng, 40, 4000)
    lo = _log(rng, 20, hi)
    if call == "score":
        return _case(None, "score", model, layers, _log(rng, 1, 8), rng.randint(2, 21), lo, hi)
    return _case(None, "step", model, layers, _log(rng, 1, 16), rng.randint(1, 8), lo, hi, rng.choice([1.0, 1.0, 0.7, 0.0]),
                 rng.choice([0, 0, 1, 2, 3]))


# ------------------------------------------------------------------ inputs


class Shape:
    def __init__(self, case):
        (self.d, self.hq, self.hkv, self.hd, self.f, self.v, self.dtype, self.base) = MODELS[case["model"]]
        self.model, self.layers = case["model"], case["layers"]
        self.bf16 = self.dtype == "bf16"
        self.gamma = {"prefill": 5, "score": case["n"] - 1}.get(case["call"], case["n"])      # max_gamma of the engine

    def matrices(self):
        d, q, k = self.d, self.hq * self.hd, self.hkv * self.hd
        return {"wq": (q, d), "wk": (k, d), "wv": (k, d), "wo": (d, q), "w_gate": (self.f, d), "w_up": (self.f, d), "w_down": (d, self.f)}

    def layer_params(self):
        return sum(a * b for a, b in self.matrices().values())


def _gen(*key):
    g = torch.Generator(device=DEV)
    g.manual_seed(zlib.crc32("/".join(str(k) for k in key).encode()))
    return g


def _store(s, x):
    """Values as the model stores them."""
    return x.to(torch.bfloat16) if s.bf16 else x


def weight(s, name, layer):
    """One tensor of the model, on the device, in the storage type."""
    g = _gen("weight", s.model, name, layer)
    if name.endswith("_norm"):
        return _store(s, 1.0 + 0.1 * torch.randn(s.d, generator=g, device=DEV))
    if name == "judge_b":
        return _store(s, torch.zeros(1, device=DEV))
    if name == "judge_w":
        return _store(s, torch.randn(s.d, generator=g, device=DEV) * 0.02)
    rows, cols = (s.v, s.d) if name in ("embed", "lm_head") else s.matrices()[name]
    std = {"embed": 0.02, "lm_head": 12.0 / math.sqrt(s.d)}.get(name, 1.28 / math.sqrt(cols))
    return _store(s, torch.randn(rows, cols, generator=g, device=DEV).mul_(std))


def _bits(x):
    """Host array of a storage-type tensor in the form the library takes."""
    return x.cpu().view(torch.int16).numpy().view(np.uint16) if x.dtype == torch.bfloat16 else x.cpu().numpy()


def cache_rows(s, seed, seq, layer, length):
    g = _gen("cache", seed, seq, layer)
    kv = torch.randn(2, s.hkv, length, s.hd, generator=g, device=DEV)
    return _store(s, kv[0]), _store(s, kv[1])


def inputs(case, seed):
    """Everything a call reads besides weights and cache rows."""
    s, b, n = Shape(case), case["batch"], case["n"]
    g = _gen("inputs", seed, case["call"], case["model"], b, n)
    ints = lambda hi, *size: torch.randint(0, hi, size, generator=g, device=DEV, dtype=torch.int32)  # noqa: E731
    uni = lambda *size: torch.rand(*size, generator=g, device=DEV).clamp_(max=1.0 - 2.0 ** -24)  # noqa: E731
    lo, hi = case["ctx_lo"], case["ctx_hi"]
    x = {"lens": (ints(hi - lo + 1, b) + lo).tolist() if hi else [0] * b, "pending": ints(s.v, b).tolist()}
    if case["call"] in ("step", "head"):
        x["probs"] = torch.softmax(12.0 * torch.randn(b, n, s.v, generator=g, device=DEV), dim=-1)
        x["tokens"] = torch.multinomial(x["probs"].reshape(b * n, s.v), 1, generator=g).reshape(b, n).to(torch.int32)
        x["uniforms"] = uni(b, n + 1)
    if case["call"] == "head":
        x["hidden"] = _store(s, torch.randn(b * (n + 1), s.d, generator=g, device=DEV))
    if case["call"] == "draft":
        x["uniforms"] = uni(n, b)
    if case["call"] == "prefill":
        x["prompt"] = ints(s.v, n).tolist()
    if case["call"] in ("prefill", "score"):
        m = s.gamma + 1
        x["block"], x["targets"], x["row"] = ints(s.v, b, m), ints(s.v, b, m), m // 2
    if case["call"] == "train":
        # hidden states of unit scale; labels (61 % acceptable) shift them along a few directions with a random strength
        dirs = torch.randn(4, s.d, generator=_gen("directions", s.d), device=DEV)
        dirs /= dirs.norm(dim=1, keepdim=True)
        for part, rows in (("train", n), ("val", max(64, n // 8))):
            y = (torch.rand(rows, generator=g, device=DEV) < 0.61).to(torch.int32)
            strength = -0.5 * torch.log(torch.rand(rows, 4, 2, generator=g, device=DEV).clamp_(min=1e-30)).sum(dim=2)     # Gamma(2, 1/2)
            shift = ((2.0 * y[:, None] - 1.0) * strength) @ dirs / 2.0
            x["h_" + part], x["y_" + part] = torch.randn(rows, s.d, generator=g, device=DEV) + shift, y
    return x


# ------------------------------------------------------------------ states


class Model:
    def __init__(self, s, temperature):
        cfg = sj.SJConfig(n_layers=s.layers, d_model=s.d, n_q_heads=s.hq, n_kv_heads=s.hkv, head_dim=s.hd, d_ffn=s.f, vocab=s.v,
                          dtype=1 if s.bf16 else 0, rope_base=s.base, rms_eps=EPS, temperature=temperature, max_gamma=s.gamma)
        staging = torch.empty(max(s.v, s.f) * s.d, dtype=torch.bfloat16 if s.bf16 else torch.float32, pin_memory=True)

        def provider(name, layer):
            w = weight(s, name, layer).reshape(-1)
            staging[:w.numel()].copy_(w)
            return _bits(staging[:w.numel()])

        self.handle = sj.sj_model_load(cfg, provider)

    def __del__(self):
        if getattr(self, "handle", None):
            sj.sj_model_free(self.handle)


_models: "OrderedDict[tuple, Model]" = OrderedDict()


def _model(s, temperature):
    """The loaded model of a shape; the last four are kept."""
    key = (s.model, s.layers, s.gamma, temperature)
    if key not in _models:
        while len(_models) >= 4:
            _models.popitem(last=False)
        _models[key] = Model(s, temperature)
    _models.move_to_end(key)
    return _models[key]


class State:
    """One batch's cache and inputs, and the buffers its results go to."""

    def __init__(self, case, seed):
        s, b, n = Shape(case), case["batch"], case["n"]
        self.call, self.n, self.kv, self.model = case["call"], n, None, None
        self.__dict__.update(inputs(case, seed))
        if self.call == "train":
            return
        self.model = _model(s, case["temperature"])
        room = n + s.gamma + 1 if self.call == "prefill" else s.gamma + 2
        self.kv = sj.sj_kv_create(self.model.handle, b, [l + room for l in self.lens] if s.layers else None)
        for seq in range(b if s.layers and case["ctx_hi"] else 0):
            for layer in range(s.layers):
                k, v = cache_rows(s, seed, seq, layer, self.lens[seq])
                sj.sj_kv_set_layer(self.kv, seq, layer, _bits(k), _bits(v), self.lens[seq])
        for seq in range(b if s.layers else 0):
            sj.sj_kv_set_state(self.kv, seq, self.lens[seq], self.pending[seq])
        sj.sj_set_mode(self.kv, case["mode"])
        ints = lambda *size: torch.zeros(size, dtype=torch.int32, device=DEV)  # noqa: E731
        if self.call in ("step", "head"):
            self.accepted, self.next = ints(b), ints(b)
            host = lambda *size: torch.zeros(size, pin_memory=True).numpy()  # noqa: E731
            rows = b * (n + 1)
            self.report = {"p_at_draft": (sj.SJ_DBG_P_AT_DRAFT, host(b, n))}
            if self.call == "head":
                self.report["judge"] = (sj.SJ_DBG_JUDGE_SCORES, host(b, n))
            elif rows <= 8:
                self.report = {"logits": (sj.SJ_DBG_LOGITS, host(rows, s.v))}
            else:
                self.report["hidden"] = (sj.SJ_DBG_HIDDEN, host(rows, s.d))
        if self.call == "draft":
            self.tokens, self.probs = ints(b, n), torch.zeros(b, n, s.v, device=DEV)
        if self.call in ("prefill", "score"):
            self.logprob, self.feature = torch.zeros(b, s.gamma + 1, device=DEV), torch.zeros(b, s.d, device=DEV)

    def __del__(self):
        if getattr(self, "kv", None):
            sj.sj_kv_free(self.kv)


def prepare(case, seed):
    return State(case, seed)


def run(st):
    stream = torch.cuda.current_stream()
    if st.call == "train":
        out = sj.sj_judge_train(st.h_train, st.y_train, st.h_val, st.y_val, C_GRID, stream)
        return {k: out[k] for k in ("w_all", "auc", "best_index", "w", "b", "theta_f1", "theta_recall")}
    m = st.model.handle
    if st.call in ("step", "draft", "prefill"):
        sj.sj_kv_rewind(st.kv, st.lens, st.pending, stream)
    if st.call in ("step", "head"):
        if st.call == "step":
            sj.sj_verify_step(m, st.kv, st.n, st.tokens, st.probs, st.uniforms, THETA, st.accepted, st.next, stream)
        else:
            sj.sj_verify_head(m, st.kv, st.n, st.hidden, st.tokens, st.probs, st.uniforms, THETA, st.accepted, st.next, stream)
        # the serving loop has to see what was accepted before it drafts again: the step's outcome is read on the host
        out = {k: sj.sj_debug_fetch(st.kv, what, a) for k, (what, a) in st.report.items()}
        return {"accepted": st.accepted, "next": st.next, **out}
    if st.call == "draft":
        sj.sj_draft_block(m, st.kv, st.n, st.uniforms, True, st.tokens, st.probs, stream)
        return {"tokens": st.tokens, "probs": st.probs}
    if st.call == "prefill":
        sj.sj_prefill(m, st.kv, 0, st.prompt, stream)
    sj.sj_score_block(m, st.kv, st.logprob.shape[1], st.block, st.targets, st.logprob, st.row, st.feature, stream)
    return {"logprob": st.logprob, "feature": st.feature}


# ------------------------------------------------------------------ what a pass cannot do without


def _rows(case):
    """(query rows per sequence and forward, forwards over all layers, of those with the LM head)"""
    n = case["n"]
    return {"step": (n + 1, 1, 1), "head": (n + 1, 0, 1), "draft": (1, n + 1, n), "score": (n, 1, 1),
            "prefill": (n, 1, 1)}[case["call"]]


def work(case):
    s, b, n = Shape(case), case["batch"], case["n"]
    es = 2 if s.bf16 else 4
    if case["call"] == "train":
        rows = n + max(64, n // 8)
        # the matrices read once; a gradient and a Hessian product (two multiply-adds each) per C is the least a solver makes
        return {"bytes": 4.0 * rows * s.d, "flops": 8.0 * len(C_GRID) * n * s.d}
    r, forwards, heads = _rows(case)
    ctx = (case["ctx_lo"] + case["ctx_hi"]) / 2.0
    weights = forwards * s.layers * s.layer_params() + heads * s.v * s.d
    cached = forwards * s.layers * 2 * s.hkv * s.hd * b * (ctx + r)
    other = {"step": 4 * b * s.v, "head": 4 * b * s.v + es * b * r * s.d, "draft": 4 * b * n * s.v}.get(case["call"], 4 * b * s.d)
    lm_rows = s.gamma + 1 if case["call"] == "prefill" else b * r
    flops = 2.0 * forwards * s.layers * b * r * (s.layer_params() + 2 * s.hq * s.hd * (ctx + r / 2.0)) + 2.0 * heads * lm_rows * s.v * s.d
    return {"bytes": float(es * (weights + cached) + other), "flops": flops}


def tolerance(case):
    # Weights and cache are stored in bf16, activations between products carry 16 bits or more and sums 32.  A new K / V
    # row is rounded to bf16 when it is appended: where two correct implementations straddle a rounding boundary they
    # store neighbouring values (2^-8 apart), and the layers above carry that on.
    # Measured against 64 bits: logits, hidden states and log-probabilities 2e-5 .. 8e-4, probabilities up to 3e-3.
    if case["call"] == "train":
        return {"rel": 1e-7}             # 64-bit sums; the stopping rule bounds the distance to the optimum (up to 6e-10)
    if case["call"] == "head" or MODELS[case["model"]][6] == "fp32":
        return {"rel": 1e-4}             # 32-bit logits of up to +-50: 1e-6 of them is 2e-5 of a probability
    if case["call"] in ("prefill", "score"):
        return {"rel": 4e-3}
    return {"rel": 1e-2}


# ------------------------------------------------------------------ 64-bit results


def _w64(s, name, layer=-1):
    return weight(s, name, layer).double()


def _norm64(x, gain):
    return x / torch.sqrt((x * x).mean(dim=-1, keepdim=True) + EPS) * gain


def _rope64(s, x, pos):
    """x [heads, rows, hd] at positions pos [rows]; pairs (i, i + hd / 2)."""
    half = s.hd // 2
    ang = pos.double()[:, None] * s.base ** (-2.0 * torch.arange(half, device=DEV, dtype=torch.float64) / s.hd)
    c, t = torch.cos(ang), torch.sin(ang)
    return torch.cat([x[..., :half] * c - x[..., half:] * t, x[..., half:] * c + x[..., :half] * t], dim=-1)


def _forward64(s, tokens, caches):
    """Final normed hidden states of token blocks (one 1-D tensor per sequence) on top of caches[layer][seq] = (K, V).
    Layer by layer over the whole batch, so that a layer's weights are made once; the block's rows join the caches."""
    embed = weight(s, "embed", -1)
    xs = [embed[t.long()].double() for t in tokens]
    del embed
    for layer in range(s.layers):
        w = {k: _w64(s, k, layer) for k in s.matrices()}
        ga, gf = _w64(s, "attn_norm", layer), _w64(s, "ffn_norm", layer)
        for i, x in enumerate(xs):
            k_old, v_old = caches[layer][i]
            past, r = k_old.shape[1], x.shape[0]
            pos = past + torch.arange(r, device=DEV)
            h = _norm64(x, ga)
            heads = lambda y, count: y.reshape(r, count, s.hd).transpose(0, 1)  # noqa: E731
            q = _rope64(s, heads(h @ w["wq"].T, s.hq), pos)
            k_new = _store(s, _rope64(s, heads(h @ w["wk"].T, s.hkv), pos).float())
            v_new = _store(s, heads(h @ w["wv"].T, s.hkv).float())
            caches[layer][i] = torch.cat([k_old, k_new], 1), torch.cat([v_old, v_new], 1)
            k, v = (t.double().repeat_interleave(s.hq // s.hkv, dim=0) for t in caches[layer][i])
            score = torch.bmm(q, k.transpose(1, 2).contiguous()) / math.sqrt(s.hd)
            score.masked_fill_(torch.arange(past + r, device=DEV)[None, None, :] > pos[None, :, None], -math.inf)
            o = torch.bmm(torch.softmax(score, dim=-1), v).transpose(0, 1).reshape(r, s.hq * s.hd)
            x = x + o @ w["wo"].T
            h = _norm64(x, gf)
            xs[i] = x + (torch.nn.functional.silu(h @ w["w_gate"].T) * (h @ w["w_up"].T)) @ w["w_down"].T
    gain = _w64(s, "final_norm")
    return [_norm64(x, gain) for x in xs]


def _law64(logits, temperature):
    if temperature > 0:
        return torch.softmax(logits / temperature, dim=-1)
    return torch.nn.functional.one_hot(logits.argmax(dim=-1), logits.shape[-1]).double()


def _train64(x):
    """The optimum of every C by Newton's method with dense Hessians, and the selection rules on the validation set."""
    h, y, hv = x["h_train"].double(), x["y_train"].double(), x["h_val"].double()
    ones = lambda m: torch.cat([m, torch.ones_like(m[:, :1])], dim=1)  # noqa: E731
    h, hv, pos = ones(h), ones(hv), x["y_val"] == 1
    ridge = torch.ones(h.shape[1], dtype=torch.float64, device=DEV)
    ridge[-1] = 0.0
    w, all_w, aucs, scores = torch.zeros(h.shape[1], dtype=torch.float64, device=DEV), [], [], []
    loss = lambda w, c: 0.5 * (ridge * w * w).sum() + c * torch.nn.functional.softplus((1 - 2 * y) * (h @ w)).sum()  # noqa: E731
    for c in C_GRID:
        for _ in range(60):
            p = torch.sigmoid(h @ w)
            g = ridge * w + c * (h.T @ (p - y))
            if g.abs().max() <= 1e-11 * max(1.0, c * h.shape[0]):
                break
            step = torch.linalg.solve((h.T * (c * p * (1 - p))) @ h + torch.diag(ridge), -g)
            t, f0, slope = 1.0, loss(w, c), (g * step).sum()
            while t > 1e-6 and loss(w + t * step, c) > f0 + 1e-4 * t * slope and abs(slope) > 1e-9 * abs(f0):
                t *= 0.5
            w = w + t * step
        z = torch.sigmoid(hv @ w)
        neg = z[~pos].sort().values
        lo, up = torch.searchsorted(neg, z[pos]), torch.searchsorted(neg, z[pos], right=True)
        all_w.append(w)
        aucs.append(float((lo + up).double().sum()) / (2.0 * int(pos.sum()) * int((~pos).sum())))
        scores.append(z)
    best = int(np.argmax(aucs))
    z = scores[best]
    theta = torch.cat([torch.zeros(1, dtype=torch.float64, device=DEV), z.sort().values])
    above = lambda v: v.numel() - torch.searchsorted(v.sort().values, theta, right=True)  # noqa: E731
    tp, fp = above(z[pos]).double(), above(z[~pos]).double()
    f1 = 2 * tp / (tp + fp + int(pos.sum()))
    return {"w_all": torch.stack(all_w).cpu().numpy(), "auc": np.array(aucs), "best_index": best, "w": all_w[best][:-1].cpu().numpy(),
            "b": float(all_w[best][-1]), "theta_f1": float(theta[int((f1 == f1.max()).nonzero()[0])]), "theta_recall": float(z[~pos].max())}


def exact(case, seed):
    s, b, n = Shape(case), case["batch"], case["n"]
    x = inputs(case, seed)
    if case["call"] == "train":
        return _train64(x)
    caches = [[cache_rows(s, seed, i, layer, x["lens"][i]) for i in range(b)] for layer in range(s.layers)]
    pending = torch.tensor(x["pending"], device=DEV)
    if case["call"] == "draft":
        lm = _w64(s, "lm_head")
        probs = torch.zeros(b, n, s.v, dtype=torch.float64, device=DEV)
        tok = pending
        for j in range(n):
            hidden = torch.cat(_forward64(s, [tok[i:i + 1] for i in range(b)], caches))
            probs[:, j] = _law64(hidden @ lm.T, case["temperature"])
            cdf = probs[:, j].cumsum(dim=-1)
            tok = torch.searchsorted(cdf, x["uniforms"][j].double()[:, None] * cdf[:, -1:], right=True)[:, 0]
        return {"tokens": None, "probs": probs}
    if case["call"] == "prefill":
        _forward64(s, [torch.tensor(x["prompt"], device=DEV)], caches)
    if case["call"] in ("prefill", "score"):
        hidden = torch.stack(_forward64(s, list(x["block"]), caches))
        law = torch.log_softmax(hidden @ _w64(s, "lm_head").T, dim=-1)
        return {"logprob": torch.gather(law, 2, x["targets"].long()[:, :, None])[..., 0], "feature": hidden[:, x["row"]]}
    if case["call"] == "step":
        blocks = torch.cat([pending[:, None], x["tokens"].long()], dim=1)
        hidden = torch.cat(_forward64(s, list(blocks), caches))
    else:
        hidden = x["hidden"].double()
    lm = _w64(s, "lm_head")
    logits = hidden @ lm.T
    out = {"accepted": None, "next": None}           # draws: whole numbers, compared between implementations
    if case["call"] == "step" and b * (n + 1) <= 8:
        return {**out, "logits": logits}
    p = _law64(logits, case["temperature"]).reshape(b, n + 1, s.v)[:, :n]
    out["p_at_draft"] = torch.gather(p, 2, x["tokens"].long()[:, :, None])[..., 0]
    if case["call"] == "step":
        return {**out, "hidden": hidden}
    score = torch.sigmoid(hidden.reshape(b, n + 1, s.d)[:, 1:] @ _w64(s, "judge_w") + _w64(s, "judge_b"))
    return {**out, "judge": score}
