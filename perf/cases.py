"""The calls this library is measured on: teacher-forced scoring of candidate
sets against shared question prefixes, through the C ABI's Python binding.

A case is one model shape (whole, or its first layers where the whole model
would take too long to prepare), one compute mode and one request:

* ``ask``: a request as it arrives: jet_prefill_prefix on the questions, then
  jet_score_candidates on their candidates, then the prefix is freed;
* ``rescore``: new candidates against a prefix that the program retains
  (jet_score_candidates), or with ``noalloc`` the allocation-free entry point
  that serving loops use;
* ``trace``: prefill, a sampled reasoning trace of ``steps`` tokens frozen into
  the prefix (jet_generate_trace), then the candidates are scored.

A program loads its model once and keeps it, so models are loaded once per
process here; every request's tokens come from the seed. Prefix lengths are
spread over [p_lo, p_hi] and candidate lengths over [m_lo, m_hi] by the case
alone, so that a case's work does not depend on the seed. Prefix ids follow a
Zipf law and candidate ids are uniform, as in the library's own workloads.
"""
import json
import math
import os
import struct

import numpy as np
import torch

import jet_synth
from paper_2609_33874_amd import jet as J

MODES = {"f16": J.JET_F16, "bf16": J.JET_BF16}

# model shape -> layers kept. The 1.5B shape runs whole; of the others the
# first layers: one period of the layer pattern (delta-rule x 3 + attention),
# or two of the 27B's (a prefill runs its last attention layer for the last
# rows only, so the first of two is a full one).
LAYERS = {"dense_1p5b": 28, "dense_1p5b_q4": 8, "hybrid_4b": 4, "dense_27b": 2, "moe_35b_a3b": 4}


def _case(name, model, mode, do, q, p_lo, p_hi, k, m_lo, m_hi, steps=0, noalloc=False):
    c = dict(model=model, mode=mode, do=do, q=q, p_lo=p_lo, p_hi=p_hi, k=k, m_lo=m_lo, m_hi=m_hi, steps=steps,
             noalloc=noalloc)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one multiple-choice question as an interactive request: latency
        _case("1.5B one question", "dense_1p5b", "f16", "ask", 1, 237, 237, 4, 1, 24),
        # further candidates for a question whose prefix is kept, in a serving loop
        _case("1.5B kept prefix", "dense_1p5b", "f16", "rescore", 1, 731, 731, 4, 1, 24, noalloc=True),
        # a small batch of requests
        _case("1.5B 16 questions", "dense_1p5b", "f16", "ask", 16, 150, 900, 4, 1, 24),
        # bulk evaluation of a multiple-choice set: throughput
        _case("1.5B 128 questions", "dense_1p5b", "f16", "ask", 128, 150, 900, 4, 1, 24),
        # yes/no decisions over long contexts: two one-token answers each
        _case("1.5B yes/no", "dense_1p5b", "f16", "ask", 24, 300, 2000, 2, 1, 1),
        # ratings of retained long contexts, a few tokens per level
        _case("1.5B ratings", "dense_1p5b", "f16", "rescore", 128, 300, 2000, 5, 1, 3),
        # a short reasoning trace before the decision: decode steps
        _case("1.5B trace", "dense_1p5b", "f16", "trace", 8, 150, 300, 4, 1, 24, steps=16),
        # block-quantized weights (int4), a few questions at a time
        _case("1.5B int4 4 questions", "dense_1p5b_q4", "f16", "ask", 4, 150, 900, 4, 1, 24),
        # the recurrent hybrid: one request, and a batch
        _case("hybrid one question", "hybrid_4b", "bf16", "ask", 1, 611, 611, 4, 1, 24),
        _case("hybrid 32 questions", "hybrid_4b", "bf16", "ask", 32, 200, 1500, 4, 1, 24),
        # the 27B shape: long prefixes, many candidates
        _case("27B 6 questions", "dense_27b", "bf16", "ask", 6, 1024, 4096, 10, 8, 40),
        # routed experts: a batch
        _case("experts 24 questions", "moe_35b_a3b", "f16", "ask", 24, 200, 1500, 4, 1, 24),
    ]


def draw(rng):
    def around(lo, hi):  # whole numbers spread over the logarithm of the range
        return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    kind = rng.choice(["1.5B", "1.5B", "1.5B", "1.5B kept", "1.5B kept", "trace", "int4", "hybrid", "hybrid", "27B",
                       "27B", "experts"])
    if kind == "1.5B":
        q = around(1, 112)
        if rng.random() < 0.3:
            return _case("", "dense_1p5b", "f16", "ask", min(q, 24), 300, around(301, 2000), rng.choice([2, 5]), 1,
                         rng.choice([1, 3]))
        p = around(150, 880)
        hi = rng.randint(p, 900)
        return _case("", "dense_1p5b", "f16", "ask", min(q, 60000 // hi), p, hi, 4, 1, around(2, 24))
    if kind == "1.5B kept":
        q, p = around(1, 128), around(150, 1990)
        return _case("", "dense_1p5b", "f16", "rescore", q, p, rng.randint(p, 2000), rng.choice([2, 4, 5]), 1,
                     around(1, 24), noalloc=rng.random() < 0.3 and q <= 16)
    if kind == "trace":
        p = around(150, 290)
        return _case("", "dense_1p5b", "f16", "trace", around(1, 8), p, rng.randint(p, 300), 4, 1, 24,
                     steps=around(4, 16))
    if kind == "int4":
        p = around(150, 880)
        return _case("", "dense_1p5b_q4", "f16", "ask", around(1, 32), p, rng.randint(p, 900), 4, 1, around(2, 24))
    if kind == "hybrid":
        p = around(200, 1480)
        return _case("", "hybrid_4b", "bf16", "ask", around(1, 32), p, rng.randint(p, 1500), 4, 1, around(2, 24))
    if kind == "27B":
        p = around(1024, 4000)
        return _case("", "dense_27b", "bf16", "ask", around(1, 6), p, rng.randint(p, 4096), 10, 8, around(9, 40))
    p = around(200, 1480)
    return _case("", "moe_35b_a3b", "f16", "ask", around(1, 24), p, rng.randint(p, 1500), 4, 1, around(2, 24))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _spread(lo, hi, n, phase):
    """n whole numbers spread over [lo, hi] (golden-ratio steps)."""
    return [lo + int((hi - lo + 1) * ((phase + i * 0.6180339887498949) % 1.0)) for i in range(n)]


def _lengths(c):
    plen = _spread(c["p_lo"], c["p_hi"], c["q"], 0.37)
    mlen = _spread(c["m_lo"], c["m_hi"], c["q"] * c["k"], 0.71)
    return plen, mlen


def _spec(model):
    s = dict(jet_synth.MODEL_SPECS[model])
    s["n_layers"] = LAYERS[model]
    return jet_synth.full_spec(s)


def _model_path(model):
    path = os.path.join(jet_synth.model_cache_dir(), f"{model}_first{LAYERS[model]}_s{jet_synth.MASTER_SEED}.jetm")
    if not os.path.exists(path):
        jet_synth.write_model(path, _spec(model))
    return path


_loaded = {}


def _model(c):
    key = (c["model"], c["mode"])
    if key not in _loaded:
        _loaded[key] = J.jet_model_load(_model_path(c["model"]), dtype=MODES[c["mode"]])
    return _loaded[key]


class _Prefix:
    """A retained prefix, freed with its owner."""

    def __init__(self, model, offsets, tokens):
        self.h = J.jet_prefill_prefix(model, offsets, tokens)

    def __del__(self):
        J.jet_prefix_free(self.h)


def _tokens(c, seed):
    V = jet_synth.MODEL_SPECS[c["model"]]["vocab"]
    plen, mlen = _lengths(c)
    g = np.random.Generator(np.random.Philox(key=[seed, 1]))
    pre = jet_synth.zipf_ids(g, sum(plen), V)
    cand = g.integers(0, V, size=sum(mlen)).astype(np.int32)
    po = np.concatenate([[0], np.cumsum(plen)]).astype(np.int64)
    qo = np.arange(c["q"] + 1, dtype=np.int64) * c["k"]
    co = np.concatenate([[0], np.cumsum(mlen)]).astype(np.int64)
    return po, pre, qo, co, cand


def prepare(case, seed):
    c = dict(case)
    po, pre, qo, co, cand = _tokens(c, seed)
    s = dict(c=c, seed=seed, m=_model(c), po=po, pre=pre, qo=qo, co=co, cand=cand)
    if c["q"] > 1:  # a batch keeps its ids and results on the GPU, a single request on the host
        s["pre"], s["cand"] = torch.from_numpy(pre).cuda(), torch.from_numpy(cand).cuda()
    if c["do"] == "rescore":
        s["kept"] = _Prefix(s["m"], po, s["pre"])
    return s


def _score(s, prefix):
    n, nt = len(s["co"]) - 1, int(s["co"][-1])
    if s["c"]["q"] > 1:
        tok, tot = torch.empty(nt, dtype=torch.float32, device="cuda"), torch.empty(n, dtype=torch.float32, device="cuda")
    else:
        tok, tot = np.empty(nt, np.float32), np.empty(n, np.float32)
    score = J.jet_score_candidates_noalloc if s["c"]["noalloc"] else J.jet_score_candidates
    tok, tot = score(s["m"], prefix.h, s["qo"], s["co"], s["cand"], tok, tot)
    return {"token_logprob": tok, "candidate_sum": tot}


def run(s):
    do = s["c"]["do"]
    if do == "rescore":
        return _score(s, s["kept"])
    p = _Prefix(s["m"], s["po"], s["pre"])
    out = {}
    if do == "trace":
        out["trace"] = J.jet_generate_trace(s["m"], p.h, s["c"]["q"], s["c"]["steps"], 1.0, s["seed"])
    out.update(_score(s, p))
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _layer_sizes(s, lt):
    """(weights every row uses before the mixer, after it, FFN weights per row, FFN weights stored)."""
    d = s["d_model"]
    if lt == "attn":
        hq, hkv = s["n_heads"] * s["head_dim"], s["n_kv_heads"] * s["head_dim"]
        pre, post = d * (hq + 2 * hkv), d * hq
    else:
        H, dk, dv = s["gdn_heads"], s["gdn_dk"], s["gdn_dv"]
        pre, post = d * (2 * H * dk + 2 * H * dv + 2 * H), d * H * dv
    if s["n_experts"]:
        shared = 3 * d * s["shared_ffn"] + d * (s["n_experts"] + 1)
        one = 3 * d * s["moe_ffn"]
        return pre, post, shared + s["top_k"] * one, (shared, one)
    return pre, post, 3 * d * s["ffn"], (3 * d * s["ffn"], 0)


def work(case):
    c, s = dict(case), _spec(case["model"])
    plen, mlen = _lengths(c)
    T, R, NT = sum(plen), sum(mlen) - len(mlen), sum(mlen)
    d, V, hd = s["d_model"], s["vocab"], s["head_dim"]
    planes = 2 if c["mode"] == "bf16" else 1
    wbytes = 0.5 + 1 / 32 if s["dtype"] == "q4" else 2.0
    flops = weights = kv = state = 0.0
    bodies = [sum(mlen[q * c["k"]:(q + 1) * c["k"]]) - c["k"] for q in range(c["q"])]
    own = sum((m - 1) * m / 2 for m in mlen)
    last = len(s["layer_types"]) - 1
    new = c["q"] * c["steps"]  # traced tokens
    for i, lt in enumerate(s["layer_types"]):
        pre, post, ffn, (always, one) = _layer_sizes(s, lt)
        weights += pre + post + always + one * min(s["n_experts"], (T + R) * s["top_k"])
        rows_pre, rows = (T + R, T + R) if c["do"] != "rescore" else (R, R)
        if i == last and lt == "attn" and c["do"] != "rescore":
            rows = R + c["q"]
        flops += 2.0 * ((rows_pre + new) * pre + (rows + new) * (post + ffn))
        if lt == "attn":
            pairs = sum(b * (p + c["steps"]) for b, p in zip(bodies, plen)) + own
            if c["do"] != "rescore":
                pairs += sum(p * (p + 1) / 2 if i != last else p for p in plen)
            pairs += sum(c["steps"] * (p + c["steps"] / 2) for p in plen)
            flops += 4.0 * pairs * s["n_heads"] * hd
            kv += T * 2 * s["n_kv_heads"] * hd * 2 * planes
        else:
            H, dk, dv = s["gdn_heads"], s["gdn_dk"], s["gdn_dv"]
            flops += (rows_pre + new) * H * 7.0 * dk * dv
            state += c["q"] * H * dk * dv * 4
    flops += 2.0 * V * d * (NT + new)
    head = V * d * 2.0
    nbytes = weights * wbytes + head + (T + R) * d * 2.0 + NT * 8.0
    if c["do"] == "rescore":  # the retained prefix is read; one-token candidates need its last rows alone
        weights = weights if R else 0.0
        nbytes = weights * wbytes + head + (kv + state if R else 0.0) + (R + c["q"]) * d * 2.0 + NT * 8.0
    nbytes += c["steps"] * (weights * wbytes + head)  # every decode step reads the weights again
    return {"bytes": nbytes, "flops": flops}


# Four times the error of the candidates' log-probabilities against exact()
# (1.3e-4 in the fp16 mode, 1.9e-6 in the pair mode). With routed experts a
# rounding difference swaps experts of nearly equal logit, a finite step each.
TOLERANCE = {("dense_1p5b", "f16"): 5e-4, ("dense_1p5b_q4", "f16"): 4e-4, ("hybrid_4b", "bf16"): 8e-6,
             ("dense_27b", "bf16"): 8e-6, ("moe_35b_a3b", "f16"): 1.6e-2}


def tolerance(case):
    t = {"rel": TOLERANCE[case["model"], case["mode"]]}
    if case["do"] == "trace":
        t["differ"] = 0.01
    return t


# ---------------------------------------------------------------------------
# the same in 64 bits, in plain torch
# ---------------------------------------------------------------------------

class _File:
    """The model file's tensors as float64 on the GPU."""

    def __init__(self, path):
        self.path = path
        with open(path, "rb") as f:
            self.h = json.loads(f.read(struct.unpack("<Q", f.read(16)[8:])[0]))
        self.t = {t["name"]: t for t in self.h["tensors"]}

    def w(self, name):
        t = self.t[name]
        n, shape = int(np.prod(t["shape"])), t["shape"]
        raw = torch.from_numpy(np.fromfile(self.path, np.uint8, t["nbytes"], offset=t["offset"])).cuda()
        if t["dtype"] == "f32":
            return raw.view(torch.float32).double().reshape(shape)
        if t["dtype"] == "bf16":
            return raw.view(torch.bfloat16).double().reshape(shape)
        b = raw[: n // 2].to(torch.int16)  # int4, two per byte, low nibble first
        q = torch.stack([b & 15, b >> 4], 1).reshape(-1)
        q = torch.where(q > 7, q - 16, q).double().reshape(-1, 32)
        return (q * torch.exp2(raw[n // 2:].view(torch.int8).double())[:, None]).reshape(shape)


def _norm(x, g, eps):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + eps) * g


def _silu(x):
    return x * torch.sigmoid(x)


def _attn64(s, W, a, pos, spans, bodies):
    hq, hkv, hd = s["n_heads"], s["n_kv_heads"], s["head_dim"]
    q, k, v = ((a @ W(n).T).reshape(len(a), -1, hd) for n in ("wq", "wk", "wv"))
    inv = s["rope_theta"] ** (-torch.arange(hd // 2, dtype=torch.float64, device="cuda") * 2 / hd)
    ang = (pos.double()[:, None] * inv)[:, None, :]

    def rot(x):
        x1, x2 = x[..., : hd // 2], x[..., hd // 2:]
        return torch.cat([x1 * ang.cos() - x2 * ang.sin(), x2 * ang.cos() + x1 * ang.sin()], -1)

    q, k = rot(q), rot(k)
    out = torch.empty_like(q)
    for (p0, p1), (b0, b1, cand) in zip(spans, bodies):
        rows = torch.cat([torch.arange(p0, p1, device="cuda"), torch.arange(b0, b1, device="cuda")])
        who = torch.cat([torch.full((p1 - p0,), -1, device="cuda"), cand])
        at = pos[rows]
        sees = (at[None, :] <= at[:, None]) & ((who[None, :] == -1) | (who[None, :] == who[:, None]))
        for j in range(hkv):
            kj, vj = k[rows, j], v[rows, j]
            for h in range(j * (hq // hkv), (j + 1) * (hq // hkv)):
                z = (q[rows, h] @ kj.T.contiguous()) / math.sqrt(hd)
                out[rows, h] = torch.softmax(z.masked_fill_(~sees, -math.inf), -1) @ vj
    return out.reshape(len(a), -1) @ W("wo").T


def _delta64(s, W, a, spans, cands):
    """Gated delta rule over the questions, then over each candidate from its question's state."""
    H, dk, dv, kc = s["gdn_heads"], s["gdn_dk"], s["gdn_dv"], s["conv_kernel"]
    x = torch.cat([a @ W(n).T for n in ("gdn_wq", "gdn_wk", "gdn_wv")], 1)
    beta = torch.sigmoid(a @ W("gdn_wb").T)
    alpha = torch.exp(-torch.exp(W("gdn_A_log")) * torch.nn.functional.softplus(a @ W("gdn_wa").T + W("gdn_dt_bias")))
    w, zero = W("gdn_conv"), torch.zeros(kc - 1, x.shape[1], dtype=torch.float64, device="cuda")
    xc = torch.empty_like(x)
    for r0, r1, q in [(p0, p1, None) for p0, p1 in spans] + cands:
        full = torch.cat([zero if q is None else torch.cat([zero, x[spans[q][0]:spans[q][1]]])[1 - kc:], x[r0:r1]])
        xc[r0:r1] = sum(full[j:j + r1 - r0] * w[:, j] for j in range(kc))
    xc = _silu(xc)
    unit = lambda t: t * torch.rsqrt((t * t).sum(-1, keepdim=True) + 1e-6)  # noqa: E731
    q = unit(xc[:, : H * dk].reshape(-1, H, dk)) / math.sqrt(dk)
    k, v = unit(xc[:, H * dk: 2 * H * dk].reshape(-1, H, dk)), xc[:, 2 * H * dk:].reshape(-1, H, dv)
    o = torch.empty_like(v)

    def steps(start, length, S):
        order = sorted(range(len(start)), key=lambda i: -length[i])
        S = S[order]
        first = torch.tensor([start[i] for i in order], device="cuda")
        for t in range(max(length, default=0)):
            n = sum(1 for i in order if length[i] > t)
            r, A = first[:n] + t, S[:n]
            A *= alpha[r][..., None, None]
            A += (beta[r][..., None] * (v[r] - (A * k[r][:, :, None]).sum(-1)))[..., None] * k[r][:, :, None]
            o[r] = (A * q[r][:, :, None]).sum(-1)
        back = torch.empty_like(S)
        back[order] = S
        return back

    S = steps([p0 for p0, _ in spans], [p1 - p0 for p0, p1 in spans],
              torch.zeros(len(spans), H, dv, dk, dtype=torch.float64, device="cuda"))
    if cands:
        steps([c[0] for c in cands], [c[1] - c[0] for c in cands], S[[c[2] for c in cands]])
    y = _norm(o, W("gdn_norm"), s["rms_eps"]).reshape(len(a), -1) * _silu(a @ W("gdn_wz").T)
    return y @ W("gdn_wo").T


def _ffn64(s, W, a):
    glu = lambda t, g, u, d: (_silu(t @ g.T) * (t @ u.T)) @ d.T  # noqa: E731
    if not s["n_experts"]:
        g, u, d = W("w_gate"), W("w_up"), W("w_down")
        return torch.cat([glu(t, g, u, d) for t in a.split(16384)])
    z, sel = torch.topk(a @ W("moe_router").T, s["top_k"])
    wts = torch.softmax(z, -1)
    out = torch.sigmoid(a @ W("shared_router").T) * glu(a, W("shared_gate"), W("shared_up"), W("shared_down"))
    G, U, D = W("moe_gate"), W("moe_up"), W("moe_down")
    for e in range(s["n_experts"]):
        r, j = torch.nonzero(sel == e, as_tuple=True)
        if len(r):
            out[r] += wts[r, j][:, None] * glu(a[r], G[e], U[e], D[e])
    return out


def exact(case, seed):
    """token_logprob and candidate_sum in float64; a trace's tokens are discrete choices, so a traced case has none."""
    c, s = dict(case), _spec(case["model"])
    if c["do"] == "trace" or work(c)["flops"] > 3e14:
        return None
    po, pre, qo, co, cand = _tokens(c, seed)
    f = _File(_model_path(c["model"]))
    T = int(po[-1])
    spans = [(int(po[q]), int(po[q + 1])) for q in range(c["q"])]
    ids, pos = [torch.from_numpy(pre).long()], [torch.arange(b - a) for a, b in spans]
    bodies, cands, last, r = [], [], [], T  # body rows follow the prefix rows
    for q in range(c["q"]):
        r_q, who = r, []
        for j in range(int(qo[q]), int(qo[q + 1])):
            y = cand[co[j]:co[j + 1]]
            n = len(y) - 1
            ids.append(torch.from_numpy(y[:n]).long())
            pos.append(torch.arange(n) + (spans[q][1] - spans[q][0]))
            last += [spans[q][1] - 1] + list(range(r, r + n))  # the row that predicts each token
            who += [j] * n
            if n:
                cands.append((r, r + n, q))
            r += n
        bodies.append((r_q, r, torch.tensor(who, dtype=torch.long, device="cuda")))
    ids, pos = torch.cat(ids).cuda(), torch.cat(pos).cuda()
    x = f.w("tok_embed")[ids]
    for i, lt in enumerate(s["layer_types"]):
        def W(name, i=i):
            return f.w(f"blk.{i}.{name}")
        a = _norm(x, W("attn_norm"), s["rms_eps"])
        x = x + (_attn64(s, W, a, pos, spans, bodies) if lt == "attn" else _delta64(s, W, a, spans, cands))
        x = x + _ffn64(s, W, _norm(x, W("ffn_norm"), s["rms_eps"]))
    x = _norm(x[torch.tensor(last, device="cuda")], f.w("final_norm"), s["rms_eps"])
    head, y = f.w("lm_head"), torch.from_numpy(cand).long().cuda()
    tok = torch.cat([torch.log_softmax(t @ head.T, -1).gather(1, yt[:, None])[:, 0]
                     for t, yt in zip(x.split(2048), y.split(2048))])
    tot = torch.stack([tok[int(co[j]):int(co[j + 1])].sum() for j in range(len(co) - 1)])
    return {"token_logprob": tok, "candidate_sum": tot}
