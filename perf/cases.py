"""The work that is timed when a kernel changes: single layers through the mc_op_* entry points,
and whole session calls, over the sizes that the workloads, the tests and bench.py use.

A case is a plain dict.  Its "kind" names the path:

  attn_decode   one layer-step of shared-prefix decode attention
  attn_prefill  causal attention of many rows: a context that grows, or candidates that are scored
  mlp           norm, gate/up with SwiGLU, down projection into the residual, norm
  head          LM head and sampling of the next tokens
  rollout       a session that samples and decodes a stretch of tokens from a shared prefix
  depth         a session that goes through one depth of the search: context prefilled, critique
                appended, candidates scored

The model widths are those of synth.WORKLOADS.  Sessions run a two-layer model of full width with a
32000-token vocabulary (tiny: the whole model as it stands).
"""
import math

import numpy as np
import torch

from paper_2601_05475_amd import binding, synth

DEV = "cuda:0"
PG = 64                      # keys per KV page of every bf16 workload
EPS = 1e-6
F64 = torch.float64
# d_model, query heads, KV heads, head_dim, d_ffn, vocabulary, rotary base
WIDTHS = {
    "tiny": (256, 4, 2, 64, 688, 4096, 1.0e4),
    "1b": (2048, 32, 8, 64, 8192, 32000, 1.0e4),
    "8b": (4096, 32, 8, 128, 14336, 128256, 5.0e5),
    "32b": (5120, 40, 8, 128, 27648, 152064, 1.0e6),
}


def listed():
    return [
        # the fp32 workload as it stands: 4 candidates, 16 tokens, the host reads every token to see
        # whether a candidate has ended; launches and latency
        dict(name="rollout tiny fp32", kind="rollout", width="tiny", cands=4, prefix=128, steps=16, temperature=0.8, top_k=50),
        # eight candidates (the fan-out of one search state) on a 1B width: the small decode step
        dict(name="rollout 1b 8 cands", kind="rollout", width="1b", cands=8, prefix=2048, steps=16, temperature=0.7, top_k=50),
        # few candidates, an odd short context, candidates that differ in length
        dict(name="attn decode small ragged", kind="attn_decode", width="1b", cands=8, prefix=777, suffix=37, ragged=True),
        # the headline decode workload at its mean suffix length
        dict(name="attn decode 8b", kind="attn_decode", width="8b", cands=32, prefix=4096, suffix=257, ragged=False),
        # long-context search
        dict(name="attn decode 32b", kind="attn_decode", width="32b", cands=64, prefix=16384, suffix=512, ragged=False),
        # a critique of a few hundred tokens appended to the context
        dict(name="attn extend 8b 300", kind="attn_prefill", width="8b", seqs=1, rows=300, prefix=4096, ragged=False),
        # eight of the candidates of the reranking workload
        dict(name="attn rerank 8b 8x1024", kind="attn_prefill", width="8b", seqs=8, rows=1024, prefix=4096, ragged=False),
        # the feed-forward block of a decode step, of an appended critique, of a reranking chunk
        dict(name="mlp 8b 32 rows", kind="mlp", width="8b", rows=32),
        dict(name="mlp 8b 300 rows", kind="mlp", width="8b", rows=300),
        dict(name="mlp 8b 8192 rows", kind="mlp", width="8b", rows=8192),
        # logits and next tokens of the headline decode workload
        dict(name="head 8b 32 rows", kind="head", width="8b", rows=32, temperature=0.7, top_k=50),
        # one depth of the search with k = 8 candidates of different lengths
        dict(name="depth 8b 8 cands", kind="depth", width="8b", cands=8, prefix=1000, critique=211, suffix=150),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["attn_decode", "attn_decode", "attn_prefill", "attn_prefill", "mlp", "mlp", "mlp", "head", "rollout", "depth"])
    if kind == "attn_decode":
        return dict(kind=kind, width=rng.choice(["1b", "8b", "32b"]), cands=_log_int(rng, 1, 64), prefix=_log_int(rng, 64, 16384),
                    suffix=_log_int(rng, 1, 1024), ragged=rng.random() < 0.4)
    if kind == "attn_prefill":
        # scored candidates or (seqs = 1) mostly a context that grows
        return dict(kind=kind, width=rng.choice(["1b", "8b", "32b"]), seqs=rng.choice([1, 1, 2, 5, 8]), rows=_log_int(rng, 65, 1024),
                    prefix=_log_int(rng, 256, 4096), ragged=rng.random() < 0.5)
    if kind == "mlp":
        width = rng.choice(["1b", "8b", "32b"])
        return dict(kind=kind, width=width, rows=_log_int(rng, 1, {"1b": 8192, "8b": 4096, "32b": 2048}[width]))
    if kind == "head":
        return dict(kind=kind, width=rng.choice(["1b", "8b", "32b"]), rows=_log_int(rng, 1, 64), temperature=rng.choice([0.6, 0.7, 0.8]),
                    top_k=rng.choice([1, 20, 50, 64, 200]))
    if kind == "rollout":
        return dict(kind=kind, width=rng.choice(["tiny", "1b", "8b"]), cands=_log_int(rng, 1, 32), prefix=_log_int(rng, 64, 512), steps=rng.randint(3, 12),
                    temperature=0.7, top_k=50)
    return dict(kind=kind, width=rng.choice(["1b", "8b"]), cands=_log_int(rng, 2, 16), prefix=_log_int(rng, 128, 2048),
                critique=_log_int(rng, 16, 500), suffix=_log_int(rng, 16, 400))


# ---- inputs, from the seed alone ----------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _normal(g, *shape, std=1.0, mean=0.0, dtype=torch.bfloat16):
    out = torch.empty(shape, dtype=dtype, device=DEV)
    out.normal_(mean, std, generator=g)
    return out


def _lengths(g, n, most, ragged):
    """n lengths in [max(1, most / 2), most], one of them `most`; all of them `most` if not ragged."""
    if not ragged:
        return [most] * n
    lens = torch.randint(max(1, most // 2), most + 1, (n,), generator=g, device=DEV).tolist()
    lens[n // 2] = most
    return lens


def _tokens(g, *shape, vocab):
    return torch.randint(0, vocab, shape, generator=g, device=DEV, dtype=torch.int32)


def _attn_decode_inputs(c, seed):
    g = _gen(seed)
    _, Hq, Hkv, hd, _, _, _ = WIDTHS[c["width"]]
    B, P, t = c["cands"], c["prefix"], c["suffix"]
    pp, sp = -(-P // PG), -(-t // PG)
    return dict(q=_normal(g, B, Hq, hd), kp=_normal(g, pp, Hkv, PG, hd), vp=_normal(g, pp, Hkv, PG, hd),
                ks=_normal(g, B * sp, Hkv, PG, hd), vs=_normal(g, B * sp, Hkv, PG, hd),
                table=torch.randperm(B * sp, generator=g, device=DEV).to(torch.int32).reshape(B, sp),
                lens=_lengths(g, B, t, c["ragged"]))


def _attn_prefill_inputs(c, seed):
    """One sequence: the new rows' keys lie in the prefix pages, as when a context grows.  Several:
    each has suffix pages of its own, as candidates that are scored."""
    g = _gen(seed)
    _, Hq, Hkv, hd, _, _, _ = WIDTHS[c["width"]]
    S, L, P = c["seqs"], c["rows"], c["prefix"]
    lens = _lengths(g, S, L, c["ragged"])
    pp, sp = -(-(P + (L if S == 1 else 0)) // PG), -(-L // PG)
    d = dict(q=_normal(g, sum(lens), Hq, hd), kp=_normal(g, pp, Hkv, PG, hd), vp=_normal(g, pp, Hkv, PG, hd), lens=lens)
    if S > 1:
        d.update(ks=_normal(g, S * sp, Hkv, PG, hd), vs=_normal(g, S * sp, Hkv, PG, hd),
                 table=torch.randperm(S * sp, generator=g, device=DEV).to(torch.int32).reshape(S, sp))
    return d


def _mlp_inputs(c, seed):
    g = _gen(seed)
    d, _, _, _, F, _, _ = WIDTHS[c["width"]]
    return dict(x=_normal(g, c["rows"], d, dtype=torch.float32), g1=_normal(g, d, mean=1.0, std=0.02), g2=_normal(g, d, mean=1.0, std=0.02),
                wg=_normal(g, F, d, std=0.02), wu=_normal(g, F, d, std=0.02), wd=_normal(g, d, F, std=0.02))


def _head_inputs(c, seed):
    g = _gen(seed)
    d, _, _, _, _, V, _ = WIDTHS[c["width"]]
    u = torch.empty(c["rows"], dtype=torch.float32, device=DEV)
    u.uniform_(0.0, 0.999, generator=g)
    return dict(a=_normal(g, c["rows"], d), w=_normal(g, V, d, std=0.02), u=u)


def _shape(c):
    d, Hq, Hkv, hd, F, V, base = WIDTHS[c["width"]]
    tiny = c["width"] == "tiny"
    return synth.Shape("two-layer " + c["width"], 2, d, Hq, Hkv, hd, F, V if tiny else 32000, base, "f32" if tiny else "bf16")


_LAYER = ("attn_norm", "wq", "wk", "wv", "wo", "ffn_norm", "w_gate", "w_up", "w_down")


def _weights(s, g):
    dt = torch.float32 if s.dtype == "f32" else torch.bfloat16
    d, q, kv, F = s.d_model, s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim, s.d_ffn
    shapes = dict(attn_norm=(d,), wq=(q, d), wk=(kv, d), wv=(kv, d), wo=(d, q), ffn_norm=(d,), w_gate=(F, d), w_up=(F, d), w_down=(d, F))
    make = lambda name, shape: _normal(g, *shape, std=0.02, mean=1.0 if name.endswith("norm") else 0.0, dtype=dt)  # noqa: E731
    return dict(embed=make("embed", (s.vocab, d)), final_norm=make("final_norm", (d,)), lm_head=make("lm_head", (s.vocab, d)),
                layers=[{n: make(n, shapes[n]) for n in _LAYER} for _ in range(s.n_layers)])


def _session_inputs(c, seed):
    g = _gen(seed)
    s = _shape(c)
    d = dict(shape=s, weights=_weights(s, g), prefix=_tokens(g, c["prefix"], vocab=s.vocab))
    if c["kind"] == "rollout":
        d["suffix"] = _tokens(g, c["cands"], c["steps"], vocab=s.vocab)
        u = torch.empty((c["steps"] + 1, c["cands"]), dtype=torch.float32, device=DEV)
        u.uniform_(0.0, 0.999, generator=g)
        d["u"] = u
    else:
        d["critique"] = _tokens(g, c["critique"], vocab=s.vocab)
        d["suffix"] = _tokens(g, c["cands"], c["suffix"], vocab=s.vocab)
        d["lens"] = _lengths(g, c["cands"], c["suffix"], True)
        d["reward"] = torch.randperm(s.vocab, generator=g, device=DEV)[:8].to(torch.int32)
    return d


# ---- what a user's program has in hand ------------------------------------------------------
def _host_weights(w):
    def conv(t):
        return t.cpu().numpy() if t.dtype == torch.float32 else t.view(torch.int16).cpu().numpy().view(np.uint16)
    out = {k: conv(v) for k, v in w.items() if k != "layers"}
    out["layers"] = [{k: conv(v) for k, v in lw.items()} for lw in w["layers"]]
    return out


def prepare(case, seed):
    c = case
    if c["kind"] == "attn_decode":
        i = _attn_decode_inputs(c, seed)
        kp, vp = binding.kv_pages_pack(i["kp"], i["vp"])
        ks, vs = binding.kv_pages_pack(i["ks"], i["vs"])
        return dict(case=c, q=i["q"], kp=kp, vp=vp, ks=ks, vs=vs, table=i["table"],
                    row_len=torch.tensor(i["lens"], dtype=torch.int32, device=DEV) if c["ragged"] else None)
    if c["kind"] == "attn_prefill":
        i = _attn_prefill_inputs(c, seed)
        kp, vp = binding.kv_pages_pack(i["kp"], i["vp"])
        ks, vs = binding.kv_pages_pack(i["ks"], i["vs"]) if c["seqs"] > 1 else (None, None)
        items, row = [], 0
        for s, n in enumerate(i["lens"]):
            items += [[row + r, min(64, n - r), c["prefix"] + r, s if c["seqs"] > 1 else -1] for r in range(0, n, 64)]
            row += n
        return dict(case=c, q=i["q"], kp=kp, vp=vp, ks=ks, vs=vs, table=i.get("table"),
                    prefix_len=c["prefix"] + (i["lens"][0] if c["seqs"] == 1 else 0), items=torch.tensor(items, dtype=torch.int32, device=DEV))
    if c["kind"] == "mlp":
        i = _mlp_inputs(c, seed)
        return dict(case=c, x=i["x"], g1=i["g1"], g2=i["g2"], wg=binding.op_pack_tiled(i["wg"]), wu=binding.op_pack_tiled(i["wu"]),
                    wd=binding.op_pack_tiled(i["wd"]))
    if c["kind"] == "head":
        i = _head_inputs(c, seed)
        return dict(case=c, a=binding.op_pack_tiled(i["a"]), w=binding.op_pack_tiled(i["w"]), u=i["u"])
    i = _session_inputs(c, seed)
    model = binding.Model(i["shape"], _host_weights(i["weights"]), device=DEV)
    host = {k: v.cpu().numpy() for k, v in i.items() if isinstance(v, torch.Tensor)}
    if c["kind"] == "rollout":
        sess = binding.Session(model, max_prefix=c["prefix"], max_cands=c["cands"], max_suffix=c["steps"],
                               page_tokens=4 if c["width"] == "tiny" else PG)
        sess.prefill_shared(host["prefix"])
        return dict(case=c, model=model, sess=sess, suffix=[np.ascontiguousarray(host["suffix"][:, t]) for t in range(c["steps"])], u=host["u"])
    sess = binding.Session(model, max_prefix=c["prefix"] + c["critique"], max_cands=c["cands"], max_suffix=c["suffix"], page_tokens=PG)
    return dict(case=c, model=model, sess=sess, prefix=host["prefix"], critique=host["critique"], suffix=host["suffix"],
                lens=np.array(i["lens"], np.int32), reward=host["reward"], values=np.arange(8, dtype=np.float32))


# ---- one pass ---------------------------------------------------------------------------------
def run(state):
    s, c = state, state["case"]
    if c["kind"] == "attn_decode":
        return binding.op_attention_decode(s["q"], s["kp"], s["vp"], s["ks"], s["vs"], s["table"], c["prefix"], c["suffix"], PG,
                                           out_tiled=True, row_len=s["row_len"])
    if c["kind"] == "attn_prefill":
        return binding.op_attention_prefill(s["q"], s["items"], s["kp"], s["vp"], s["ks"], s["vs"], s["table"], s["prefix_len"], PG,
                                            out_tiled=True)
    if c["kind"] == "mlp":
        d, F, M = WIDTHS[c["width"]][0], WIDTHS[c["width"]][4], c["rows"]
        h = binding.op_add_rmsnorm(s["x"], None, s["g1"], EPS, tiled=True)
        act = binding.op_linear_swiglu(h, s["wg"], s["wu"], tiled_shape=(M, F, d))
        if M <= 64:           # few rows: partial sums that the next norm adds to the residual
            n = binding.op_linear_splits("bf16", M, d, F, True)
            part = binding.op_linear(act, s["wd"], n_splits=n, tiled_shape=(M, d, F))
        else:                 # many rows: the product adds to the residual itself
            part = None
            binding.op_linear_accumulate(act, s["wd"], s["x"], (M, d, F))
        h = binding.op_add_rmsnorm(s["x"], part, s["g2"], EPS, tiled=True)
        return dict(x=s["x"], h=h)
    if c["kind"] == "head":
        d, V, M = WIDTHS[c["width"]][0], WIDTHS[c["width"]][5], c["rows"]
        if M <= 32 and V >= 65536:
            logits, lists = binding.op_lm_head(s["a"], s["w"], (M, V, d))
            tokens = binding.op_sample_lists(logits, lists, c["temperature"], c["top_k"], s["u"])
        else:
            logits = binding.op_linear(s["a"], s["w"], tiled_shape=(M, V, d))[0]
            tokens = binding.op_sample(logits, c["temperature"], c["top_k"], s["u"])
        return dict(logits=logits, tokens=tokens)
    sess = s["sess"]
    if c["kind"] == "rollout":
        # The program reads every sampled token (the tiny workload's loop) or leaves them on the
        # device; the tokens that go on are given, so that two runs stay comparable.
        sess.reset_candidates()
        drawn = []
        for t in range(c["steps"]):
            tok = sess.sample(c["cands"], c["temperature"], c["top_k"], s["u"][t], want_tokens=c["width"] == "tiny")
            if tok is not None:
                drawn.append(tok)
            sess.decode_step(s["suffix"][t])
        drawn.append(sess.sample(c["cands"], c["temperature"], c["top_k"], s["u"][c["steps"]]))
        return dict(logits=sess.logits(c["cands"]), tokens=np.stack(drawn))
    sess.prefill_shared(s["prefix"])
    sess.extend_shared(s["critique"])
    lp, score, rank = sess.score_candidates(s["suffix"], s["lens"], s["reward"], s["values"])
    return dict(logprobs=lp, scores=score, rank=rank)


# ---- what a pass cannot do without --------------------------------------------------------------
def _model_work(s, rows, head_rows, kv_read, pairs):
    """bytes and flops of one pass of the two-layer model over `rows` new rows: weights once, keys
    and values of kv_read positions read and of `rows` written, `pairs` (row, key) pairs per head."""
    b = 4 if s.dtype == "f32" else 2
    q, kv = s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim
    per_layer = s.d_model * (2 * q + 2 * kv + 3 * s.d_ffn)
    by = s.n_layers * (per_layer * b + 2 * kv * (kv_read + rows) * b) + rows * s.d_model * b + head_rows * s.vocab * 4
    fl = s.n_layers * (2 * rows * per_layer + 4 * q * pairs)
    if head_rows:
        by, fl = by + s.vocab * s.d_model * b, fl + 2 * head_rows * s.vocab * s.d_model
    return by, fl


def work(case):
    c = case
    d, Hq, Hkv, hd, F, V, _ = WIDTHS[c["width"]]
    if c["kind"] == "attn_decode":
        B, P = c["cands"], c["prefix"]
        t = c["suffix"] * (0.75 if c["ragged"] else 1.0)     # the mean of the drawn lengths
        return dict(bytes=(P + B * t) * 2 * Hkv * hd * 2 + 2 * B * Hq * hd * 2, flops=4 * Hq * hd * B * (P + t))
    if c["kind"] == "attn_prefill":
        S, P = c["seqs"], c["prefix"]
        L = c["rows"] * (0.75 if c["ragged"] and S > 1 else 1.0)
        return dict(bytes=(P + S * L) * 2 * Hkv * hd * 2 + 2 * S * L * Hq * hd * 2, flops=4 * Hq * hd * S * L * (P + (L + 1) / 2))
    if c["kind"] == "mlp":
        M = c["rows"]
        return dict(bytes=3 * d * F * 2 + M * d * (4 + 4 + 2), flops=6 * M * d * F)
    if c["kind"] == "head":
        M = c["rows"]
        return dict(bytes=V * d * 2 + M * d * 2 + M * V * 4, flops=2 * M * V * d)
    s = _shape(c)
    by = fl = 0.0
    if c["kind"] == "rollout":
        B, P = c["cands"], c["prefix"]
        for t in range(1, c["steps"] + 1):
            x, y = _model_work(s, B, B, P + B * (t - 1), B * (P + t))
            by, fl = by + x, fl + y
        return dict(bytes=by, flops=fl)
    P, E, B = c["prefix"], c["critique"], c["cands"]
    L = c["suffix"] * 0.75
    for rows, seen, pairs, head in ((P, 0, P * (P + 1) / 2, 1), (E, P, E * (P + (E + 1) / 2), 1),
                                    (B * L, P + E, B * L * (P + E + (L + 1) / 2), B)):
        x, y = _model_work(s, rows, head, seen, pairs)
        by, fl = by + x, fl + y
    return dict(bytes=by, flops=fl)


def tolerance(case):
    c = case
    if c["kind"] in ("attn_decode", "attn_prefill"):
        return {"rel": 1e-2}           # bf16 results and probabilities
    if c["kind"] == "mlp":
        return {"rel": 1e-2}           # bf16 normalised rows and SwiGLU product
    if c["kind"] == "head":
        return {"rel": 3e-6, "differ": 0.1}
    if c["width"] == "tiny":
        return {"rel": 3e-6, "differ": 0.1}
    # two layers of bf16 activations: logits 7e-3 from the 64-bit ones, log-probabilities and scores
    # 1e-3 to 4e-3; sampled ids and ranks follow them
    return {"rel": 3e-2 if c["kind"] == "rollout" else 1.5e-2, "differ": 0.6}


# ---- the same in 64 bits, plain torch -----------------------------------------------------------
def _tiled(m):
    """[rows, K] in the tiled operand layout (flat; rows padded to a multiple of 32 with zeros)."""
    rows, K = m.shape
    rp = (rows + 31) // 32 * 32
    if rp != rows:
        m = torch.cat([m, torch.zeros((rp - rows, K), dtype=m.dtype, device=m.device)])
    return m.reshape(rp // 32, 32, K // 64, 2, 4, 8).permute(0, 2, 4, 3, 1, 5).reshape(-1)


def _heads(pages, n):
    """[pages, Hkv, PG, hd] -> [Hkv, n, hd] in 64 bits: the first n keys in order."""
    p, H, g, hd = pages.shape
    return pages.permute(1, 0, 2, 3).reshape(H, p * g, hd)[:, :n].to(F64)


def _attend(q, k, v, visible=None):
    """q [H, n, hd], k and v [H, m, hd], all 64 bits; visible [n, m] or None."""
    s = torch.matmul(q, k.transpose(1, 2).contiguous()) / math.sqrt(q.shape[-1])
    if visible is not None:
        s.masked_fill_(~visible, float("-inf"))
    return torch.matmul(torch.softmax(s, -1), v)


def _norm(x, gain, eps=EPS):
    return x * gain.to(F64) / torch.sqrt((x * x).mean(-1, keepdim=True) + eps)


def _exact_attn_decode(c, seed):
    i = _attn_decode_inputs(c, seed)
    B, Hq, hd = i["q"].shape
    Hkv = WIDTHS[c["width"]][2]
    G = Hq // Hkv
    kp, vp = _heads(i["kp"], c["prefix"]), _heads(i["vp"], c["prefix"])
    out = torch.empty((B, Hq, hd), dtype=F64, device=DEV)
    for b in range(B):
        t = i["lens"][b]
        pages = i["table"][b].long()
        k = torch.cat([kp, _heads(i["ks"][pages], t)], 1)
        v = torch.cat([vp, _heads(i["vs"][pages], t)], 1)
        out[b] = _attend(i["q"][b].to(F64).reshape(Hkv, G, hd), k, v).reshape(Hq, hd)
    return _tiled(out.reshape(B, Hq * hd))


def _causal(n, m, device):
    """[n, m]: row r of the last n of m positions sees keys 0 .. m - n + r."""
    return torch.arange(m, device=device)[None, :] <= torch.arange(n, device=device)[:, None] + (m - n)


def _gqa(q, k, v, G):
    """q [n, Hq, hd] at the last n positions of k, v [Hkv, m, hd]; causal.  [n, Hq, hd]."""
    n, Hq, hd = q.shape
    Hkv, m = k.shape[0], k.shape[1]
    vis = _causal(n, m, q.device)
    out = torch.empty((n, Hq, hd), dtype=F64, device=q.device)
    for h in range(Hkv):
        for a in range(h * G, (h + 1) * G):
            out[:, a] = _attend(q[:, a].to(F64)[None], k[h:h + 1], v[h:h + 1], vis)[0]
    return out


def _exact_attn_prefill(c, seed):
    i = _attn_prefill_inputs(c, seed)
    Hq, Hkv = WIDTHS[c["width"]][1:3]
    outs, row = [], 0
    for s, n in enumerate(i["lens"]):
        if c["seqs"] == 1:
            k, v = _heads(i["kp"], c["prefix"] + n), _heads(i["vp"], c["prefix"] + n)
        else:
            pages = i["table"][s].long()
            k = torch.cat([_heads(i["kp"], c["prefix"]), _heads(i["ks"][pages], n)], 1)
            v = torch.cat([_heads(i["vp"], c["prefix"]), _heads(i["vs"][pages], n)], 1)
        outs.append(_gqa(i["q"][row:row + n], k, v, Hq // Hkv))
        row += n
    out = torch.cat(outs)
    return _tiled(out.reshape(out.shape[0], -1))


def _swiglu(h, wg, wu):
    g = h @ wg.to(F64).T
    return g / (1 + torch.exp(-g)) * (h @ wu.to(F64).T)


def _exact_mlp(c, seed):
    i = _mlp_inputs(c, seed)
    x = i["x"].to(F64)
    x = x + _swiglu(_norm(x, i["g1"]), i["wg"], i["wu"]) @ i["wd"].to(F64).T
    return dict(x=x, h=_tiled(_norm(x, i["g2"])))


class _Model64:
    """The decoder in 64 bits, one sequence at a time, with the keys and values of what it has read."""

    def __init__(self, s, w):
        self.s, self.w = s, w

    def run(self, tokens, past=None):
        """tokens: [n] after `past` (list of (k, v) per layer, or None).  Hidden rows [n, d] and the new past."""
        s, w = self.s, self.w
        half = s.head_dim // 2
        n, G = tokens.shape[0], s.n_q_heads // s.n_kv_heads
        start = past[0][0].shape[1] if past else 0
        pos = torch.arange(start, start + n, device=DEV, dtype=F64)
        ang = pos[:, None] * (float(s.rope_base) ** (-2.0 * torch.arange(half, device=DEV, dtype=F64) / s.head_dim))[None, :]
        cos, sin = torch.cos(ang)[:, None], torch.sin(ang)[:, None]

        def rope(t):
            lo, hi = t[..., :half], t[..., half:]
            return torch.cat([lo * cos - hi * sin, hi * cos + lo * sin], -1)

        x, new = w["embed"][tokens.long()].to(F64), []
        for l, lw in enumerate(w["layers"]):
            h = _norm(x, lw["attn_norm"], s.rms_eps)
            q = rope((h @ lw["wq"].to(F64).T).reshape(n, s.n_q_heads, s.head_dim))
            k = rope((h @ lw["wk"].to(F64).T).reshape(n, s.n_kv_heads, s.head_dim)).transpose(0, 1)
            v = (h @ lw["wv"].to(F64).T).reshape(n, s.n_kv_heads, s.head_dim).transpose(0, 1)
            if past:
                k, v = torch.cat([past[l][0], k], 1), torch.cat([past[l][1], v], 1)
            new.append((k, v))
            x = x + _gqa(q, k, v, G).reshape(n, -1) @ lw["wo"].to(F64).T
            x = x + _swiglu(_norm(x, lw["ffn_norm"], s.rms_eps), lw["w_gate"], lw["w_up"]) @ lw["w_down"].to(F64).T
        return x, new

    def logits(self, x):
        return _norm(x, self.w["final_norm"], self.s.rms_eps) @ self.w["lm_head"].to(F64).T


def _exact_session(c, seed):
    i = _session_inputs(c, seed)
    m = _Model64(i["shape"], i["weights"])
    _, past = m.run(i["prefix"])
    if c["kind"] == "rollout":
        rows = [m.run(i["suffix"][b], past)[0][-1] for b in range(c["cands"])]
        return dict(logits=m.logits(torch.stack(rows)), tokens=None)
    _, past = m.run(i["critique"], past)
    rows = torch.stack([m.run(i["suffix"][b][:n], past)[0][-1] for b, n in enumerate(i["lens"])])
    lp = torch.log_softmax(m.logits(rows), -1)[:, i["reward"].long()]
    return dict(logprobs=lp, scores=torch.softmax(lp, -1) @ torch.arange(8, dtype=F64, device=DEV), rank=None)


def exact(case, seed):
    c = case
    if c["kind"] == "attn_decode":
        return _exact_attn_decode(c, seed)
    if c["kind"] == "attn_prefill":
        return _exact_attn_prefill(c, seed)
    if c["kind"] == "mlp":
        return _exact_mlp(c, seed)
    if c["kind"] == "head":
        i = _head_inputs(c, seed)
        return dict(logits=i["a"].to(F64) @ i["w"].to(F64).T, tokens=None)
    return _exact_session(c, seed)
