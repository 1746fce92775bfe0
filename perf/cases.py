"""What the library is timed on: the calls a rollout or head-training program makes, through
paper_2609_16648_amd.gm, over the sizes such programs use.

Seven kinds of pass, named by a case's "op":
  step         a whole speculative step of a small float32 decoder (verify, accept, commit, draft)
  verify       the verify forward of one decoder layer and the LM head
  attention    the verify attention of one layer
  accept       the accept rule and the index commit, at the options a rollout runs it with
  draft        the MTP head's extend and draft chain
  reconstruct  the batched re-run of recorded drafting cycles (head training)
  dca          the draft-acceptance loss and its gradient over recorded cycles (head training)

Inputs are made on the GPU from the seed alone.  `exact` computes the same outputs in float64
with plain torch from the same inputs, on the logical (row-major) weights and unpacked KV pages.
"""
from __future__ import annotations

import ctypes
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2609_16648_amd import gm

# One layer of each backbone shape with its LM head (a deeper model repeats the layer), and two
# small float32 decoders.
MODELS = {
    "qwen3_4b": dict(n_layers=1, hidden=2560, n_heads=32, n_kv_heads=8, head_dim=128, ffn=9728, vocab=151936,
                     dtype="bf16"),
    "mimo_7b": dict(n_layers=1, hidden=4096, n_heads=32, n_kv_heads=8, head_dim=128, ffn=11008, vocab=151680,
                    dtype="bf16"),
    "tiny": dict(n_layers=2, hidden=256, n_heads=4, n_kv_heads=4, head_dim=64, ffn=1024, vocab=1024, dtype="f32"),
    "small": dict(n_layers=2, hidden=512, n_heads=8, n_kv_heads=2, head_dim=64, ffn=1472, vocab=5003, dtype="f32"),
}


def _shape(name):
    return SimpleNamespace(rope_base=10000.0, rms_eps=1e-6, qk_norm=False, tie_embed=False, **MODELS[name])


# ------------------------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest call: a whole step of the 2-layer float32 decoder, bound by launches
        dict(name="step_tiny_f32", op="step", model="tiny", batch=4, k=3, ctx_lo=128, ctx_hi=128, page=16),
        # one interactive sequence: every byte of the weights for four rows
        dict(name="verify_b1", op="verify", model="qwen3_4b", batch=1, k=3, ctx_lo=4001, ctx_hi=4001, page=16),
        # the rollout batch that the repository's benchmark runs by default
        dict(name="verify_b64", op="verify", model="qwen3_4b", batch=64, k=3, ctx_lo=1024, ctx_hi=4096, page=16),
        # a full rollout batch of the Qwen3-4B configuration (one of its 36 layers)
        dict(name="verify_b256", op="verify", model="qwen3_4b", batch=256, k=3, ctx_lo=512, ctx_hi=8704, page=16),
        # the MiMo-7B configuration (one layer): one draft per step, long contexts
        dict(name="verify_mimo_b128_k1", op="verify", model="mimo_7b", batch=128, k=1, ctx_lo=2048, ctx_hi=16384,
             page=16),
        # long contexts and the deepest chain, attention alone
        dict(name="attention_long_k7", op="attention", model="qwen3_4b", batch=32, k=7, ctx_lo=16384, ctx_hi=32768,
             page=16),
        # the accept of a training rollout: sampled at T = 1, the head's statistics handed over, the
        # cycle record taken
        dict(name="accept_record_b64", op="accept", batch=64, k=3, vocab=151936, mode="sample", temperature=1.0,
             top_p=1.0, record=64, handoff=True),
        # the evaluation setting: top-p 0.7
        dict(name="accept_top_p_b64", op="accept", batch=64, k=3, vocab=151936, mode="sample", temperature=1.0,
             top_p=0.7, record=0, handoff=False),
        # the draft of the default rollout batch
        dict(name="draft_b64", op="draft", model="qwen3_4b", batch=64, k=3, ctx_lo=1024, ctx_hi=4096, page=16,
             mode="sample", top_p=1.0),
        # a small batch drafting a deep chain under the evaluation setting
        dict(name="draft_top_p_b7_k5", op="draft", model="qwen3_4b", batch=7, k=5, ctx_lo=300, ctx_hi=2000, page=16,
             mode="sample", top_p=0.7),
        # head training: a chunk of 1024 recorded cycles re-run, then the loss and its gradient
        dict(name="reconstruct_r1024", op="reconstruct", model="qwen3_4b", batch=1024, k=3, ctx_lo=1024, ctx_hi=4096,
             page=16),
        dict(name="dca_n1024", op="dca", batch=1024, k=3, vocab=151936, topk=64, vgm=True),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["step", "verify", "verify", "verify", "attention", "accept", "accept", "draft", "draft",
                     "reconstruct", "dca"])
    page = rng.choice([16, 16, 32, 64])
    if op == "step":
        hi = _log_int(rng, 16, 1024)
        return dict(op=op, model=rng.choice(["tiny", "small"]), batch=_log_int(rng, 1, 32), k=rng.randint(1, 7),
                    ctx_lo=max(1, hi // rng.choice([1, 2, 8])), ctx_hi=hi, page=page)
    if op in ("verify", "attention", "draft", "reconstruct"):
        c = dict(op=op, model=rng.choice(["qwen3_4b", "qwen3_4b", "mimo_7b"]))
        if op == "reconstruct":
            c.update(batch=_log_int(rng, 16, 1024))
            c.update(k=rng.randint(1, min(5, 3072 // c["batch"])))
        elif op == "draft":
            c.update(batch=_log_int(rng, 1, 256))
            c.update(k=rng.randint(1, min(7, 1024 // c["batch"])))
        else:
            c.update(batch=_log_int(rng, 1, 256), k=rng.randint(0 if op == "verify" else 1, 7))
        tokens = 2_000_000 if op == "reconstruct" else 1_000_000   # cached positions over the batch
        hi = _log_int(rng, 64, max(65, min(32768, tokens // c["batch"])))
        c.update(ctx_lo=max(1, hi // rng.choice([1, 2, 4, 16])), ctx_hi=hi, page=page)
        if op == "draft":
            c.update(mode=rng.choice(["sample", "sample", "greedy"]), top_p=rng.choice([1.0, 1.0, 0.7, 0.95]))
        return c
    vocab = rng.choice([151936, 151680, 50257, 32001, 128256])
    if op == "accept":
        B = _log_int(rng, 1, 256)
        return dict(op=op, batch=B, k=rng.randint(1, min(7, 1024 // B)), vocab=vocab,
                    mode=rng.choice(["sample", "sample", "sample", "greedy"]), temperature=rng.choice([1.0, 1.0, 0.7]),
                    top_p=rng.choice([1.0, 1.0, 0.7, 0.95]), record=rng.choice([0, 0, 64, 16]),
                    handoff=rng.choice([True, False]))
    N = _log_int(rng, 8, 1024)
    return dict(op="dca", batch=N, k=rng.randint(1, min(7, 3072 // N)), vocab=vocab, topk=rng.choice([64, 64, 32, 8]),
                vgm=rng.choice([True, True, False]))


# ------------------------------------------------------------------------------------- inputs
_DEV = "cuda"
_TAGS = {t: i for i, t in enumerate(["weights", "mtp", "kv", "mtp_kv", "tokens", "logits", "lens", "pages", "misc"])}
_PEAK = 0.6      # how far the LM head's row of a token's successor leans towards that token's embedding
_PASS = 4.0      # gain of the draft head's projection on the token embedding


def _gen(seed, tag):
    g = torch.Generator(device=_DEV)
    g.manual_seed(seed * 1009 + _TAGS[tag])
    return g


def _normal(g, *shape, scale=1.0, dtype=torch.float32):
    t = torch.empty(shape, dtype=dtype, device=_DEV).normal_(generator=g)
    return t if scale == 1.0 else t.mul_(scale)


def _dtype(s):
    return torch.bfloat16 if s.dtype == "bf16" else torch.float32


def _layer_weights(g, s):
    dt = _dtype(s)
    H, d, F = s.hidden, s.head_dim, s.ffn
    lin = lambda o, i: _normal(g, o, i, scale=0.02, dtype=dt)
    ones = lambda n: torch.ones(n, dtype=dt, device=_DEV)
    return dict(attn_norm=ones(H), w_qkv=lin((s.n_heads + 2 * s.n_kv_heads) * d, H), w_o=lin(H, s.n_heads * d),
                ffn_norm=ones(H), w_gate_up=lin(2 * F, H), w_down=lin(H, F))


def _successor(V):
    """A permutation of the vocabulary: the token a confident head expects after each token."""
    step = next(p for p in (7919, 7907, 7901) if math.gcd(p, V) == 1)
    return (torch.arange(V, device=_DEV) * step + 13) % V


def _weights(seed, s, head=False):
    """Row-major weights: N(0, 0.02) as a random-init model's.  head=True leans each LM-head row
    towards the embedding of one predecessor token and lets the draft head's projection pass the
    embedding on, so that the head is as sure of its next token as a trained one."""
    g, dt = _gen(seed, "weights"), _dtype(s)
    V, H = s.vocab, s.hidden
    w = dict(embed=_normal(g, V, H, scale=0.02, dtype=dt), final_norm=torch.ones(H, dtype=dt, device=_DEV),
             lm_head=_normal(g, V, H, scale=0.02, dtype=dt), layers=[_layer_weights(g, s) for _ in range(s.n_layers)])
    if head:
        nxt = _successor(V)
        for v0 in range(0, V, 32768):
            e = w["embed"][v0:v0 + 32768].float()
            rows = nxt[v0:v0 + 32768]
            w["lm_head"][rows] = (w["lm_head"][rows].float() + _PEAK * e / e.norm(dim=1, keepdim=True)).to(dt)
    return w


def _mtp_weights(seed, s):
    g, dt = _gen(seed, "mtp"), _dtype(s)
    H = s.hidden
    ones = lambda: torch.ones(H, dtype=dt, device=_DEV)
    proj = _normal(g, H, 2 * H, scale=0.02, dtype=dt)
    proj[:, H:].diagonal().add_(_PASS)
    return dict(norm_h=ones(), norm_e=ones(), w_proj=proj, final_norm=ones(), layer=_layer_weights(g, s))


def _lens(case, seed):
    """Committed lengths spread evenly over the range and dealt in a shuffled order, so that every
    seed holds the same number of positions."""
    B, lo, hi = case["batch"], case["ctx_lo"], case["ctx_hi"]
    lens = lo + ((hi - lo + 1) * (2 * np.arange(B) + 1)) // (2 * B)
    return np.random.default_rng([seed, _TAGS["lens"]]).permutation(lens)


def _table(case, seed, lens, extra):
    """Page table: the pages of every sequence dealt from a shuffled pool."""
    need = (lens + extra + case["page"] - 1) // case["page"]
    perm = np.random.default_rng([seed, _TAGS["pages"]]).permutation(int(need.sum()))
    table = np.full((len(lens), int(need.max())), -1, dtype=np.int32)
    o = 0
    for b, n in enumerate(need):
        table[b, :n] = perm[o:o + n]
        o += n
    return table


def _pools(seed, tag, s, case, table, layers, out=None):
    """K and V pools of N(0, 1) entries in page order (into `out`'s tensors when given)."""
    g, n = _gen(seed, tag), int(table.max()) + 1
    blk = s.n_kv_heads * case["page"] * s.head_dim
    ks, vs = out if out else ([torch.empty((n, blk), dtype=_dtype(s), device=_DEV) for _ in range(layers)]
                              for _ in range(2))
    for t in list(ks) + list(vs):
        t.normal_(generator=g)
    return ks, vs


def _rand_tokens(seed, *shape, vocab):
    return torch.randint(0, vocab, shape, generator=_gen(seed, "tokens"), device=_DEV, dtype=torch.int32)


def _spiky(g, rows, V):
    """Logits as a language model's at T = 1: a broad floor and sixteen likely ids falling off by
    about 1.2 each (the first holds about half of the mass).  Returns (logits, likely ids)."""
    z = _normal(g, rows, V, scale=1.5)
    ids = torch.randint(0, V, (rows, 16), generator=g, device=_DEV)
    z.scatter_(1, ids, 16.0 - 1.2 * torch.arange(16, device=_DEV) + _normal(g, rows, 16, scale=0.5))
    return z, ids


def _near(g, z, ids):
    """Another model's logits for the same rows: its own floor, the likely ids moved by N(0, 0.7)."""
    y = _normal(g, *z.shape, scale=1.5)
    return y.scatter_(1, ids, z.gather(1, ids) + _normal(g, *ids.shape, scale=0.7))


def _accept_inputs(case, seed):
    B, k, V, T = case["batch"], case["k"], case["vocab"], case["temperature"]
    g = _gen(seed, "logits")
    zt, ids = _spiky(g, B * (k + 1), V)
    zt = zt.view(B, k + 1, V)
    zq = _near(g, zt[:, :k].reshape(B * k, V), ids.view(B, k + 1, 16)[:, :k].reshape(B * k, 16)).view(B, k, V)
    # drafts as the head draws them: from softmax(z / T), or from its nucleus
    p = torch.softmax(zq.double() / T, -1)
    top, at = p.topk(64, -1)
    if case["mode"] == "greedy":
        drafts = at[..., 0]
    else:
        keep = (top.cumsum(-1) - top) < case["top_p"]
        m = (top * keep).cumsum(-1)
        u = torch.rand((B, k, 1), generator=g, device=_DEV, dtype=torch.float64)
        drafts = at.gather(-1, torch.searchsorted(m, u * m[..., -1:], right=True).clamp_(max=63))[..., 0]
    d = dict(zt=zt, zq=zq, drafts=drafts.to(torch.int32).contiguous(),
             u_accept=torch.rand((B, k), generator=g, device=_DEV), u_final=torch.rand((B,), generator=g, device=_DEV))
    if case["handoff"] and case["top_p"] >= 1.0 and case["mode"] == "sample":
        y = zq * (1.0 / T) if T != 1.0 else zq
        mx = y.max(-1)
        st = torch.zeros((B, k, gm.ROW_STATS_BYTES), dtype=torch.uint8, device=_DEV)
        st[..., 0:4].view(torch.float32)[..., 0] = mx.values
        st[..., 4:8].view(torch.int32)[..., 0] = mx.indices.to(torch.int32)
        st[..., 8:16].view(torch.float64)[..., 0] = (y.double() - mx.values.double()[..., None]).exp().sum(-1)
        d["stats"] = st
    return d


def _dca_inputs(case, seed):
    N, K, V = case["batch"], case["k"], case["vocab"]
    g = _gen(seed, "logits")
    z = torch.empty((N * K, V), dtype=torch.float32, device=_DEV)
    lp, ids = [], []
    for r in range(0, N * K, 256):     # the record of the target's rows, in parts
        t, at = _spiky(g, min(256, N * K - r), V)
        z[r:r + 256] = _near(g, t, at)
        top = t.topk(case["topk"], -1)
        lp.append((top.values.double() - torch.logsumexp(t.double(), -1, keepdim=True)).to(torch.bfloat16))
        ids.append(top.indices.to(torch.int32))
    return dict(z=z.view(N, K, V), logp=torch.cat(lp).view(N, K, -1), ids=torch.cat(ids).view(N, K, -1),
                n=torch.randint(0, K + 1, (N,), generator=g, device=_DEV, dtype=torch.int32))


def _draft_inputs(case, seed, s):
    """What the step before hands the draft: the verify's hiddens, the accepted counts, the tokens."""
    B, R = case["batch"], case["k"] + 1
    g = _gen(seed, "misc")
    n = torch.randint(0, R, (B,), generator=g, device=_DEV, dtype=torch.int32)
    toks = _rand_tokens(seed, B, R, vocab=s.vocab)
    toks[torch.arange(R, device=_DEV)[None, :] > n[:, None]] = -1
    return dict(hidden=_normal(g, B, R, s.hidden, scale=3.0), n=n, tokens=toks,
                u=torch.rand((B, case["k"]), generator=g, device=_DEV))


def _recon_inputs(case, seed, s):
    R, g = case["batch"], _gen(seed, "misc")
    return dict(hidden=_normal(g, R, s.hidden, scale=3.0),
                tokens=torch.randint(0, s.vocab, (R,), generator=g, device=_DEV, dtype=torch.int32),
                drafts=_rand_tokens(seed, R, case["k"], vocab=s.vocab))


# ------------------------------------------------------------------------------------- device state
def _pack(s, w):
    """A linear weight in the layout gm.h gives its dtype (tiles of 16 x 32 for bf16)."""
    if s.dtype != "bf16":
        return w
    n, k = w.shape
    return w.view(n // 128, 8, 16, k // 32, 4, 8).permute(0, 3, 1, 4, 2, 5).contiguous()


def _p(t):
    return ctypes.c_void_p(t.data_ptr())


def _layer_struct(s, L):
    packed = {n: _pack(s, t) if n.startswith("w_") else t for n, t in L.items()}
    st = gm.LayerWeights(_p(packed["attn_norm"]), _p(packed["w_qkv"]), None, None, _p(packed["w_o"]),
                         _p(packed["ffn_norm"]), _p(packed["w_gate_up"]), _p(packed["w_down"]))
    return st, packed


def _device_model(s, w):
    parts = [_layer_struct(s, L) for L in w["layers"]]
    arr = (gm.LayerWeights * len(parts))(*[p[0] for p in parts])
    head = _pack(s, w["lm_head"])
    st = gm.ModelWeights(_p(w["embed"]), _p(w["final_norm"]), _p(head),
                         ctypes.cast(arr, ctypes.POINTER(gm.LayerWeights)))
    return SimpleNamespace(shape=s, cfg=gm.model_config(s), struct=st, keep=(w["embed"], w["final_norm"], head, arr,
                                                                             [p[1] for p in parts]))


def _device_mtp(s, w):
    L, kept = _layer_struct(s, w["layer"])
    proj = _pack(s, w["w_proj"])
    st = gm.MtpWeights(_p(w["norm_h"]), _p(w["norm_e"]), _p(proj), _p(w["final_norm"]), L)
    return SimpleNamespace(struct=st, keep=(w["norm_h"], w["norm_e"], proj, w["final_norm"], kept))


def _cache(case, seed, s, layers, tag, extra):
    lens = _lens(case, seed)
    table = _table(case, seed, lens, extra)
    c = gm.PagedCache(s, layers, lens, lens + extra, page_size=case["page"], fill="empty", table=table)
    _pools(seed, tag, s, case, table, layers, out=(c.k, c.v))
    return c


def _extra(case):
    return 2 * case["k"] + 2


def prepare(case, seed):
    op, B, k = case["op"], case["batch"], case["k"]
    R = k + 1
    f32, i32 = dict(dtype=torch.float32, device=_DEV), dict(dtype=torch.int32, device=_DEV)
    st = SimpleNamespace(case=case, op=op, k=k, ws=gm.Workspace(), ws2=gm.Workspace(), ws3=gm.Workspace())
    if op == "accept":
        st.__dict__.update(_accept_inputs(case, seed))
        st.n, st.out = torch.zeros(B, **i32), torch.zeros((B, R), **i32)
        st.mode = gm.GM_SAMPLE if case["mode"] == "sample" else gm.GM_GREEDY
        st.record = None
        if case["record"]:
            st.record = (torch.zeros((B, k, case["record"]), dtype=torch.bfloat16, device=_DEV),
                         torch.zeros((B, k, case["record"]), **i32))
        return st
    if op == "dca":
        st.__dict__.update(_dca_inputs(case, seed))
        st.loss, st.alpha, st.grad = torch.zeros(B, **f32), torch.zeros((B, k), **f32), torch.empty_like(st.z)
        return st
    s = st.shape = _shape(case["model"])
    if op == "attention":
        st.cfg = gm.model_config(s)
        st.cache = _cache(case, seed, s, 1, "kv", _extra(case))
        st.q = _normal(_gen(seed, "misc"), B, R, s.n_heads, s.head_dim, dtype=_dtype(s))
        st.out = torch.empty_like(st.q)
        return st
    st.model = _device_model(s, _weights(seed, s, head=op in ("draft", "reconstruct")))
    if op in ("verify", "step"):
        st.cache = _cache(case, seed, s, s.n_layers, "kv", _extra(case))
        st.tokens = _rand_tokens(seed, B, R, vocab=s.vocab)
        st.logits, st.hidden = torch.empty((B, R, s.vocab), **f32), torch.empty((B, R, s.hidden), **f32)
    if op in ("draft", "step", "reconstruct"):
        st.mtp = _device_mtp(s, _mtp_weights(seed, s))
        st.mcache = _cache(case, seed, s, 1, "mtp_kv", _extra(case))
        st.lens0 = st.mcache.seq_lens.clone()
    if op in ("draft", "step"):
        st.drafts, st.dlog = torch.zeros((B, k), **i32), torch.empty((B, k, s.vocab), **f32)
    if op == "step":
        st.n, st.out = torch.zeros(B, **i32), torch.zeros((B, R), **i32)
        st.block = st.tokens[:, 1:].contiguous()
    if op == "draft":
        d = _draft_inputs(case, seed, s)
        st.hidden, st.n, st.tokens, st.u = d["hidden"], d["n"], d["tokens"], d["u"]
        st.mode = gm.GM_SAMPLE if case["mode"] == "sample" else gm.GM_GREEDY
        top_p = case["mode"] == "sample" and case["top_p"] < 1.0
        st.stats = None if top_p else gm.new_row_stats(B, k)
        st.nuclei = gm.new_nuclei(B, k) if top_p else None
    if op == "reconstruct":
        d = _recon_inputs(case, seed, s)
        st.hidden, st.tokens, st.drafts = d["hidden"], d["tokens"], d["drafts"]
        st.logits = torch.empty((B, k, s.vocab), **f32)
    return st


def run(st):
    c, k = st.case, st.k
    if st.op == "verify":
        gm.verify_forward(st.model, st.cache, st.tokens, st.logits, st.hidden, st.ws)
        return dict(logits=st.logits, hidden=st.hidden, k_pages=st.cache.k, v_pages=st.cache.v)
    if st.op == "attention":
        gm.verify_attention(st.cfg, st.cache, 0, st.q, st.out, st.ws)
        return dict(out=st.out)
    if st.op == "accept":
        gm.spec_accept(st.zt, st.zq, st.drafts, st.u_accept, st.u_final, st.n, st.out, st.mode, st.ws,
                       temperature=c["temperature"], draft_stats=getattr(st, "stats", None), record=st.record,
                       top_p=c["top_p"])
        out = dict(n_accept=st.n, tokens=st.out)
        if st.record:
            out.update(logp=st.record[0], ids=st.record[1])
        return out
    if st.op == "draft":
        # the head's committed lengths move with every call; a program's next block starts from the
        # new ones, here each pass drafts the same block again
        st.mcache.seq_lens.copy_(st.lens0)
        gm.mtp_draft(st.model, st.mtp, st.mcache, k, st.mode, st.hidden, st.n, st.tokens, st.u, st.drafts, st.dlog,
                     st.ws, draft_stats=st.stats, top_p=c["top_p"], draft_nucleus=st.nuclei)
        out = dict(drafts=st.drafts, logits=st.dlog, lens=st.mcache.seq_lens, k_pages=st.mcache.k, v_pages=st.mcache.v)
        if st.stats is not None:
            out.update(max=st.stats[..., 0:4].view(torch.float32), argmax=st.stats[..., 4:8].view(torch.int32),
                       sum=st.stats[..., 8:16].view(torch.float64))
        else:
            out.update(mass=st.nuclei[..., 8:16].view(torch.float64), last=st.nuclei[..., 20:24].view(torch.int32))
        return out
    if st.op == "step":
        # both caches start every pass from the same committed lengths
        st.mcache.seq_lens.copy_(st.lens0)
        st.cache.seq_lens.copy_(st.lens0)
        gm.verify_forward(st.model, st.cache, st.tokens, st.logits, st.hidden, st.ws)
        gm.spec_accept(st.logits, None, st.block, None, None, st.n, st.out, gm.GM_GREEDY, st.ws2)
        gm.kv_commit(st.cache, k, st.n)
        gm.mtp_draft(st.model, st.mtp, st.mcache, k, gm.GM_GREEDY, st.hidden, st.n, st.out, None, st.drafts, st.dlog,
                     st.ws3)
        return dict(logits=st.logits, hidden=st.hidden, n_accept=st.n, tokens=st.out, drafts=st.drafts,
                    draft_logits=st.dlog, lens=st.cache.seq_lens, head_lens=st.mcache.seq_lens, k_pages=st.cache.k,
                    v_pages=st.cache.v, head_k=st.mcache.k, head_v=st.mcache.v)
    if st.op == "reconstruct":
        gm.mtp_reconstruct(st.model, st.mtp, st.mcache, k, st.hidden, st.tokens, st.drafts, st.logits, st.ws)
        return dict(logits=st.logits)
    gm.dca_loss(st.z, st.logp, st.ids, st.n, st.loss, st.alpha, st.grad, st.ws, vgm=c["vgm"])
    return dict(loss=st.loss, alpha=st.alpha, grad=st.grad)


# ------------------------------------------------------------------------------------- work
def work(case):
    op, B, k = case["op"], case["batch"], case["k"]
    R = k + 1
    if op == "accept":
        V = case["vocab"]
        # the target rows once; the draft rows once, or, where their statistics are handed over,
        # the one row per sequence that a residual draw needs
        rows = B * R
        if case["mode"] == "sample":
            rows += B * (1 if case["handoff"] and case["top_p"] >= 1.0 else k)
        return dict(bytes=4.0 * rows * V + 6.0 * B * k * case["record"], flops=2.0 * rows * V)
    if op == "dca":
        n = B * k * case["vocab"]
        return dict(bytes=8.0 * n + 6.0 * B * k * case["topk"], flops=4.0 * n)
    s = _shape(case["model"])
    e = 2.0 if s.dtype == "bf16" else 4.0
    H, F, V, d, nq, nkv, L = s.hidden, s.ffn, s.vocab, s.head_dim, s.n_heads, s.n_kv_heads, s.n_layers
    ctx = (case["ctx_lo"] + case["ctx_hi"]) / 2.0
    kv = B * (ctx + R) * nkv * d * 2 * e
    M = B * R
    attn = 4.0 * M * nq * d * (ctx + R / 2.0)
    if op == "attention":
        return dict(bytes=kv + 2 * e * M * nq * d, flops=attn)
    layer = H * (nq + 2 * nkv) * d + nq * d * H + 3.0 * H * F
    verify = dict(bytes=e * (L * layer + V * H + M * H) + L * kv + 4.0 * M * (V + H),
                  flops=2.0 * M * (L * layer + V * H) + L * attn)
    if op == "verify":
        return verify
    # the chain is serial and the head's weights and caches are larger than any cache of the
    # chip: every depth reads them again
    head = 2.0 * H * H + layer + V * H
    chain = dict(bytes=k * (e * head + B * (ctx + 1) * nkv * d * 2 * e + 4.0 * B * V),
                 flops=k * (2.0 * B * head + 4.0 * B * nq * d * ctx))
    if op in ("draft", "step"):     # the extend's further rows: the projection and the K/V columns
        chain["bytes"] += 4.0 * M * H
        chain["flops"] += 2.0 * (M - B) * (2.0 * H * H + 2 * nkv * d * H)
    if op == "step":
        return dict(bytes=verify["bytes"] + chain["bytes"], flops=verify["flops"] + chain["flops"])
    return chain


# ------------------------------------------------------------------------------------- tolerance
def tolerance(case):
    op = case["op"]
    if op == "step":         # float32 sums in another order, through two layers and the head
        return dict(rel=4e-6, max=1e-4)
    if op == "attention":    # one bf16 rounding of the output
        return dict(rel=6e-3, max=3e-2)
    if op == "accept":       # decisions; the record's log-probabilities are bf16 of a float64 value
        return dict(rel=1e-3, max=1e-2, differ=0.002)
    if op == "dca":          # float32 exponentials scaled by float64 normalisers
        return dict(rel=1e-6, max=1e-5)
    # bf16 operands, float32 sums: a layer, the LM head (and the chain's layers one after another)
    return dict(rel=1.5e-2, max=0.15, differ=0.002)


# ------------------------------------------------------------------------------------- float64
def _rms64(x, w, eps):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + eps) * w.double()


def _lin64(x, w):
    """x W^T in float64, the weight widened in parts."""
    out = torch.empty(x.shape[0], w.shape[0], dtype=torch.float64, device=x.device)
    for r in range(0, w.shape[0], 16384):
        out[:, r:r + 16384] = x @ w[r:r + 16384].double().t()
    return out


def _rope64(x, pos, base):
    """Rotate-half over the last axis of [rows, heads, d]."""
    h = x.shape[-1] // 2
    ang = pos.double()[:, None, None] * base ** (-torch.arange(h, device=x.device, dtype=torch.float64) / h)
    c, s = ang.cos(), ang.sin()
    a, b = x[..., :h], x[..., h:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


class _Kv64:
    """The logical K and V entries of every sequence of one layer: the prefix unpacked from the
    pages, then the entries appended so far."""

    def __init__(self, case, s, pool_k, pool_v, table, lens):
        self.s, self.page, self.table, self.lens = s, case["page"], torch.from_numpy(table).to(_DEV).long(), lens
        n = pool_k.shape[0]
        tiles = (n, s.n_kv_heads, case["page"] // 16, s.head_dim // 32)
        self.k = pool_k.view(*tiles, 4, 16, 8)        # [.., column block, token, column]
        self.v = pool_v.view(*tiles, 4, 16, 2, 4)     # [.., token / 4, column % 16, column / 16, token % 4]
        self.new = [([], []) for _ in lens]

    def length(self, b):
        return int(self.lens[b]) + sum(t.shape[0] for t in self.new[b][0])

    def add(self, b, k, v):
        self.new[b][0].append(k)
        self.new[b][1].append(v)

    def entries(self, b):
        m, s = int(self.lens[b]), self.s
        pages = self.table[b, :(m + self.page - 1) // self.page]
        # -> [page, tile, token, head, column]
        k = self.k[pages].permute(0, 2, 5, 1, 3, 4, 6).reshape(-1, s.n_kv_heads, s.head_dim)[:m].double()
        v = self.v[pages].permute(0, 2, 4, 7, 1, 3, 6, 5).reshape(-1, s.n_kv_heads, s.head_dim)[:m].double()
        return torch.cat([k] + self.new[b][0]), torch.cat([v] + self.new[b][1])


def _attend64(q, k, v, first):
    """q [R, nq, d] against k, v [T, nkv, d]; row i sees entries 0 .. first + i."""
    R, nq, d = q.shape
    T, nkv = k.shape[0], k.shape[1]
    G = nq // nkv
    qq = q.view(R, nkv, G, d).permute(1, 2, 0, 3).reshape(nkv, G * R, d)
    sc = torch.matmul(qq, k.permute(1, 2, 0).contiguous()) / math.sqrt(d)
    see = torch.arange(T, device=q.device)[None, :] <= (first + torch.arange(R, device=q.device))[:, None]
    sc = sc.view(nkv, G, R, T).masked_fill(~see, -math.inf).softmax(-1).view(nkv, G * R, T)
    o = torch.matmul(sc, v.permute(1, 0, 2).contiguous())
    return o.view(nkv, G, R, d).permute(2, 0, 1, 3).reshape(R, nq * d)


def _layer64(s, L, x, pos, kv, rows):
    """One decoder layer on x [M, H]; rows: (sequence, first row, count) of the rows that attend."""
    d, nq, nkv = s.head_dim, s.n_heads, s.n_kv_heads
    M = x.shape[0]
    qkv = _lin64(_rms64(x, L["attn_norm"], s.rms_eps), L["w_qkv"]).view(M, nq + 2 * nkv, d)
    q, k, v = _rope64(qkv[:, :nq], pos, s.rope_base), _rope64(qkv[:, nq:nq + nkv], pos, s.rope_base), qkv[:, nq + nkv:]
    att = torch.zeros(M, nq * d, dtype=torch.float64, device=x.device)
    for b, r, n in rows:
        first = kv.length(b)
        kv.add(b, k[r:r + n], v[r:r + n])
        K, V = kv.entries(b)
        att[r:r + n] = _attend64(q[r:r + n], K, V, first)
    x = x + _lin64(att, L["w_o"])
    gu = _lin64(_rms64(x, L["ffn_norm"], s.rms_eps), L["w_gate_up"])
    return x + _lin64(torch.nn.functional.silu(gu[:, :s.ffn]) * gu[:, s.ffn:], L["w_down"])


def _verify64(case, seed, s, w):
    B, R = case["batch"], case["k"] + 1
    lens = _lens(case, seed)
    table = _table(case, seed, lens, _extra(case))
    ks, vs = _pools(seed, "kv", s, case, table, s.n_layers)
    toks = _rand_tokens(seed, B, R, vocab=s.vocab)
    x = w["embed"][toks.view(-1).long()].double()
    pos = (torch.from_numpy(lens).to(_DEV)[:, None] + torch.arange(R, device=_DEV)).view(-1)
    for l in range(s.n_layers):
        x = _layer64(s, w["layers"][l], x, pos, _Kv64(case, s, ks[l], vs[l], table, lens),
                     [(b, b * R, R) for b in range(B)])
    z = _lin64(_rms64(x, w["final_norm"], s.rms_eps), w["lm_head"])
    return toks, z.view(B, R, -1), x.view(B, R, -1)


def _head_input64(s, w, m, h, toks):
    e = w["embed"][toks.clamp(min=0).long()].double()
    return _lin64(torch.cat([_rms64(h, m["norm_h"], s.rms_eps), _rms64(e, m["norm_e"], s.rms_eps)], -1), m["w_proj"])


def _choose64(z, u, mode, top_p):
    """The draft of each row: the argmax, or the inverse-CDF draw (from the nucleus)."""
    if mode == "greedy":
        return z.argmax(-1)
    p = torch.softmax(z, -1)
    if top_p < 1.0:
        sp, at = p.sort(dim=-1, descending=True, stable=True)
        p = torch.zeros_like(p).scatter_(-1, at, sp * ((sp.cumsum(-1) - sp) < top_p))
    c = p.cumsum(-1)
    return torch.searchsorted(c, u.double()[:, None] * c[:, -1:], right=True).clamp_(max=z.shape[-1] - 1)[:, 0]


def _head_cache64(case, seed, s):
    lens = _lens(case, seed)
    table = _table(case, seed, lens, _extra(case))
    ks, vs = _pools(seed, "mtp_kv", s, case, table, 1)
    return lens, _Kv64(case, s, ks[0], vs[0], table, lens)


def _draft64(case, seed, s, w, hidden, n, toks, u, mode, top_p):
    B, k, R = case["batch"], case["k"], case["k"] + 1
    m = _mtp_weights(seed, s)
    lens, kv = _head_cache64(case, seed, s)
    ld, nn = torch.from_numpy(lens).to(_DEV), n.long()
    x = _head_input64(s, w, m, hidden.double().reshape(B * R, -1), toks.reshape(-1))
    pos = (ld[:, None] + torch.arange(R, device=_DEV) + 1).view(-1)
    cnt = (nn + 1).tolist()
    g = _layer64(s, m["layer"], x, pos, kv, [(b, b * R, cnt[b]) for b in range(B)])
    g = g.view(B, R, -1)[torch.arange(B, device=_DEV), nn]
    logits, drafts = [], []
    for j in range(k):
        if j:
            x = _head_input64(s, w, m, g, drafts[-1])
            g = _layer64(s, m["layer"], x, ld + nn + 1 + j, kv, [(b, b, 1) for b in range(B)])
        z = _lin64(_rms64(g, m["final_norm"], s.rms_eps), w["lm_head"])
        logits.append(z)
        drafts.append(_choose64(z, None if u is None else u[:, j], mode, top_p))
    return torch.stack(logits, 1), torch.stack(drafts, 1), ld + nn + 1


def exact(case, seed):
    op, B, k = case["op"], case["batch"], case["k"]
    if op == "accept":
        if not case["record"]:
            return None
        y = _accept_inputs(case, seed)["zt"][:, :k].double() / case["temperature"]
        return dict(n_accept=None, tokens=None, ids=None,
                    logp=y.topk(case["record"], -1).values - torch.logsumexp(y, -1, keepdim=True))
    if op == "dca":
        return _dca64(case, seed)
    s = _shape(case["model"])
    if op == "attention":
        lens = _lens(case, seed)
        table = _table(case, seed, lens, _extra(case))
        ks, vs = _pools(seed, "kv", s, case, table, 1)
        kv = _Kv64(case, s, ks[0], vs[0], table, lens + k + 1)
        q = _normal(_gen(seed, "misc"), B, k + 1, s.n_heads, s.head_dim, dtype=_dtype(s)).double()
        o = [_attend64(q[b], *kv.entries(b), int(lens[b])) for b in range(B)]
        return dict(out=torch.stack(o).view(q.shape))
    w = _weights(seed, s, head=op in ("draft", "reconstruct"))
    if op == "verify":
        _, z, x = _verify64(case, seed, s, w)
        return dict(logits=z, hidden=x)
    if op == "reconstruct":
        d, m = _recon_inputs(case, seed, s), _mtp_weights(seed, s)
        lens, kv = _head_cache64(case, seed, s)
        ld = torch.from_numpy(lens).to(_DEV)
        out = torch.empty(B, k, s.vocab, dtype=torch.float64, device=_DEV)
        g = d["hidden"].double()
        for j in range(k):
            x = _head_input64(s, w, m, g, d["tokens"] if j == 0 else d["drafts"][:, j - 1])
            g = _layer64(s, m["layer"], x, ld + j + 1, kv, [(b, b, 1) for b in range(B)])
            out[:, j] = _lin64(_rms64(g, m["final_norm"], s.rms_eps), w["lm_head"])
        return dict(logits=out)
    if op == "draft":
        d = _draft_inputs(case, seed, s)
        z, _, _ = _draft64(case, seed, s, w, d["hidden"], d["n"], d["tokens"], d["u"], case["mode"], case["top_p"])
        out = dict(logits=z)
        if case["mode"] == "greedy" or case["top_p"] >= 1.0:
            mx = z.max(-1, keepdim=True).values
            out.update(max=mx, sum=(z - mx).exp().sum(-1, keepdim=True))
        return out
    toks, z, x = _verify64(case, seed, s, w)
    am = z.argmax(-1).to(torch.int32)
    n = (toks[:, 1:] == am[:, :k]).long().cumprod(-1).sum(-1)
    fin = am.gather(1, n[:, None])
    at = torch.arange(k + 1, device=_DEV)[None, :]
    out = torch.where(at < n[:, None], torch.cat([toks[:, 1:], toks[:, :1]], 1), torch.full_like(am, -1))
    out = torch.where(at == n[:, None], fin, out)
    dz, _, _ = _draft64(case, seed, s, w, x, n, out, None, "greedy", 1.0)
    return dict(logits=z, hidden=x, draft_logits=dz)


def _dca64(case, seed):
    """Loss, overlaps and gradient from their closed forms: q over the whole vocabulary, p on the
    record's ids, one residual bin for the mass outside them."""
    d = _dca_inputs(case, seed)
    N, K, V = d["z"].shape
    ids, p = d["ids"].long(), d["logp"].double().exp()
    L = (d["n"].long() + 1).clamp(max=K) if case["vgm"] else torch.full((N,), K, device=_DEV)
    lse = torch.stack([torch.logsumexp(d["z"][:, j].double(), -1) for j in range(K)], 1)
    q = (d["z"].gather(-1, ids).double() - lse[..., None]).exp()
    p_r, q_r = (1 - p.sum(-1)).clamp(min=0), 1 - q.sum(-1)
    alpha = torch.minimum(p, q).sum(-1) + torch.minimum(p_r, q_r)
    own, rest = (q < p).double(), (q_r < p_r).double()
    mean = (own * q).sum(-1) + rest * q_r
    pre = alpha.cumprod(-1)
    inside = torch.arange(K, device=_DEV)[None, :] < L[:, None]
    chain = (pre * inside).sum(-1)
    # coefficient of position i: -(sum over l >= i of the products up to l) / (alpha_i * chain)
    tail = (pre * inside).flip(-1).cumsum(-1).flip(-1)
    coef = torch.where(inside, -tail / (alpha * chain[:, None]), torch.zeros_like(tail))
    grad = torch.empty(N, K, V, dtype=torch.float64, device=_DEV)
    for j in range(K):
        g = (d["z"][:, j].double() - lse[:, j, None]).exp() * ((rest - mean)[:, j] * coef[:, j])[:, None]
        grad[:, j] = g.scatter(-1, ids[:, j], q[:, j] * (own[:, j] - mean[:, j, None]) * coef[:, j, None])
    return dict(loss=-chain.log(), alpha=alpha, grad=grad)
