"""GPU parity of the top-p variant of gm_spec_accept (the evaluation setting of
App. "Evaluation Configuration": rejection sampling at T = 1, top-p 0.7) against
the oracle on the same seeded logits.  The drafts are samples of the head's
nucleus (and, in the handoff test, the oracle's own draft head's draws).  Accept
counts and committed tokens must match bit for bit outside the flag windows (|u - min(1, p/q)| < 1e-3, a final draw within the derived float32
bound ``draw_window`` of a CDF edge, and a nucleus whose boundary lies within
5e-9 of top_p); the flagged count is printed."""
import numpy as np
import pytest
import torch

import oracle
import synth
from helpers import need_gpu, t32, i32, flag_report, draw_window
from paper_2609_16648_amd import gm

pytestmark = pytest.mark.gpu
NUC_EPS = 5e-9         # >= V 2^-45, the largest distance of the kernel's fixed-point sums from float64


def _nucleus_drafts(zq, ud, top_p, temperature):
    """d_i ~ nucleus(q_i) by the inverse CDF."""
    B, k, V = zq.shape
    q = oracle.softmax(zq.astype(np.float64) / temperature)
    qn = oracle.nucleus(zq, q, top_p)[0]
    d = np.zeros((B, k), np.int64)
    for i in range(k):
        d[:, i] = oracle.inverse_cdf_rows(qn[:, i], ud[:, i])[0]
    return d


def _run(zt, zq, drafts, ua, uf, mode, temperature, top_p):
    B, k1, V = zt.shape
    n = torch.zeros(B, dtype=torch.int32, device="cuda")
    out = torch.zeros((B, k1), dtype=torch.int32, device="cuda")
    gm.spec_accept(t32(zt), t32(zq) if zq is not None else None, i32(drafts), t32(ua) if ua is not None else None,
                   t32(uf) if uf is not None else None, n, out, mode, gm.Workspace(), temperature=temperature,
                   top_p=top_p)
    torch.cuda.synchronize()
    return n.cpu().numpy(), out.cpu().numpy()


def _logits(shape, kind, *tags):
    z = synth.normal_logits(shape, 3, *tags)
    if kind == "ties":          # values on a 0.5 grid: long runs of equal logits at every boundary
        z = np.round(z * 2.0) / 2.0
    elif kind == "flat":        # nearly every logit equal: the boundary inside a run of ~10^5 ties
        z = np.where(synth.stream(3, "flat", *tags).random(shape) < 1e-3, z * 3.0, 0.0)
    elif kind in ("peaked", "plateau", "wide", "tail"):
        g, V = synth.stream(3, "peak", *tags), shape[-1]
        rows = z.reshape(-1, V)
        for r in rows:
            if kind == "peaked":      # a language model's row: sixteen likely ids over a broad floor
                r[g.integers(0, V, 16)] = 14.0 - 1.2 * np.arange(16) + 0.5 * g.standard_normal(16)
            elif kind == "plateau":   # 400 equal logits around the boundary, more than are ranked by counting
                r[g.integers(0, V, 400)] = 8.0
                r[g.integers(0, V)] = 13.5
            elif kind == "wide":      # 20000 equal likely ids side by side, more than are queued
                lo = int(g.integers(0, V - 20000))
                r[:] = -20.0
                r[lo:lo + 20000] = 0.0
                r[g.integers(0, V)] = 6.1
            else:                     # one likely id, the rest of the mass in ids too unlikely to queue
                r[g.integers(0, V)] = np.log(0.1 * np.exp(r.astype(np.float64)).sum())
    return z.astype(np.float32)


@pytest.mark.parametrize("B,k,V,T,top_p,kind", [
    (64, 3, 151936, 1.0, 0.7, "normal"),       # the evaluation setting at the layer workload's shape
    (32, 7, 151936, 0.7, 0.9, "normal"),
    (257, 2, 1000, 1.0, 0.5, "normal"),        # ragged vocabulary, more sequences than CUs
    (40, 3, 5000, 1.0, 0.7, "ties"),           # the boundary inside a run of equal logits
    (8, 1, 4096, 1.3, 0.2, "ties"),
    (8, 2, 151936, 1.0, 0.5, "flat"),          # too many ties for LDS: the passes over the row
    (3, 0, 5000, 1.0, 0.7, "normal"),          # no drafts: the bonus draw from the target's nucleus
    (16, 2, 1001, 1.0, 0.6, "normal"),         # rows not a multiple of 4 ids: unaligned row reads
    (1, 1, 151936, 1.0, 0.7, "normal"),        # one sequence: the first pass split over 16 workgroups
    # few rows of a middle vocabulary: split as far as its ids go, in 12 slices off 16-byte boundaries
    (4, 3, 50257, 1.0, 0.7, "normal"),
    (6, 1, 50257, 1.0, 0.7, "peaked"),
    (1, 2, 50257, 1.0, 0.95, "wide"),
    (2, 1, 32768, 1.0, 0.7, "peaked"),         # the least number of ids that is cut into eight slices
    # a head close to the target (zq = zt + 0.1 N(0, 1)): most drafts accepted, so the deep
    # prefixes and the bonus draw from the last target row's nucleus are compared
    # peaked rows, queued in one pass: ranked by counting, by the radix selection over the queue, too
    # many to queue, and the boundary past the queue; one block per row and split over blocks
    (64, 3, 151936, 1.0, 0.7, "peaked"),
    (5, 2, 32001, 0.7, 0.95, "peaked"),
    (48, 2, 20000, 1.0, 0.7, "plateau"),
    (6, 1, 151936, 1.0, 0.8, "plateau"),
    (44, 2, 50257, 1.0, 0.95, "wide"),
    (16, 0, 151936, 1.0, 0.95, "wide"),
    (44, 2, 50256, 1.0, 0.7, "tail"),
    (16, 0, 151936, 1.0, 0.7, "tail"),
    (64, 3, 151936, 1.0, 0.7, "overlap"),
    (32, 7, 151936, 1.0, 0.7, "overlap"),
])
def test_top_p_accept_matches_oracle(B, k, V, T, top_p, kind):
    need_gpu()
    zt = _logits((B, k + 1, V), kind, "tp-t", B, k, V)
    if kind == "overlap":
        zq = (zt[:, :k] + np.float32(0.1) * synth.normal_logits((B, k, V), 3, "tp-q", B, k, V)).astype(np.float32)
    else:
        zq = _logits((B, k, V), kind, "tp-q", B, k, V)
    ua, uf, ud = synth.uniforms(B, k, 4, "tp", B, k, V)
    drafts = _nucleus_drafts(zq, ud, top_p, T)
    ref = oracle.spec_accept(zt, zq, drafts, ua, uf, temperature=T, top_p=top_p, nucleus_eps=NUC_EPS,
                             final_abs=draw_window(zt, zq, T, top_p))
    n, out = _run(zt, zq, drafts, ua, uf, gm.GM_SAMPLE, T, top_p)
    name = "top-p %.2f T=%.1f B=%d k=%d V=%d %s" % (top_p, T, B, k, V, kind)
    flag_report(name, ref.flagged, B)
    ok, oka = ~ref.flagged, ~ref.flag_accept     # a flagged final draw leaves the accept count comparable
    np.testing.assert_array_equal(n[oka], ref.n_accept[oka])
    np.testing.assert_array_equal(out[ok], ref.out_tokens[ok])
    assert ref.flagged.sum() <= max(1, 0.1 * B)
    if kind == "overlap":       # deep prefixes and bonus draws are among the compared sequences
        assert n[ok].mean() > k / 2 and (n[ok] == k).sum() >= 4, (n.mean(), (n == k).sum())
    # every committed final token lies in the nucleus of its target row (all sequences)
    p = oracle.softmax(zt.astype(np.float64) / T)
    for b in range(B):
        row = oracle.nucleus(zt[b, n[b]], p[b, n[b]], top_p)
        if row[1] >= NUC_EPS:
            assert row[0][out[b, n[b]]] > 0, (b, n[b], out[b, n[b]])
    print("[%s] mean accepted %.2f, all k accepted in %d" % (name, n.mean(), (n == k).sum()), flush=True)


def test_top_p_one_is_the_plain_rule():
    need_gpu()
    B, k, V = 32, 3, 151936
    zt = _logits((B, k + 1, V), "normal", "tp1-t")
    zq = _logits((B, k, V), "normal", "tp1-q")
    ua, uf, ud = synth.uniforms(B, k, 4, "tp1")
    drafts = _nucleus_drafts(zq, ud, 1.0, 1.0)
    a = _run(zt, zq, drafts, ua, uf, gm.GM_SAMPLE, 1.0, 1.0)
    b = _run(zt, zq, drafts, ua, uf, gm.GM_SAMPLE, 1.0, 0.999999)   # a nucleus of nearly all ids
    np.testing.assert_array_equal(a[0], b[0])


def test_tiny_top_p_is_greedy():
    # every nucleus is the row's argmax: with drafts = the head's argmax, sampled
    # acceptance at top_p -> 0 takes the greedy rule's decisions and tokens
    need_gpu()
    B, k, V = 48, 3, 151936
    zt = _logits((B, k + 1, V), "normal", "tp0-t")
    zq = _logits((B, k, V), "normal", "tp0-q")
    agree = np.random.default_rng(4).random((B, k)) < 0.6
    zq[agree] = zt[:, :k][agree]
    drafts = zq.argmax(-1)
    ua, uf, _ = synth.uniforms(B, k, 4, "tp0")
    n, out = _run(zt, zq, drafts, ua, uf, gm.GM_SAMPLE, 1.0, 1e-6)
    ng, outg = _run(zt, None, drafts, None, None, gm.GM_GREEDY, 1.0, 1.0)
    np.testing.assert_array_equal(n, ng)
    np.testing.assert_array_equal(out, outg)
    assert 0 < n.mean() < k


def test_top_p_nucleus_handoff():
    # gm_mtp_draft's nuclei handed to gm_spec_accept stand in for the accept's own passes
    # over the draft rows: the same decisions and tokens, bit for bit
    need_gpu()
    from helpers import device_cache
    shape = synth.QWEN3_4B_LAYER
    W, Wm = synth.model_weights(shape), synth.mtp_weights(shape)
    B, k, top_p = 32, 3, 0.7
    g = np.random.default_rng(21)
    lens = g.integers(1, 600, B)
    ks, vs = synth.kv_prefix(shape, lens, layer=500)
    hidden = g.standard_normal((B, k + 1, shape.hidden)).astype(np.float32)
    n0 = g.integers(0, k + 1, B).astype(np.int32)
    out0 = g.integers(0, shape.vocab, (B, k + 1)).astype(np.int32)
    ua, uf, ud = synth.uniforms(B, k, 4, "handoff")
    model, mtp = gm.DeviceModel(shape, W), gm.DeviceMtp(shape, Wm)
    cache = device_cache(shape, [(ks, vs)], lens, 2 * k + 2)
    drafts = torch.zeros((B, k), dtype=torch.int32, device="cuda")
    dlog = torch.zeros((B, k, shape.vocab), dtype=torch.float32, device="cuda")
    nuc = gm.new_nuclei(B, k)
    gm.mtp_draft(model, mtp, cache, k, gm.GM_SAMPLE, t32(hidden), i32(n0), i32(out0), t32(ud), drafts, dlog,
                 gm.Workspace(), top_p=top_p, draft_nucleus=nuc)
    zt = t32(_logits((B, k + 1, shape.vocab), "normal", "handoff-t"))
    res = []
    for handoff in (None, nuc):
        n = torch.zeros(B, dtype=torch.int32, device="cuda")
        out = torch.zeros((B, k + 1), dtype=torch.int32, device="cuda")
        gm.spec_accept(zt, dlog, drafts, t32(ua), t32(uf), n, out, gm.GM_SAMPLE, gm.Workspace(), top_p=top_p,
                       draft_nucleus=handoff)
        torch.cuda.synchronize()
        res.append((n.cpu().numpy(), out.cpu().numpy()))
    np.testing.assert_array_equal(res[0][0], res[1][0])
    np.testing.assert_array_equal(res[0][1], res[1][1])
    # the handed-over nuclei hold the head's own masses: every draft lies in its nucleus
    h = nuc.cpu().numpy().reshape(B, k, 24)
    key = h[..., 16:20].copy().view(np.uint32)[..., 0]
    last = h[..., 20:24].copy().view(np.int32)[..., 0]
    z = dlog.cpu().numpy()
    d = drafts.cpu().numpy()
    zd = np.take_along_axis(z, d[..., None], -1)[..., 0].astype(np.float32)
    u = zd.view(np.uint32)
    okey = np.where(u & 0x80000000, ~u, u | 0x80000000).astype(np.uint32)
    assert ((okey > key) | ((okey == key) & (d <= last))).all()
    print("[top-p handoff] mean accepted %.2f" % res[0][0].mean(), flush=True)


def _head_rows(kinds, B, V, top_p):
    """Logits rows of a confident head, one id holding most of the mass over a floor N(0, 1) (kind, the
    floor's share of the mass), cycling through the kinds."""
    g = synth.stream(3, "head-rows", B, V, top_p)
    rows = np.empty((B, V), np.float32)
    for b in range(B):
        kind, share = kinds[b % len(kinds)]
        r = g.standard_normal(V)
        if kind == "dense":        # the whole floor within a sixteenth of an exponent
            r *= 0.005
        elif kind.startswith("ties"):
            n = float(kind[4:])
            r = np.round(r * n) / n
        r[g.integers(0, V)] = np.log(np.exp(r).sum() * (1.0 - share) / share)
        rows[b] = r
    return rows


@pytest.mark.parametrize("B,V,top_p", [(16, 151936, 0.95), (16, 50257, 0.85), (136, 20000, 0.95), (130, 50256, 0.99)])
def test_top_p_nuclei_of_chosen_rows(B, V, top_p):
    # The nuclei that gm_mtp_draft hands over, id by id, for boundaries among ids too unlikely to be queued:
    # found through the bands of the exponent and gathered ("floor"; with runs of ties ranked in LDS,
    # "ties64", and past that, "ties8"), in a band that overflows the gather ("dense"), and among the queued
    # ids (a floor of a tenth of 1 - top_p).  The first pass is split over blocks in the first two cases.
    # The head passes row b's logits through: a one-hot hidden selects column b of the LM head.
    need_gpu()
    import dataclasses
    from helpers import device_cache
    rest = 1.0 - top_p
    kinds = [("floor", 6 * rest), ("ties64", 5 * rest), ("ties8", 6 * rest), ("dense", 4 * rest), ("floor", 0.1 * rest),
             ("floor", 1.3 * rest)]
    shape = dataclasses.replace(synth.TINY, vocab=V)
    H, k = shape.hidden, 1
    rows = _head_rows(kinds, B, V, top_p)
    lm = np.zeros((V, H), np.float32)
    lm[:, :B] = rows.T / np.float32(16.0)              # RMSNorm of a one-hot of H = 256 channels is 16 at it
    W = dict(embed=np.zeros((V, H), np.float32), final_norm=np.ones(H, np.float32), lm_head=lm, layers=[])
    Wm = dict(synth.mtp_weights(shape))
    Wm["w_proj"] = np.concatenate([np.eye(H, dtype=np.float32), np.zeros((H, H), np.float32)], 1)
    Wm["layer"] = dict(Wm["layer"], wo=np.zeros_like(Wm["layer"]["wo"]), w_down=np.zeros_like(Wm["layer"]["w_down"]))
    lens = np.ones(B, np.int64)
    cache = device_cache(shape, [synth.kv_prefix(shape, lens, layer=7)], lens, 2 * k + 2)
    hidden = np.zeros((B, k + 1, H), np.float32)
    hidden[np.arange(B), :, np.arange(B)] = 1.0
    u = synth.uniforms(B, k, 4, "head-rows", V)[2]
    drafts = torch.zeros((B, k), dtype=torch.int32, device="cuda")
    dlog = torch.zeros((B, k, V), dtype=torch.float32, device="cuda")
    nuc = gm.new_nuclei(B, k)
    gm.mtp_draft(gm.DeviceModel(shape, W), gm.DeviceMtp(shape, Wm), cache, k, gm.GM_SAMPLE, t32(hidden),
                 i32(np.zeros(B)), i32(np.zeros((B, k + 1))), t32(u), drafts, dlog, gm.Workspace(), top_p=top_p,
                 draft_nucleus=nuc)
    torch.cuda.synchronize()
    z, h, x = dlog.cpu().numpy()[:, 0], nuc.cpu().numpy()[:, 0], drafts.cpu().numpy()[:, 0]
    assert np.abs(z - rows).max() < 1e-5
    m, mass = (h[:, o:o + 8].copy().view(np.float64)[:, 0] for o in (0, 8))
    key, last = h[:, 16:20].copy().view(np.uint32)[:, 0], h[:, 20:24].copy().view(np.int32)[:, 0]
    flagged = 0
    for b in range(B):
        kind, share = kinds[b % len(kinds)]
        p = oracle.softmax(z[b].astype(np.float64))
        # the inputs meet the paths they are meant for (the selection queues ids above rest / 2048 of the mass)
        assert (p[p > rest / 2048].sum() < top_p) == (share > rest), (b, kind, share)
        kept, dist = oracle.nucleus(z[b], p, top_p)
        if dist < NUC_EPS:
            flagged += 1
            continue
        bits = z[b].view(np.uint32)
        okey = np.where(bits == 0x80000000, np.uint32(0x80000000),
                        np.where(bits & 0x80000000, ~bits, bits | 0x80000000)).astype(np.uint32)
        got = (okey > key[b]) | ((okey == key[b]) & (np.arange(V) <= last[b]))
        np.testing.assert_array_equal(got, kept > 0, err_msg="%d %s" % (b, kind))
        # each kept id's term is rounded to 2^-44 of the largest
        assert m[b] == z[b].max() and abs(mass[b] - np.exp(z[b][got].astype(np.float64) - m[b]).sum()) < V * 2.0 ** -45 + 1e-12
        assert got[x[b]]
    print("[nuclei of chosen rows B=%d V=%d top-p %.2f] flagged %d" % (B, V, top_p, flagged), flush=True)
    assert flagged <= 0.1 * B


def _chain_flags(zt, zq, d_ref, n_ref, dev, ua, uf, ud, top_p, window):
    """Per sequence, how far the oracle's draft-and-accept chain (at T = 1) stays comparable when
    the GPU's draft logits sit within dev[b, j] (max over the row) of the oracle's.  Walks the examined
    events in order -- draw j, accept test j, then the final draw -- and stops at the first one
    that such a deviation D could move:
      * the draw of d_j from the nucleus of q_j: the nucleus changes if the logit just below its
        boundary lies within 2 D of the boundary's, or its running masses lie within e^{2D} - 1
        (+ 5e-9) of top_p; the inverse-CDF draw moves if u lies within e^{4D} - 1 (+ 1e-6) of an
        edge (each nucleus mass moves by a factor within e^{+-4D});
      * accept test j: |u - min(1, p'/q')| < max(1e-3, 5 D), or p's nucleus within 5e-9 of top_p;
      * the final draw: within window[b] + 8 D / top_p of an edge (residual) or window[b] (bonus).
    Returns per sequence: drawn (leading drafts that must be the oracle's), upto (leading accept
    decisions that must agree), known (the accept count must agree) and whole (every committed
    token must agree)."""
    B, k1, V = zt.shape
    k = k1 - 1
    drawn = np.zeros(B, np.int64)
    upto = np.zeros(B, np.int64)
    known = np.zeros(B, bool)
    whole = np.zeros(B, bool)
    for b in range(B):
        n = int(n_ref[b])
        stopped = False
        for j in range(min(n + 1, k)):
            D = float(dev[b, j])
            qn, dist_n = oracle.nucleus(zq[b, j], oracle.softmax(zq[b, j].astype(np.float64)), top_p)
            zs = np.sort(zq[b, j].astype(np.float32))[::-1]
            m = int((qn > 0).sum())
            gap = zs[m - 1] - zs[m] if m < V else np.inf
            dist_d = oracle.inverse_cdf(qn, ud[b, j])[1]
            if gap < 2 * D or dist_n < np.expm1(2 * D) + 5e-9 or dist_d < np.expm1(4 * D) + 1e-6:
                stopped = True
                break
            drawn[b] = j + 1
            pn, dist_p = oracle.nucleus(zt[b, j], oracle.softmax(zt[b, j].astype(np.float64)), top_p)
            r = min(1.0, pn[d_ref[b, j]] / qn[d_ref[b, j]])
            if dist_p < 5e-9 or abs(float(ua[b, j]) - r) < max(1e-3, 5 * D):
                stopped = True
                break
            upto[b] = min(j + 1, n)
        if stopped:
            continue
        known[b] = True
        pn, dist_p = oracle.nucleus(zt[b, n], oracle.softmax(zt[b, n].astype(np.float64)), top_p)
        if dist_p < 5e-9:
            continue
        if n < k:
            qn = oracle.nucleus(zq[b, n], oracle.softmax(zq[b, n].astype(np.float64)), top_p)[0]
            w = np.maximum(pn - qn, 0.0)
            if not w.sum() > 0:
                w = pn
            lim = window[b] + 8 * float(dev[b, n]) / top_p
        else:
            w, lim = pn, window[b]
        whole[b] = oracle.inverse_cdf(w, uf[b])[1] >= lim
    return drawn, upto, known, whole


def test_top_p_nucleus_handoff_matches_oracle():
    # The whole top-p step with the handoff -- gm_mtp_draft's nuclei, draws and logits taken by
    # gm_spec_accept in place of its own passes over the draft rows -- against the oracle's draft
    # head and accept on the same seeded inputs.  A float32 head over a 151936-id vocabulary
    # whose final norm is scaled by 16 (logits ~ N(0, 5^2): nuclei of tens of ids, so a 1e-5
    # deviation moves few draws) and a target within 0.1 N(0, 1) of the oracle's draft logits
    # (most drafts accepted).  Decisions are compared up to each sequence's first event that the
    # measured logit deviation could move (``_chain_flags``).
    need_gpu()
    import dataclasses
    from helpers import device_cache, EXACT
    shape = dataclasses.replace(synth.TINY, vocab=151936)
    W = synth.model_weights(shape)
    Wm = dict(synth.mtp_weights(shape))
    Wm["final_norm"] = (Wm["final_norm"] * np.float32(16.0)).astype(np.float32)
    B, k, top_p = 32, 3, 0.7
    g = np.random.default_rng(31)
    lens = g.integers(1, 200, B)
    caches = [synth.kv_prefix(shape, lens, layer=131)]
    hidden = g.standard_normal((B, k + 1, shape.hidden)).astype(np.float32)
    n0 = g.integers(0, k + 1, B).astype(np.int32)
    out0 = g.integers(0, shape.vocab, (B, k + 1)).astype(np.int32)
    for b in range(B):
        out0[b, n0[b] + 1:] = -1
    ua, uf, ud = synth.uniforms(B, k, 4, "handoff-f32")
    ref_d = oracle.mtp_draft(shape, Wm, W, caches[0][0], caches[0][1], lens, hidden, n0, out0, ud, k, "sample", 1.0,
                             EXACT, top_p=top_p)
    zq = ref_d["draft_logits"].astype(np.float32)
    noise = synth.normal_logits((B, k + 1, shape.vocab), 31, "handoff-f32-t")
    zt = np.concatenate([zq, np.zeros((B, 1, shape.vocab), np.float32)], 1) + np.float32(0.1) * noise
    zt[:, k] = np.float32(5.0) * noise[:, k]
    zt = zt.astype(np.float32)
    ref = oracle.spec_accept(zt, zq, ref_d["drafts"], ua, uf, top_p=top_p, nucleus_eps=NUC_EPS)

    model, mtp = gm.DeviceModel(shape, W), gm.DeviceMtp(shape, Wm)
    cache = device_cache(shape, caches, lens, 2 * k + 2)
    drafts = torch.zeros((B, k), dtype=torch.int32, device="cuda")
    dlog = torch.zeros((B, k, shape.vocab), dtype=torch.float32, device="cuda")
    nuc = gm.new_nuclei(B, k)
    gm.mtp_draft(model, mtp, cache, k, gm.GM_SAMPLE, t32(hidden), i32(n0), i32(out0), t32(ud), drafts, dlog,
                 gm.Workspace(), top_p=top_p, draft_nucleus=nuc)
    n = torch.zeros(B, dtype=torch.int32, device="cuda")
    out = torch.zeros((B, k + 1), dtype=torch.int32, device="cuda")
    gm.spec_accept(t32(zt), dlog, drafts, t32(ua), t32(uf), n, out, gm.GM_SAMPLE, gm.Workspace(), top_p=top_p,
                   draft_nucleus=nuc)
    torch.cuda.synchronize()
    n, out = n.cpu().numpy(), out.cpu().numpy()
    got_d, got_l = drafts.cpu().numpy(), dlog.cpu().numpy()

    dev = np.abs(got_l.astype(np.float64) - zq).max(-1)          # [B, k]
    drawn, upto, known, whole = _chain_flags(zt, zq, ref_d["drafts"], ref.n_accept, dev, ua, uf, ud, top_p,
                                             draw_window(zt, zq, 1.0, top_p))
    for b in range(B):
        np.testing.assert_array_equal(got_d[b, :drawn[b]], ref_d["drafts"][b, :drawn[b]])
        assert n[b] >= upto[b], (b, n[b], upto[b])
        np.testing.assert_array_equal(out[b, :upto[b]], ref.out_tokens[b, :upto[b]])
        if known[b]:
            assert n[b] == ref.n_accept[b], (b, n[b], ref.n_accept[b])
        if whole[b]:
            np.testing.assert_array_equal(out[b, :n[b] + 1], ref.out_tokens[b, :n[b] + 1])
    examined = np.minimum(ref.n_accept + 1, k)
    print("[top-p handoff vs oracle] logit deviation max %.2e; drafts compared %d, accept decisions compared "
          "%d of %d examined (counts known %d), whole sequences %d of %d; mean accepted %.2f (oracle %.2f)"
          % (dev.max(), drawn.sum(), upto.sum() + (known & (ref.n_accept < k)).sum(), examined.sum(), known.sum(),
             whole.sum(), B, n.mean(), ref.n_accept.mean()), flush=True)
    assert known.sum() >= B // 2 and whole.sum() >= B // 4 and upto.sum() >= B
