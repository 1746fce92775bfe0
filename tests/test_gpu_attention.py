"""GPU parity of gm_verify_attention against the oracle's grouped causal
attention on the same seeded Q and KV (bf16 within 2e-2 relative error,
float32 within 1e-4), across ragged contexts, block lengths and page sizes."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
import synth
from helpers import need_gpu, rel_err, t32, i32
from paper_2609_16648_amd import gm, layout

pytestmark = pytest.mark.gpu


def _case(shape, lens, k, page_size, seed):
    B, R = len(lens), k + 1
    ctx = np.asarray(lens) + R
    ks, vs = synth.kv_prefix(shape, ctx, layer=seed, seed=2)
    q = synth.normal_tensor((B, R, shape.n_heads, shape.head_dim), 5, shape.dtype, "q", seed)
    cache = gm.PagedCache(shape, 1, lens, ctx, page_size=page_size, seed=seed, fill="empty")
    for b in range(B):
        cache.write(0, b, np.arange(ctx[b]), ks[b], vs[b])
    dt = gm.torch_dtype(shape)
    qd = t32(q, dt)
    out = torch.empty_like(qd)
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    gm.verify_attention(gm.model_config(shape), cache, 0, qd, out, gm.Workspace(), err)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy()
    ref = np.stack([oracle.attention(q[b].astype(np.float64), ks[b].astype(np.float64), vs[b].astype(np.float64),
                                     lens[b] + np.arange(R) + 1) for b in range(B)])
    assert int(err.item()) == 0
    return got, ref, cache


@pytest.mark.parametrize("lens,k,page_size", [
    ([1, 15, 16, 17, 100, 1023, 2500, 4096], 3, 16),
    ([5, 333, 2049, 4000], 3, 64),
    ([7, 300, 3001], 0, 16),
    ([1, 64, 1000], 15, 32),
    ([0, 3, 40], 1, 16),
])
def test_bf16_attention_matches_oracle(lens, k, page_size):
    need_gpu()
    shape = synth.QWEN3_4B_LAYER
    got, ref, _ = _case(shape, np.array(lens), k, page_size, seed=len(lens) + k)
    e = rel_err(got, ref)
    print("[attention bf16 k=%d] rel err %.3e" % (k, e), flush=True)
    assert e < 2e-2
    # the only bf16 rounding left is the output's: agreement to one bf16 step
    assert np.abs(got - oracle.round_bf16(ref)).max() <= 2.0 ** -7 * np.abs(ref).max()


def test_bf16_attention_long_context():
    need_gpu()
    shape = synth.QWEN3_4B_LAYER
    lens = synth.context_lengths(synth.WORKLOADS["long_ctx"])[:3]
    got, ref, _ = _case(shape, lens, 7, 16, seed=11)
    e = rel_err(got, ref)
    print("[attention bf16 long] lens %s rel err %.3e" % (list(lens), e), flush=True)
    assert e < 2e-2


@pytest.mark.parametrize("lens,k,page_size", [
    ([20000] + [0, 17, 1] * 100, 0, 32),    # more sequences than threads of a workgroup, many in one range
    ([3] * 256, 3, 16),                     # one tile each: fewer tiles than workgroups times heads
    ([500, 0, 0, 9000, 31], 1, 16),
])
def test_bf16_attention_many_sequences(lens, k, page_size):
    need_gpu()
    shape = dataclasses.replace(synth.QWEN3_4B_LAYER, n_heads=12, n_kv_heads=6)   # a head group with spare waves
    got, ref, _ = _case(shape, np.array(lens), k, page_size, seed=41 + k)
    assert np.abs(got - oracle.round_bf16(ref)).max() <= 2.0 ** -7 * np.abs(ref).max()


def _long_case(lens, k, heads):
    """Verify attention over N(0, 1) pools with 40 KV heads: ten head groups, so a range (of 25 on 256
    CUs) holds a fortieth of the tiles of all sequences.  Returns the GPU's rows and the float64
    inputs of the given heads, per sequence: (got, q, k, v, visible tokens)."""
    shape = dataclasses.replace(synth.QWEN3_4B_LAYER, n_heads=40, n_kv_heads=40)
    lens = np.array(lens)
    cache = gm.PagedCache(shape, 1, lens, lens + k + 1, page_size=16, seed=3, fill="empty")
    for t in cache.k + cache.v:
        t.normal_(generator=torch.Generator(device="cuda").manual_seed(5))
    q = synth.normal_tensor((len(lens), k + 1, 40, 128), 5, "bf16", "q-window")
    out = torch.empty(q.shape, dtype=torch.bfloat16, device="cuda")
    gm.verify_attention(gm.model_config(shape), cache, 0, t32(q, torch.bfloat16), out, gm.Workspace())
    torch.cuda.synchronize()
    for b, m in enumerate(lens):
        kv = []
        for which in ("k", "v"):
            page, elem = layout.element_index(np.arange(m + k + 1), cache.block_table_host[b], 16, 128, which)
            pool = cache._pool(0, which)
            kv.append(pool[torch.from_numpy(page).cuda()[:, None, None], torch.tensor(heads).cuda()[None, :, None],
                           torch.from_numpy(elem).cuda()[:, None, :]].float().cpu().numpy().astype(np.float64))
        yield (out[b][:, heads].float().cpu().numpy(), q[b][:, heads].astype(np.float64), kv[0], kv[1],
               m + np.arange(k + 1) + 1)


def _row_err(got, ref):      # the largest error of a (row, head) in the 2-norm, relative to its result
    return (np.linalg.norm(got - ref, axis=-1) / np.linalg.norm(ref, axis=-1)).max()


# The output's rounding to bf16 is at most 2^-9 of each value; everything before it is float32 or carries
# 16 bits of the weights.  A tile of 16 tokens lost or counted twice moves a row over 60000 tokens by 1 to 2%.
LONG_TOL = 2.0 ** -8


def test_bf16_attention_sequences_after_a_window():
    # ranges of more tiles than a window of the page list: sequences 0 and 2 run on from window to window
    # and range to range, the short ones begin in the later windows behind a sequence that began before them
    need_gpu()
    lens = [60000, 300, 50000, 17, 40]
    for b, (got, q, k, v, vis) in enumerate(_long_case(lens, 1, [0, 17, 39])):
        ref = oracle.attention(q, k, v, vis)
        e = _row_err(got, ref)
        print("[attention windows] sequence %d of %d tokens: rel err %.2e" % (b, lens[b], e), flush=True)
        assert e < LONG_TOL, b
        if b == 0:          # the bound sees a single lost tile, here the one behind the first window
            lost = np.r_[0:16 * 256, 16 * 257:len(k)]
            assert _row_err(oracle.attention(q, k[lost], v[lost], vis - 16), ref) > 2 * LONG_TOL


@pytest.mark.parametrize("tiles", [1, 2, 3, 4, 5, 6, 7, 8, 127, 129, 256, 257, 258, 260])
def test_bf16_attention_tiles_per_range(tiles):
    # the ring's turns and the tiles behind them, at every remainder, and windows of one to four tiles
    need_gpu()
    for got, q, k, v, vis in _long_case([16 * 25 * tiles - 2], 1, [5, 38]):
        assert _row_err(got, oracle.attention(q, k, v, vis)) < LONG_TOL


class _Guarded(gm.Workspace):
    """Hands out exactly the bytes that are asked for, in front of a guard."""
    GUARD = 1 << 20

    def get(self, nbytes):
        self.n = nbytes
        self.buf = torch.full((nbytes + self.GUARD,), 0xA5, dtype=torch.uint8, device="cuda")
        return self.buf[:nbytes]


@pytest.mark.parametrize("lens,k", [([9000] * 3, 7), ([700] * 150, 3), ([40] * 600, 0), ([30000], 1)])
def test_bf16_attention_stays_in_its_workspace(lens, k):
    # sequences at the context bound, cut over as many ranges as there are: nothing past the reported size
    need_gpu()
    shape, lens = synth.QWEN3_4B_LAYER, np.array(lens)
    cache = gm.PagedCache(shape, 1, lens, lens + k + 1, page_size=16, seed=1)
    q = torch.randn((len(lens), k + 1, shape.n_heads, 128), device="cuda").to(torch.bfloat16)
    ws, out = _Guarded(), torch.empty_like(q)
    gm.verify_attention(gm.model_config(shape), cache, 0, q, out, ws)
    torch.cuda.synchronize()
    assert (ws.buf[ws.n:] == 0xA5).all() and (ws.buf[:ws.n] != 0xA5).any()
    assert (out == 0).all()                      # zero values, whatever the weights


def test_f32_attention_matches_oracle():
    need_gpu()
    shape = synth.TINY
    got, ref, _ = _case(shape, np.array([1, 20, 128, 131]), 3, 16, seed=4)
    e = rel_err(got, ref)
    print("[attention f32] rel err %.3e" % e, flush=True)
    assert e < 1e-4


@pytest.mark.parametrize("head_dim,n_kv,page_size,lens,k", [
    (64, 4, 16, [0, 1, 15, 60, 61, 62, 253, 254, 255], 2),     # edges of 16-token tiles, 64-token chunks, the 4 waves
    (128, 2, 32, [0, 63, 192, 256, 700, 1029], 1),             # two channels per lane, GQA, several rounds
])
def test_f32_attention_chunk_edges(head_dim, n_kv, page_size, lens, k):
    need_gpu()
    shape = dataclasses.replace(synth.TINY, head_dim=head_dim, n_kv_heads=n_kv)
    got, ref, _ = _case(shape, np.array(lens), k, page_size, seed=31 + head_dim)
    # a score is a float32 sum of head_dim products of N(0, 1) values over sqrt(head_dim): its error
    # is below head_dim * 2^-24 * (a few) = 2e-5, which moves each weight by as much, relatively
    assert rel_err(got, ref) < 2e-5


@pytest.mark.parametrize("bad", [(0, 64), (64, 128), (5, 6), (0, 202)])   # whole chunks of a wave, one token, all
def test_f32_attention_nan_scores_reach_the_row(bad):
    need_gpu()
    shape, lens, R = synth.TINY, np.array([200]), 2
    ctx = lens + R
    ks, vs = synth.kv_prefix(shape, ctx, layer=9, seed=2)
    ks[0] = np.array(ks[0])
    ks[0][bad[0]:bad[1], 1] = np.nan                # head 1 only
    q = synth.normal_tensor((1, R, shape.n_heads, shape.head_dim), 5, shape.dtype, "q-nan")
    cache = gm.PagedCache(shape, 1, lens, ctx, page_size=16, fill="empty")
    cache.write(0, 0, np.arange(ctx[0]), ks[0], vs[0])
    out = torch.empty(q.shape, dtype=torch.float32, device="cuda")
    gm.verify_attention(gm.model_config(shape), cache, 0, t32(q), out, gm.Workspace())
    torch.cuda.synchronize()
    ref = oracle.attention(q[0].astype(np.float64), ks[0].astype(np.float64), vs[0].astype(np.float64),
                           lens[0] + np.arange(R) + 1)
    assert np.isnan(ref[:, 1]).all() and np.isfinite(ref[:, [0, 2, 3]]).all()
    np.testing.assert_allclose(out[0].cpu().numpy(), ref, rtol=0, atol=2e-5 * np.abs(ref[:, 0]).max())


def test_gqa_group_of_eight_and_odd_rows():
    # 32 query heads on 4 KV heads with k = 2: 24 rows in two 16-row tiles
    need_gpu()
    shape = dataclasses.replace(synth.QWEN3_4B_LAYER, n_kv_heads=4)
    got, ref, _ = _case(shape, np.array([9, 700, 1600]), 2, 16, seed=21)
    assert rel_err(got, ref) < 2e-2


def test_bad_page_sets_device_error():
    need_gpu()
    shape = synth.QWEN3_4B_LAYER
    lens = np.array([40, 40])
    cache = gm.PagedCache(shape, 1, lens, lens + 4, page_size=16, seed=1)
    bt = cache.block_table_host.copy()
    bt[1, 1] = -1                                  # a hole inside sequence 1's context
    cache.block_table.copy_(torch.from_numpy(bt))
    q = torch.zeros((2, 4, shape.n_heads, 128), dtype=torch.bfloat16, device="cuda")
    out = torch.empty_like(q)
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    gm.verify_attention(gm.model_config(shape), cache, 0, q, out, gm.Workspace(), err)
    torch.cuda.synchronize()
    assert int(err.item()) & gm.GM_DEVERR_PAGE
    assert torch.isfinite(out.float()).all()
