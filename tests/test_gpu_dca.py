"""GPU parity of gm_dca_loss (the DCA loss with verify-gated masking over the
cycle record's top-k support plus a residual bin, and its gradient in the head
logits) against the oracle on the same seeded inputs: loss and alpha within
1e-6 relative (both are float64 sums of the same float32 logits), the gradient
within 1e-5 of its largest entry (float32 on the GPU)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from helpers import need_gpu, t32, i32
from paper_2609_16648_amd import gm

pytestmark = pytest.mark.gpu


def _inputs(N, K, V, topk, seed):
    g = np.random.default_rng(seed)
    zt = synth.normal_logits((N, K + 1, V), 3, "dca", N, K, V) * np.float32(2.0)
    zq = (zt[:, :K] + g.standard_normal((N, K, V)).astype(np.float32)).astype(np.float32)
    ids, logp = oracle.record_topk(zt, K, 1.0, topk)
    n = g.integers(0, K + 1, N)
    return zq, ids, logp, n


def _gpu(zq, ids, logp, n, vgm, with_grad=True):
    N, K, V = zq.shape
    topk = ids.shape[-1]
    loss = torch.zeros(N, dtype=torch.float32, device="cuda")
    alpha = torch.zeros((N, K), dtype=torch.float32, device="cuda")
    grad = torch.full((N, K, V), 7.0, dtype=torch.float32, device="cuda") if with_grad else None
    lp = torch.from_numpy(logp.astype(np.float32)).to("cuda").to(torch.bfloat16)   # bf16 values: exact
    gm.dca_loss(t32(zq), lp, i32(ids), i32(n), loss, alpha, grad, gm.Workspace(), vgm=vgm)
    torch.cuda.synchronize()
    return loss.cpu().numpy(), alpha.cpu().numpy(), grad.cpu().numpy() if with_grad else None


@pytest.mark.parametrize("N,K,V,topk,vgm", [(16, 3, 151936, 64, True), (16, 3, 151936, 64, False),
                                            (24, 3, 151936, 32, False),   # unmasked, 72 rows, past the L2s
                                            (8, 7, 20000, 64, True), (33, 1, 1000, 16, True), (5, 2, 64, 64, True),
                                            # rows past one gradient block by one id (and off 16 bytes), by four
                                            (6, 4, 4097, 33, True), (6, 3, 8196, 64, True)])
def test_dca_matches_oracle(N, K, V, topk, vgm):
    need_gpu()
    zq, ids, logp, n = _inputs(N, K, V, topk, N + K + V)
    loss, alpha, grad = _gpu(zq, ids, logp, n, vgm)
    rl, ra, rg = oracle.dca_loss(zq, ids, logp, n, vgm)
    np.testing.assert_allclose(alpha, ra, rtol=1e-6, atol=1e-7)
    np.testing.assert_allclose(loss, rl, rtol=1e-6, atol=1e-7)
    err = np.abs(grad - rg).max() / np.abs(rg).max()
    print("[dca N=%d K=%d V=%d top%d vgm=%d] loss %.4f, grad rel err %.2e" % (N, K, V, topk, vgm, rl.mean(), err),
          flush=True)
    assert err < 1e-5
    if vgm:   # positions past the first rejection get no gradient
        for b in range(N):
            assert (grad[b, min(int(n[b]) + 1, K):] == 0).all()


@pytest.mark.parametrize("N,K,V,off", [(9, 2, 50257, 0), (6, 3, 8196, 1), (5, 1, 4099, 3), (16, 3, 30000, 2),   # small
                                       (40, 5, 50257, 0), (41, 5, 50256, 0), (41, 5, 50256, 1),                 # medium
                                       (700, 2, 50257, 0), (1400, 1, 50256, 0), (1400, 1, 50256, 3)])           # large
def test_dca_gradient_paths(N, K, V, off):
    # gradients up to 32 MB, below 256 MB and above, rows on 16-byte boundaries and off them (an odd vocabulary,
    # buffers `off` floats past one); NaN in the logits past the first rejection stays out of the gradient
    need_gpu()
    g = torch.Generator(device="cuda").manual_seed(N + V + off)
    buf = lambda: torch.empty(N * K * V + 4, device="cuda")[off:off + N * K * V].view(N, K, V)
    z, grad = buf(), buf()
    z.normal_(generator=g).mul_(2.0)
    ids = torch.rand((N, K, V), device="cuda", generator=g).topk(16, -1).indices.to(torch.int32).contiguous()
    lp = torch.log_softmax(torch.rand((N, K, 17), device="cuda", generator=g) * 4.0, -1)[..., :16].contiguous()
    lp = lp.to(torch.bfloat16)
    n = torch.randint(0, K + 1, (N,), generator=g, device="cuda", dtype=torch.int32)
    past = torch.arange(K, device="cuda")[None, :] > n[:, None]
    some = np.unique(np.r_[0:8, N // 2:N // 2 + 8, max(N - 8, 0):N] % N)
    zs, ids_s, lp_s, n_s = (t[torch.from_numpy(some).cuda()].cpu() for t in (z, ids, lp.float(), n))
    z[past] = float("nan")
    grad.fill_(7.0)
    loss = torch.zeros(N, dtype=torch.float32, device="cuda")
    alpha = torch.zeros((N, K), dtype=torch.float32, device="cuda")
    gm.dca_loss(z, lp, ids, n, loss, alpha, grad, gm.Workspace(), vgm=True)
    torch.cuda.synchronize()
    assert (grad[past] == 0).all() and torch.isfinite(grad).all()
    rl, _, rg = oracle.dca_loss(zs.numpy(), ids_s.numpy(), lp_s.numpy().astype(np.float64), n_s.numpy(), True)
    np.testing.assert_allclose(loss.cpu().numpy()[some], rl, rtol=1e-6, atol=1e-7)
    got = grad[torch.from_numpy(some).cuda()].cpu().numpy()
    assert np.abs(got - rg).max() < 1e-5 * np.abs(rg).max()


def test_dca_without_gradient_and_on_the_accepts_own_record():
    # the record taken by gm_spec_accept feeds the loss directly
    need_gpu()
    N, K, V = 24, 3, 151936
    zt = synth.normal_logits((N, K + 1, V), 3, "dca2", N, K, V) * np.float32(2.0)
    zq = (zt[:, :K] + np.random.default_rng(2).standard_normal((N, K, V)).astype(np.float32)).astype(np.float32)
    rec_lp = torch.zeros((N, K, 64), dtype=torch.bfloat16, device="cuda")
    rec_id = torch.zeros((N, K, 64), dtype=torch.int32, device="cuda")
    n = torch.zeros(N, dtype=torch.int32, device="cuda")
    out = torch.zeros((N, K + 1), dtype=torch.int32, device="cuda")
    drafts = np.argmax(zq, -1)
    gm.spec_accept(t32(zt), None, i32(drafts), None, None, n, out, gm.GM_GREEDY, gm.Workspace(), record=(rec_lp, rec_id))
    torch.cuda.synchronize()
    ids, logp, na = rec_id.cpu().numpy(), rec_lp.float().cpu().numpy().astype(np.float64), n.cpu().numpy()
    loss, alpha, _ = _gpu(zq, ids, logp, na, True, with_grad=False)
    rl, ra, _ = oracle.dca_loss(zq, ids, logp, na, True)
    np.testing.assert_allclose(alpha, ra, rtol=1e-6, atol=1e-7)
    np.testing.assert_allclose(loss, rl, rtol=1e-6, atol=1e-7)
