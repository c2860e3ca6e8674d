"""The float32 model's GEMM and the sampling helpers at the edges of their
tiles and chunks, against the CPU oracle and host definitions."""
import numpy as np
import pytest

import oracle
from paper_2308_04623_amd import workloads as W
from tests.helpers import host_topk

pytestmark = pytest.mark.gpu


# K of 160 and 1056 (one K step, and two with a remainder), rows and nodes off multiples of 16
@pytest.mark.parametrize("n", [1, 15, 16, 17, 130])
def test_f32_gemm_edges(n):
    from paper_2308_04623_amd import ssd
    cfg = W.GPT2Config(n_layer=2, d_model=160, n_head=5, d_mlp=1056, vocab=515, n_pos=256, dtype="f32")
    w = W.make_weights(cfg, 2, perturb_affine=True)
    P, ctx = 30, 64
    kc, vc = W.random_kv_cache(cfg, ctx, P, seed=3)
    par = W.complete_binary_tree(n)
    toks = W.tree_tokens(par, cfg.vocab, seed=n)
    om = oracle.Model(cfg, w)
    ref = oracle.tree_verify(om, kc, vc, P, toks, par, om.kv(n), om.kv(n))
    s = ssd.Session(ssd.Model(cfg, w), ctx, n, ssd.to_device(kc, cfg), ssd.to_device(vc, cfg))
    # the float32 bar of the other parity tests: sums of up to 1056 terms of size 1 at 6e-8 each stay below it
    assert np.abs(s.verify(P, toks, par).cpu().numpy() - ref).max() < 1e-4


@pytest.fixture(scope="module")
def session():
    from paper_2308_04623_amd import ssd
    cfg = W.GPT2Config(n_layer=1, d_model=64, n_head=2, d_mlp=64, vocab=9000, n_pos=64, dtype="bf16")
    return ssd.Session(ssd.Model(cfg, W.make_weights(cfg, 0)), 0, 64)


# chunks of 2048 ids: one, one full, one id more, several; rows with masked
# (-inf) ids up to whole chunks, one id holding all the mass, and a flat row
@pytest.mark.parametrize("V", [1, 255, 2048, 2049, 8999])
def test_cdf_pick_edges(session, V):
    import torch
    g = np.random.default_rng(V)
    lg = (g.standard_normal((6, V)) * 3).astype(np.float32)
    lg[1, : V // 2] = -np.inf
    lg[2, V // 3:] = -np.inf
    lg[2, 0] = 0.0
    lg[3, :] = -np.inf
    lg[3, V - 1] = 1.5
    lg[4, :] = 0.25
    rows = np.repeat(np.arange(6), 10).astype(np.int32)[g.permutation(60)]
    us = g.random(60)
    us[:6] = [0.0, 1.0 - 2.0 ** -53, 0.5, 2.0 ** -53, 0.25, 0.75]
    got = session.cdf_pick(torch.from_numpy(lg).cuda(), rows, us, 0.7).cpu().numpy()
    assert got.tolist() == [oracle.cdf_pick(lg[r], 0.7, u) for r, u in zip(rows, us)]


@pytest.mark.parametrize("k", [1, 2, 8])
def test_topk_across_chunks(session, k):
    """Every chunk of the row leaves k entries; ties in and across chunks go to the lower id."""
    import torch
    g = np.random.default_rng(k)
    lg = np.round(g.standard_normal((5, 9000)) * 2, 1).astype(np.float32)
    lg[1, 2040:2060] = 50.0
    lg[2, 8192:8200] = 60.0
    idx, val, lse = session.topk(torch.from_numpy(lg).cuda(), k)
    hi, hv, hl = host_topk(lg, k)
    assert np.array_equal(idx.cpu().numpy(), hi) and np.array_equal(val.cpu().numpy(), hv)
    assert np.abs(lse.cpu().numpy() - hl).max() < 1e-5 * np.abs(hl).max() + 1e-5


@pytest.mark.parametrize("V", [131072, 131073, 300000])
def test_topk_chunks_per_lane(V):
    """64 chunks, one a lane of the wave that merges them, and more; k of 1, 3 and the most allowed, the first
    eight of a row in one chunk, in one lane's chunks and anywhere, most of a row -inf, half of one NaN."""
    import torch
    from paper_2308_04623_amd import ssd
    cfg = W.GPT2Config(n_layer=1, d_model=64, n_head=2, d_mlp=64, vocab=V, n_pos=64, dtype="bf16")
    s = ssd.Session(ssd.Model(cfg, W.make_weights(cfg, 0)), 0, 8)
    g = np.random.default_rng(V)
    lg = np.round(g.standard_normal((5, V)) * 2, 1).astype(np.float32)
    lg[1, 2040:2060] = 50.0
    lg[2, 5 * 2048::64 * 2048] = 60.0  # (every chunk of lane 5)
    lg[2, 7 + 5 * 2048::64 * 2048] = 61.0
    lg[3, np.arange(V) % 700 > 0] = -np.inf
    lg[3, V - 1] = 0.0
    lg[4, : V // 2] = np.nan
    for k in (1, 3, 8):
        idx, val, lse = (t.cpu().numpy() for t in s.topk(torch.from_numpy(lg).cuda(), k))
        hi, hv, hl = host_topk(lg[:4], k)
        assert np.array_equal(idx[:4], hi) and np.array_equal(val[:4], hv)
        assert np.abs(lse[:4] - hl).max() < 1e-5 * np.abs(hl).max() + 1e-5
        # (NaN entries are never chosen)
        hi, hv, _ = host_topk(lg[4:, V // 2:], k)
        assert np.array_equal(idx[4:], hi + V // 2) and np.array_equal(val[4:], hv) and np.isnan(lse[4])
