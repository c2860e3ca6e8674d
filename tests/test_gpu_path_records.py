"""The records that deep root paths leave (nodes at depth 31 and more, one
kernel per sub-layer): a node with a block in a chunk always writes its own,
whatever the scores hold."""
import numpy as np
import pytest

import oracle
from paper_2308_04623_amd import workloads as W

pytestmark = pytest.mark.gpu

CFG = W.GPT2Config(n_layer=2, d_model=192, n_head=3, d_mlp=352, vocab=515, n_pos=800, dtype="bf16")
NAN_BF16 = 0x7FC0


@pytest.mark.parametrize("lost", [32, 128])
@pytest.mark.parametrize("P", [0, 100])
def test_nan_keys_reach_every_node_below_them(lost, P):
    """The first `lost` nodes of a chain sit at positions whose embedding is NaN,
    so their K and V are: one 32-key block of a chunk, or a whole chunk.  Every
    node's path holds them, so every logit is NaN, also after a pass of the
    session that left finite records."""
    from paper_2308_04623_amd import ssd
    w = W.make_weights(CFG, 3, perturb_affine=True)
    w["wpe"][P:P + lost] = NAN_BF16
    n, ctx, far = 160, 640, 400
    kc, vc = W.random_kv_cache(CFG, ctx, far, seed=3)
    par = W.chain_tree(n)
    toks = W.tree_tokens(par, CFG.vocab, seed=n)
    om = oracle.Model(CFG, w)
    ref = oracle.tree_verify(om, kc, vc, P, toks, par, om.kv(n), om.kv(n))
    assert np.isnan(ref).all()
    s = ssd.Session(ssd.Model(CFG, w), ctx, n, ssd.to_device(kc, CFG), ssd.to_device(vc, CFG))
    assert np.isfinite(s.verify(far, toks, par).cpu().numpy()).all()
    assert np.isnan(s.verify(P, toks, par).cpu().numpy()).all()


@pytest.mark.parametrize("n", [70, 160])
def test_nan_in_the_cache_reaches_every_node(n):
    """Cached rows of NaN: a whole 32-row block, and one row of another chunk."""
    from paper_2308_04623_amd import ssd
    w = W.make_weights(CFG, 3, perturb_affine=True)
    P, ctx = 300, 320
    par = W.branching_tree([4, 2, 2, 1], n)
    toks = W.tree_tokens(par, CFG.vocab, seed=n)
    for rows in (slice(0, 32), slice(270, 271)):
        kc, vc = W.random_kv_cache(CFG, ctx, P, seed=3)
        kc[:, :, rows] = NAN_BF16
        s = ssd.Session(ssd.Model(CFG, w), ctx, n, ssd.to_device(kc, CFG), ssd.to_device(vc, CFG))
        assert np.isnan(s.verify(P, toks, par).cpu().numpy()).all()
