"""Deep root paths keep float32 queries and softmax weights (nodes at depth 31
and more, one kernel per sub-layer): scores that are small differences of
large products, which 16 bits of a query would blur.

The model is built so that nothing but the attention rounds before it: rows of
x are balanced +-1 and epsilon is 1e-12, so LayerNorm's output is exactly +-1;
W_q and W_k have integer entries, so float32 sums give q and k exactly, and k
has few enough bits for bfloat16.  Dimensions come in pairs: k's two are
opposite, and q's two differ in three weights by one unit of some 200, so a
score is the sum of products some 1000 times larger than itself."""
import numpy as np
import pytest

import oracle
from paper_2308_04623_amd import workloads as W

pytestmark = pytest.mark.gpu


def paired_model(dh, seed):
    d, H = 192, 192 // dh
    cfg = W.GPT2Config(n_layer=1, d_model=d, n_head=H, d_mlp=64, vocab=257, n_pos=400, dtype="bf16", ln_eps=1e-12)
    g = np.random.default_rng(seed)
    bits = W.f32_to_bf16_bits
    w = W.make_weights(cfg, seed)
    wte = np.ones((cfg.vocab, d), np.float32)
    for row in wte:
        row[g.permutation(d)[:d // 2]] = -1
    w["wte"], w["wpe"] = bits(wte), bits(np.zeros((cfg.n_pos, d), np.float32))
    wq = (g.integers(129, 255, (d, d)) * g.choice([-1, 1], (d, d))).astype(np.float32)
    wk = np.zeros((d, d), np.float32)
    for i in range(0, d, 2):
        wq[i + 1] = wq[i]
        wq[i + 1, g.permutation(d)[:3]] += 1
        wk[i, g.permutation(d)[:5]] = g.choice([-1, 1], 5)
        wk[i + 1] = -wk[i]
    wv = g.standard_normal((d, d)).astype(np.float32) * 0.1
    w["w_qkv"][0] = bits(np.concatenate([wq, wk, wv]))
    w["w_o"][0] = bits(g.standard_normal((d, d)).astype(np.float32) * 0.2)
    w["w_fc"][0] = np.zeros_like(w["w_fc"][0])
    w["w_pr"][0] = np.zeros_like(w["w_pr"][0])
    return cfg, w


@pytest.mark.parametrize("dh", [32, 64])
@pytest.mark.parametrize("n", [128, 300])
def test_scores_of_cancelling_products(dh, n):
    from paper_2308_04623_amd import ssd
    cfg, w = paired_model(dh, 5)
    par = W.chain_tree(n)
    toks = W.tree_tokens(par, cfg.vocab, seed=n)
    om = oracle.Model(cfg, w)
    ref = oracle.tree_verify(om, W.empty_kv(cfg, 1), W.empty_kv(cfg, 1), 0, toks, par, om.kv(n), om.kv(n))
    s = ssd.Session(ssd.Model(cfg, w), 0, n)
    got = s.verify(0, toks, par).cpu().numpy().astype(np.float64)
    deep = slice(31, None)
    err = np.linalg.norm(got[deep] - ref[deep]) / np.linalg.norm(ref[deep])
    # Products of up to q k / sqrt(dh) = 11511 x 5 / 5.7, their sums rounded in float32 (2^-24 each), put a weight off
    # by some 1e-3; the attention's output and the last LayerNorm's round to float16 (2.4e-4 each); 2.8e-4 of the logits
    # seen.  Sixteen bits of q, emulated in float64, leave 6.5e-3 to 7.1e-3.
    assert err < 2e-3
