"""The persistent pass at the node counts where its instance changes: one node
(the LayerNorm row and the attention merge in every workgroup), the counts
around 16, 32 and 48 nodes (one to four tiles), from the embedding and from a
later layer, 16- and 8-bit weights.

Bar: 2e-2 max-abs on logits and K/V (float16 GEMM inputs and bfloat16 K/V,
each rounded once); passes from a later layer equal the full pass bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2308_04623_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = 2e-2
CTX = 600
# 5 heads: some XCDs without heads, 12 or 8 more row blocks than ranks in the MLP
CFG = W.GPT2Config(n_layer=3, d_model=320, n_head=5, d_mlp=1280, vocab=1003, n_pos=700, dtype="bf16")
# d above 1024: two column groups per thread in the LayerNorm
CFG_D = W.GPT2Config(n_layer=2, d_model=1088, n_head=17, d_mlp=1088, vocab=515, n_pos=700, dtype="bf16")


class Side:
    def __init__(self, cfg, q8):
        from paper_2308_04623_amd import ssd
        self.cfg, self.ssd = cfg, ssd
        self.w = W.make_weights(cfg, 5, perturb_affine=True)
        self.om = oracle.Model(cfg, self.w, q8=q8)
        self.kc, self.vc = W.random_kv_cache(cfg, CTX, 513, seed=3)
        self.m = ssd.Model(cfg, self.w, q8=q8)

    def session(self, model=None, kv=None):
        ssd, cfg = self.ssd, self.cfg
        kv = kv or (ssd.to_device(self.kc, cfg), ssd.to_device(self.vc, cfg))
        s = ssd.Session(model or self.m, CTX, 64, *kv)
        s.set_options(pass_mode=ssd.PASS_FUSED)
        return s


@pytest.fixture(scope="module")
def sides():
    made = {}

    def get(cfg, q8):
        if (cfg, q8) not in made:
            made[cfg, q8] = Side(cfg, q8)
        return made[cfg, q8]
    return get


@pytest.mark.parametrize("n", [1, 2, 16, 17, 32, 33, 47, 48, 49, 64])
@pytest.mark.parametrize("P", [0, 255, 513])
@pytest.mark.parametrize("cfg,q8", [(CFG, False), (CFG, True), (CFG_D, False)], ids=["f16", "q8", "d1088"])
def test_instances_against_oracle(sides, cfg, q8, n, P):
    side = sides(cfg, q8)
    par = W.branching_tree([2, 3, 2], n)
    toks = W.tree_tokens(par, cfg.vocab, seed=n + P)
    kt, vt = side.om.kv(64), side.om.kv(64)
    ref = oracle.tree_verify(side.om, side.kc, side.vc, P, toks, par, kt, vt)
    s = side.session()
    lg = s.verify(P, toks, par)
    assert np.abs(lg.cpu().numpy() - ref).max() < TOL
    for got, want in ((s.k_tree, kt), (s.v_tree, vt)):
        a, b = (W.bf16_bits_to_f32(x)[:, :, :n] for x in (side.ssd.to_host_bits(got), want))
        assert np.abs(a - b).max() < TOL
    again = s.verify(P, toks, par)
    assert np.array_equal(lg.cpu().numpy(), again.cpu().numpy())
    assert s.error_count() == 0


@pytest.mark.parametrize("n", [1, 33, 48])
@pytest.mark.parametrize("q8", [False, True])
def test_instances_from_a_later_layer(sides, q8, n):
    side = sides(CFG, q8)
    P = 300
    par = W.branching_tree([2, 3, 2], n)
    toks = W.tree_tokens(par, CFG.vocab, seed=n)
    o = side.session()
    d = side.session(side.m.prefix_view(2), (o.k_cache[:2], o.v_cache[:2]))
    full = o.verify(P, toks, par).cpu().numpy()
    d.verify(P, toks, par)
    x = d.reuse_into(o, np.arange(n))
    assert np.array_equal(o.verify_from(P, toks, par, 2, x).cpu().numpy(), full)
    assert o.error_count() == 0 and d.error_count() == 0


def test_one_node_equals_the_root_of_a_tree(sides):
    """A lone node's logits are those of the same root under 20 more nodes, bit for bit."""
    side = sides(CFG, False)
    par = W.branching_tree([4, 4], 21)
    toks = W.tree_tokens(par, CFG.vocab, seed=2)
    s = side.session()
    for P in (0, 200, 513):
        tree = s.verify(P, toks, par)[0].cpu().numpy()
        assert np.array_equal(s.verify(P, toks[:1], par[:1])[0].cpu().numpy(), tree)
