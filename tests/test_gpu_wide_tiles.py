"""Every tile of the wide GEMM (4 or 5 row blocks x 2, 3, 4, 6 or 8 node tiles),
with 16- and 8-bit weights, one k-split and several, against the CPU oracle;
each case names the tiles that its GEMMs take.

Bar: 2e-2 max-abs on logits and K/V, as for every bfloat16 model."""
import numpy as np
import pytest

import oracle
from paper_2308_04623_amd import ssd
from paper_2308_04623_amd import workloads as W

TOL = 2e-2
P, CTX = 40, 64


def shape(d, heads, mlp):
    return W.GPT2Config(n_layer=1, d_model=d, n_head=heads, d_mlp=mlp, vocab=515, n_pos=1200, dtype="bf16")


# (model, nodes, {(GEMM, tile, k-splits)}); GEMM 0 QKV, 1 attention output, 2 MLP up, 3 MLP down
A, B, C, D = shape(128, 4, 5120), shape(128, 4, 3840), shape(256, 8, 1024), shape(1280, 20, 5120)
CASES = [
    (A, 128, {(2, 5, 2, 1), (3, 4, 2, 8)}), (A, 177, {(2, 5, 3, 1), (3, 4, 2, 4)}), (A, 256, {(2, 5, 4, 1)}), (A, 288, {(2, 4, 6, 1)}),
    (A, 350, {(2, 5, 6, 1)}), (A, 480, {(2, 5, 8, 1), (0, 4, 2, 1)}), (B, 500, {(2, 4, 8, 1)}),
    (C, 513, {(0, 4, 3, 1)}), (C, 1024, {(0, 4, 4, 1)}),
    # GPT-2-L's layer: k-splits of the larger tiles
    (D, 400, {(0, 5, 6, 1), (1, 5, 4, 2), (2, 5, 8, 1), (3, 5, 8, 4)}), (D, 111, {(3, 5, 2, 4)}),
]


def tiles(cfg, n, q8):
    d, m = cfg.d_model, cfg.d_mlp
    return {(k, *ssd.wide_tile(k, rows, cols, n, q8)) for k, rows, cols in ((0, 3 * d, d), (1, d, d), (2, m, d), (3, d, m))}


def test_cases_name_every_tile():
    for q8 in (False, True):
        for cfg, n, want in CASES:
            assert want <= tiles(cfg, n, q8), (cfg, n, tiles(cfg, n, q8))
    assert {t[1:3] for _, _, want in CASES for t in want} == {(r, t) for r in (4, 5) for t in (2, 3, 4, 6, 8)}


def test_splits_cut_the_steps_evenly_over_the_xcds():
    """Whatever the sizes, a residual GEMM's k-ranges number 1, 2, 4 or 8; other GEMMs have one."""
    for d in range(32, 2049, 96):
        for K in (32, 64, 96, 160, 320, 352, 1056, 1280, 2976, 5120, 8160):
            for n in (65, 128, 257, 1024):
                S = ssd.wide_tile(3, d, K, n)[2]
                KC = K // 32
                kcs = -(-KC // S)
                assert -(-KC // kcs) in (1, 2, 4, 8)
                assert ssd.wide_tile(2, d, K, n)[2] == 1
    with pytest.raises(ssd.SSDError):
        ssd.wide_tile(0, 128, 128, 64)
    with pytest.raises(ssd.SSDError):
        ssd.wide_tile(5, 128, 128, 65)


def recent_tree(n, back=8):
    g = np.random.default_rng(n)
    return np.array([-1] + [int(g.integers(max(0, i - back), i)) for i in range(1, n)], np.int32)


@pytest.mark.gpu
@pytest.mark.parametrize("q8", [False, True])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_tile_against_oracle(case, q8):
    cfg, n, _ = CASES[case]
    w = W.make_weights(cfg, 3, perturb_affine=True)
    om = oracle.Model(cfg, w, q8=q8)
    kc, vc = W.random_kv_cache(cfg, CTX, P, seed=3)
    par = recent_tree(n)
    toks = W.tree_tokens(par, cfg.vocab, seed=n)
    kt, vt = om.kv(n), om.kv(n)
    ref = oracle.tree_verify(om, kc, vc, P, toks, par, kt, vt)
    s = ssd.Session(ssd.Model(cfg, w, q8=q8), CTX, n, ssd.to_device(kc, cfg), ssd.to_device(vc, cfg))
    assert np.abs(s.verify(P, toks, par).cpu().numpy() - ref).max() < TOL
    for got, want in ((s.k_tree, kt), (s.v_tree, vt)):
        a, b = (W.bf16_bits_to_f32(x) for x in (ssd.to_host_bits(got), want))
        assert np.abs(a - b).max() < TOL
    assert s.error_count() == 0
