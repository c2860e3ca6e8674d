"""Wide trees (more than 64 nodes, one kernel per sub-layer) against the CPU
oracle, at the edges of the wide GEMM's tiles and of its dispatch: node
counts around multiples of 16 and of every node-tile group, row blocks that no
tile divides, a vocabulary that is no multiple of 4, several k-splits.

Bar: 2e-2 max-abs on logits and K/V, the bfloat16 bar of the other parity
tests (float16 GEMM inputs and bfloat16 K/V, each rounded once)."""
import numpy as np
import pytest

import oracle
from paper_2308_04623_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = 2e-2
P, MAX_CTX = 40, 1100
SHAPES = {
    # 12, 6 and 22 row blocks, 6 and 11 k-steps
    "dh64": W.GPT2Config(n_layer=2, d_model=192, n_head=3, d_mlp=352, vocab=515, n_pos=1200, dtype="bf16"),
    # 48, 16 and 64 row blocks, 8 and 32 k-steps
    "dh32": W.GPT2Config(n_layer=2, d_model=256, n_head=8, d_mlp=1024, vocab=1030, n_pos=1200, dtype="bf16"),
    # enough row blocks that the tile grows with the tree (4 or 5 row blocks x 2, 3, 4, 6 or 8 node tiles)
    "mlp5120": W.GPT2Config(n_layer=1, d_model=128, n_head=4, d_mlp=5120, vocab=515, n_pos=1200, dtype="bf16"),
    "mlp3840": W.GPT2Config(n_layer=1, d_model=128, n_head=4, d_mlp=3840, vocab=515, n_pos=1200, dtype="bf16"),
    "d1280": W.GPT2Config(n_layer=1, d_model=1280, n_head=20, d_mlp=1280, vocab=515, n_pos=1200, dtype="bf16"),
}


def recent_tree(n, back=8):
    """Every node hangs from one of the `back` nodes before it."""
    g = np.random.default_rng(n)
    return np.array([-1] + [int(g.integers(max(0, i - back), i)) for i in range(1, n)], np.int32)


class Side:
    def __init__(self, cfg, q8):
        from paper_2308_04623_amd import ssd
        self.cfg, self.ssd = cfg, ssd
        w = W.make_weights(cfg, 3, perturb_affine=True)
        self.om = oracle.Model(cfg, w, q8=q8)
        self.kc, self.vc = W.random_kv_cache(cfg, MAX_CTX, P, seed=3)
        self.m = ssd.Model(cfg, w, q8=q8)

    def check(self, par, prefix):
        n, cfg, ssd = len(par), self.cfg, self.ssd
        toks = W.tree_tokens(par, cfg.vocab, seed=n)
        kt, vt = self.om.kv(n), self.om.kv(n)
        ref = oracle.tree_verify(self.om, self.kc, self.vc, prefix, toks, par, kt, vt)
        s = ssd.Session(self.m, MAX_CTX, n, ssd.to_device(self.kc, cfg), ssd.to_device(self.vc, cfg))
        lg = s.verify(prefix, toks, par).cpu().numpy()
        assert np.abs(lg - ref).max() < TOL
        for got, want in ((s.k_tree, kt), (s.v_tree, vt)):
            a, b = (W.bf16_bits_to_f32(x) for x in (ssd.to_host_bits(got), want))
            assert np.abs(a - b).max() < TOL
        assert s.error_count() == 0


@pytest.fixture(scope="module")
def sides():
    cache = {}

    def get(name, q8):
        if (name, q8) not in cache:
            cache[name, q8] = Side(SHAPES[name], q8)
        return cache[name, q8]
    return get


# node-tile groups full, ragged and of one node
@pytest.mark.parametrize("name,n", [(s, n) for s in ("dh64", "dh32")
                                    for n in (65, 80, 97, 128, 129, 177, 256, 257, 400, 513, 1024)]
                         + [("mlp5120", n) for n in (80, 128, 177, 256, 288, 350, 513)]
                         + [("mlp3840", 500), ("d1280", 111), ("d1280", 336)])
def test_wide_pass_against_oracle(sides, name, n):
    sides(name, False).check(recent_tree(n), P)


@pytest.mark.parametrize("n", [65, 129, 257])
def test_wide_pass_8bit_against_oracle(sides, n):
    sides("dh32", True).check(recent_tree(n), P)
