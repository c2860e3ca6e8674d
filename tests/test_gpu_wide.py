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
    # enough row blocks that the tile grows with the tree (to 4 x 8 and 5 x 6; every tile by name: test_gpu_wide_tiles)
    "mlp5120": W.GPT2Config(n_layer=1, d_model=128, n_head=4, d_mlp=5120, vocab=515, n_pos=1200, dtype="bf16"),
    "mlp3840": W.GPT2Config(n_layer=1, d_model=128, n_head=4, d_mlp=3840, vocab=515, n_pos=1200, dtype="bf16"),
    "d1280": W.GPT2Config(n_layer=1, d_model=1280, n_head=20, d_mlp=1280, vocab=515, n_pos=1200, dtype="bf16"),
}


def recent_tree(n, back=8):
    """Every node hangs from one of the `back` nodes before it."""
    g = np.random.default_rng(n)
    return np.array([-1] + [int(g.integers(max(0, i - back), i)) for i in range(1, n)], np.int32)


class Side:
    def __init__(self, cfg, q8, MAX_CTX=MAX_CTX, P=P):
        from paper_2308_04623_amd import ssd
        self.cfg, self.ssd, self.ctx = cfg, ssd, MAX_CTX
        w = W.make_weights(cfg, 3, perturb_affine=True)
        self.om = oracle.Model(cfg, w, q8=q8)
        self.kc, self.vc = W.random_kv_cache(cfg, MAX_CTX, P, seed=3)
        self.m = ssd.Model(cfg, w, q8=q8)

    def check(self, par, prefix):
        n, cfg, ssd = len(par), self.cfg, self.ssd
        toks = W.tree_tokens(par, cfg.vocab, seed=n)
        kt, vt = self.om.kv(n), self.om.kv(n)
        ref = oracle.tree_verify(self.om, self.kc, self.vc, prefix, toks, par, kt, vt)
        s = ssd.Session(self.m, self.ctx, n, ssd.to_device(self.kc, cfg), ssd.to_device(self.vc, cfg))
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


# root paths around full 32-entry blocks and 128-entry chunks: chains (one
# block for a whole 16-node tile), a comb whose tiles hold two paths, and
# four interleaved chains (a tile's nodes in four different blocks)
def comb(n):
    return np.array([-1] + [i - 1 if i % 2 else max(0, i - 2) for i in range(1, n)], np.int32)


def chains(n, k=4):
    return np.array([-1] + [max(0, i - k) for i in range(1, n)], np.int32)


DEEP = {"chain": W.chain_tree, "comb": comb, "chains": chains}


@pytest.mark.parametrize("tree,n", [("chain", 65), ("chain", 128), ("chain", 129), ("chain", 161), ("chain", 600),
                                    ("comb", 140), ("chains", 300), ("chains", 1000)])
@pytest.mark.parametrize("name", ["dh64", "dh32"])
@pytest.mark.parametrize("prefix", [0, P])
def test_deep_root_paths_against_oracle(sides, name, tree, n, prefix):
    sides(name, False).check(DEEP[tree](n), prefix)


# prefixes around the 32-row blocks and the 8 waves of the tile kernel, then on
# both sides of the length where the prefix is shared out over more workgroups
@pytest.mark.parametrize("prefix", [1, 31, 32, 33, 256, 257, 777, 4096, 4097, 4300])
@pytest.mark.parametrize("name", ["dh64", "dh32"])
def test_prefix_lengths_against_oracle(prefix, name):
    side = Side(SHAPES[name].with_(n_pos=4500), False, MAX_CTX=4301, P=prefix)
    side.check(recent_tree(81), prefix)
    if prefix >= 4096:
        side.check(comb(140), prefix)


def test_deep_node_independent_of_its_tree(sides):
    """The last node of a 100-node chain has the same logits, bit for bit, when
    the chain is interleaved with three others in the same 16-node tiles."""
    side = sides("dh64", False)
    cfg, ssd = side.cfg, side.ssd
    n, k = 400, 4
    par = chains(n, k)
    toks = W.tree_tokens(par, cfg.vocab, seed=1)
    path, i = [], n - 1
    while i != -1:
        path.append(i)
        i = int(par[i])
    path = path[::-1]
    s = ssd.Session(side.m, MAX_CTX, n, ssd.to_device(side.kc, cfg), ssd.to_device(side.vc, cfg))
    a = s.verify(P, toks, par)[n - 1].cpu().numpy()
    # (padded with leaves of the root to the same node count: the k-splits of the GEMMs follow the node count)
    cpar = np.concatenate([W.chain_tree(len(path)), np.zeros(n - len(path), np.int32)])
    ctoks = np.concatenate([toks[path], toks[:n - len(path)]])
    b = s.verify(P, ctoks, cpar)[len(path) - 1].cpu().numpy()
    assert np.array_equal(a, b)


def test_commit_of_a_long_path_and_of_unaligned_buffers(sides):
    """Committed rows are the tree rows, bit for bit, and no other row of the
    cache changes: a long path, and buffers only 2-byte aligned."""
    import torch
    side = sides("dh64", False)
    cfg, ssd = side.cfg, side.ssd
    n = 200
    par = W.chain_tree(n)
    toks = W.tree_tokens(par, cfg.vocab, seed=9)
    s = ssd.Session(side.m, MAX_CTX, n, ssd.to_device(side.kc, cfg), ssd.to_device(side.vc, cfg))
    s.verify(P, toks, par)
    path = torch.tensor(np.random.default_rng(4).permutation(n)[:150], dtype=torch.int32, device="cuda")
    plen = torch.tensor([150], dtype=torch.int32, device="cuda")
    idx = path.long()
    want = [c.clone() for c in (s.k_cache, s.v_cache)]
    for w, t in zip(want, (s.k_tree, s.v_tree)):
        w[:, :, P:P + 150] = t[:, :, idx]
    s.commit(P, path, plen)
    for w, c in zip(want, (s.k_cache, s.v_cache)):
        assert torch.equal(w.view(torch.int16), c.view(torch.int16))
    # the same rows through a session whose cache starts 2 bytes past a 16-byte boundary
    def shifted(t):
        flat = torch.zeros(t.numel() + 8, dtype=t.dtype, device="cuda")[1:1 + t.numel()]
        return flat.copy_(t.reshape(-1)).view(t.shape)
    kc, vc = (shifted(ssd.to_device(a, cfg)) for a in (side.kc, side.vc))
    u = ssd.Session(side.m, MAX_CTX, n, kc, vc)
    u.k_tree.copy_(s.k_tree)
    u.v_tree.copy_(s.v_tree)
    u.commit(P, path, plen)
    for w, c in zip(want, (kc, vc)):
        assert torch.equal(w.view(torch.int16), c.view(torch.int16))
    assert s.error_count() == 0 and u.error_count() == 0
