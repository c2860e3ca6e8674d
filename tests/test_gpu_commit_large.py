"""KV commit where the tree scratch passes 2 GiB: rows arrive whole, and each
skipped row is counted once."""
import numpy as np
import pytest

from paper_2308_04623_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_commit_past_two_gib():
    import torch
    from paper_2308_04623_amd import ssd
    L, n, ctx, P = 2048, 1024, 4, 1
    cfg = W.GPT2Config(n_layer=1, d_model=256, n_head=4, d_mlp=32, vocab=64, n_pos=16, dtype="f32")
    w = W.make_weights(cfg, 0)
    for k in W.LAYER_TENSORS:
        w[k] = w[k] * L
    cfg = cfg.with_(n_layer=L)
    s = ssd.Session(ssd.Model(cfg, w), ctx, n)
    assert s.k_tree.numel() * s.k_tree.element_size() >= 1 << 31
    gen = torch.Generator("cuda").manual_seed(1)
    for t in (s.k_tree, s.v_tree):
        t.normal_(generator=gen)
    want = [c.clone() for c in (s.k_cache, s.v_cache)]
    for c, t in zip(want, (s.k_tree, s.v_tree)):
        c[:, :, P] = t[:, :, 1023]
        c[:, :, P + 2] = t[:, :, 7]
    # the second entry is no node, the fourth would be past the cache
    s.commit(P, torch.tensor([1023, -1, 7, 5], dtype=torch.int32, device="cuda"),
             torch.tensor([4], dtype=torch.int32, device="cuda"))
    for c, d in zip(want, (s.k_cache, s.v_cache)):
        assert torch.equal(c, d)
    assert s.error_count() == 2
    s.commit(P, torch.zeros(4, dtype=torch.int32, device="cuda"), torch.tensor([n + 1], dtype=torch.int32, device="cuda"))
    assert s.error_count() == 3
