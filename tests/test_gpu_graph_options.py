"""The weight prefetch option counts when a graph is launched, not when it was
captured; logits are the same bit for bit either way."""
import numpy as np
import pytest

from paper_2308_04623_amd import workloads as W

pytestmark = pytest.mark.gpu

CFG = W.GPT2Config(n_layer=2, d_model=256, n_head=4, d_mlp=512, vocab=515, n_pos=400, dtype="bf16")


# wide trees prefetch inside their kernels, smaller ones (one kernel per sub-layer) by the prefetcher beside them
@pytest.mark.parametrize("n", [20, 65, 200])
@pytest.mark.parametrize("captured", [0, 1])
@pytest.mark.parametrize("q8", [False, True])
def test_prefetch_option_at_launch(n, captured, q8):
    import torch
    from paper_2308_04623_amd import ssd
    P, ctx = 70, 300
    w = W.make_weights(CFG, 1, perturb_affine=True)
    kc, vc = W.random_kv_cache(CFG, ctx, P, seed=2)
    s = ssd.Session(ssd.Model(CFG, w, q8=q8), ctx, n, ssd.to_device(kc, CFG), ssd.to_device(vc, CFG))
    s.set_options(pass_mode=ssd.PASS_KERNELS, weight_prefetch=captured)
    par = W.branching_tree([4, 2, 2, 1], n)
    toks = W.tree_tokens(par, CFG.vocab, seed=n)
    want = s.verify(P, toks, par).cpu().numpy()
    lg = torch.zeros((n, CFG.vocab), dtype=torch.float32, device="cuda")
    out = [torch.zeros(k, dtype=torch.int32, device="cuda") for k in (n, 1, 1)]
    plain = s.capture_verify(P, toks, par, lg)
    greedy = s.capture_verify_greedy(P, toks, par, lg, out)
    path, plen, nxt = s.accept(toks, par, torch.from_numpy(want).cuda())
    for on in (1, 0, 0, 1):
        # (the pass mode and GEMM path of the capture hold, whatever they are at a launch)
        s.set_options(pass_mode=ssd.PASS_AUTO, gemm_path=on, weight_prefetch=on)
        for g in (plain, greedy):
            assert g.prefetches() == (bool(on) and n > 64)
            lg.zero_()
            g.launch()
            assert np.array_equal(lg.cpu().numpy(), want)
        m = int(plen.item())
        assert int(out[1].item()) == m and torch.equal(out[0][:m], path[:m]) and torch.equal(out[2], nxt.reshape(1))
        assert s.get_options() == {"pass_mode": ssd.PASS_AUTO, "gemm_path": on, "weight_prefetch": on}
    assert s.error_count() == 0
