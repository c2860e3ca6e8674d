"""The float32 model's GELU alone, to its float32 rounding.

The embeddings and the attention's weights are zero and the up-projection
leaves only its bias, so the residual stream after the one layer is the GELU of
that bias, exactly: the down-projection is the identity."""
import numpy as np
import pytest

from paper_2308_04623_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sd", [0.25, 1.0, 2.0])
def test_gelu_error_against_64_bits(sd):
    from paper_2308_04623_amd import ssd
    d = 2048
    cfg = W.GPT2Config(n_layer=1, d_model=d, n_head=32, d_mlp=d, vocab=64, n_pos=16, dtype="f32")
    w = W.make_weights(cfg, 0)
    for name in ("wte", "wpe"):
        w[name] = np.zeros_like(w[name])
    for name in ("w_qkv", "w_o", "w_fc"):
        w[name][0] = np.zeros_like(w[name][0])
    w["w_pr"][0] = np.eye(d, dtype=np.float32)
    x = (np.random.default_rng(1).standard_normal(d) * sd).astype(np.float32)
    w["b_fc"][0] = x
    m = ssd.Model(cfg, w)
    s, to = ssd.Session(m, 0, 1), ssd.Session(m, 0, 1)
    s.verify(0, np.zeros(1, np.int32), np.array([-1], np.int32))
    got = s.reuse_into(to, np.zeros(1, np.int32)).cpu().numpy()[0].astype(np.float64)
    v = x.astype(np.float64)
    want = 0.5 * v * (1 + np.tanh(np.sqrt(2 / np.pi) * (v + 0.044715 * v ** 3)))
    err = np.linalg.norm(got - want) / np.linalg.norm(want)
    # The tanh form rounds 1 + tanh and the product (2^-24 each, at half a binade some 2.4e-8 in the mean) and tanh and
    # its argument before (which the slope of tanh weighs down): 3.4e-8 to 4.0e-8 over 4M values.  With a hardware
    # exponential and reciprocal: 4.4e-8 to 4.9e-8.
    assert err < 4.25e-8
