"""The work that users of this package have it do, as measurable cases.

A case is a dict of plain values; its "kind" says which public entry points
it goes through (paper_2308_04623_amd.ssd):

  step     one greedy decoding step: Session.verify_greedy, then commit
  verify   one verification pass alone: Session.verify
  prefill  a prompt chunk as a chain: Session.verify, then commit of all of it
  draft    the staged loop's draft step: a pass of a layer-prefix view, then topk
  reuse    the draft's work handed to the oracle: reuse_into, then verify_from
  accept   the sampling accept walk on given logits: Session.accept
  cdf      CDF-first sampling: cdf_pick for the tree's assembly, then accept

Models are random-init GPT-2 shapes (the GPT-2-Large shape of the benchmark,
and the 2-layer toy of the tests).  A model is the checkpoint that a program
holds; its layers are rotated by the seed, and the prefix cache, the tree and
the tokens are drawn from the seed.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2308_04623_amd import ssd
from paper_2308_04623_amd import workloads as W

LN_EPS = 1e-5
VOCAB = 50257


def listed():
    return [
        # the toy float32 model of the smoke run and the tests: the smallest call, all launches and host work
        {"name": "toy_f32_n15_p64", "kind": "verify", "model": "toy", "n": 15, "tree": "binary", "P": 64, "q8": False},
        # plain greedy decoding, one token a step: what speculation is compared with
        {"name": "step_n1_p512", "kind": "step", "model": "gpt2l", "n": 1, "tree": "chain", "P": 512, "q8": False},
        # the benchmark's step: a 32-node tree over a 512-token prefix
        {"name": "step_n32_p512", "kind": "step", "model": "gpt2l", "n": 32, "tree": "4221", "P": 512, "q8": False},
        # the staged loop's largest oracle tree, over a ragged prefix
        {"name": "verify_n64_p1003", "kind": "verify", "model": "gpt2l", "n": 64, "tree": "best", "P": 1003,
         "q8": False},
        # the 8-bit weight model at a ragged tree size
        {"name": "step_q8_n45_p700", "kind": "step", "model": "gpt2l", "n": 45, "tree": "best", "P": 700, "q8": True},
        # a wide tree, past what one persistent launch takes
        {"name": "verify_n128_p512", "kind": "verify", "model": "gpt2l", "n": 128, "tree": "4221", "P": 512,
         "q8": False},
        # the stress point of the benchmark: 256 nodes over 2048 cached tokens
        {"name": "verify_n256_p2048", "kind": "verify", "model": "gpt2l", "n": 256, "tree": "84221", "P": 2048,
         "q8": False},
        # a 512-token prompt in one chunk
        {"name": "prefill_n512_p0", "kind": "prefill", "model": "gpt2l", "n": 512, "tree": "chain", "P": 0,
         "q8": False},
        # the staged loop's draft step over its largest bigram tree
        {"name": "draft_n32_p300", "kind": "draft", "model": "gpt2l", "n": 32, "tree": "421111", "P": 300,
         "q8": False, "k": 2},
        # rejection sampling of the stress tree's drawn children
        {"name": "accept_wor_n256", "kind": "accept", "mode": "wor", "n": 256, "tree": "84221", "top_k": 0,
         "temperature": 1.0},
        # the paper's sampling setting (top-50, T = 1) over a staged tree
        {"name": "accept_top50_n64", "kind": "accept", "mode": "det", "n": 64, "tree": "4221", "top_k": 50,
         "temperature": 1.0},
        # CDF-first assembly of one level and its walk
        {"name": "cdf_n64", "kind": "cdf", "n": 64, "tree": "333", "picks": 54, "temperature": 1.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["toy", "step", "step", "verify", "verify", "wide", "wide", "prefill", "draft", "reuse",
                       "accept", "accept", "cdf"])
    if kind == "toy":
        return {"kind": "verify", "model": "toy", "n": _log_int(rng, 1, 128), "tree": rng.choice(["binary", "chain"]),
                "P": rng.randrange(0, 120), "q8": False}
    if kind in ("step", "verify"):
        return {"kind": kind, "model": "gpt2l", "n": _log_int(rng, 1, 64),
                "tree": rng.choice(["chain", "binary", "best", "4221"]), "P": rng.randrange(0, 2048),
                "q8": rng.random() < 0.3}
    if kind == "wide":
        return {"kind": "verify", "model": "gpt2l", "n": _log_int(rng, 65, 256),
                "tree": rng.choice(["binary", "best", "84221"]), "P": rng.randrange(0, 2048), "q8": rng.random() < 0.3}
    if kind == "prefill":
        n = _log_int(rng, 20, 512)
        return {"kind": "prefill", "model": "gpt2l", "n": n, "tree": "chain",
                "P": 0 if rng.random() < 0.5 else rng.randrange(0, 1024 - n), "q8": rng.random() < 0.2}
    if kind == "draft":
        return {"kind": "draft", "model": "gpt2l", "n": _log_int(rng, 4, 32), "tree": "421111",
                "P": rng.randrange(1, 1024), "q8": False, "k": rng.randrange(1, 9)}
    if kind == "reuse":
        return {"kind": "reuse", "model": "gpt2l", "n": _log_int(rng, 1, 32), "tree": "421111",
                "P": rng.randrange(1, 1024), "q8": False}
    if kind == "accept":
        mode = rng.choice(["wor", "det"])
        return {"kind": "accept", "mode": mode, "n": _log_int(rng, 1, 256), "tree": rng.choice(["84221", "4221"]),
                "top_k": rng.choice([0, 50]), "temperature": rng.choice([1.0, 0.7])}
    return {"kind": "cdf", "n": _log_int(rng, 2, 64), "tree": "333", "picks": rng.randrange(1, 65),
            "temperature": rng.choice([1.0, 0.7])}


# ---------------------------------------------------------------- models

def _config(case):
    if case.get("model") == "toy":
        return W.TINY
    if case["kind"] in ("accept", "cdf"):
        # the walks only need a session over the vocabulary
        return W.GPT2Config(n_layer=1, d_model=128, n_head=4, d_mlp=512, vocab=VOCAB, n_pos=256, dtype="bf16")
    cfg = W.GPT2L_LONG.with_(n_pos=2048 + 512 + 64)
    # the draft is a view of the oracle's first 4 layers: it needs no more than those and one past them
    return cfg.with_(n_layer=5) if case["kind"] == "draft" else cfg


@functools.lru_cache(maxsize=4)
def _checkpoint(cfg):
    """Host parameters of a random-init model: N(0, 0.02) matrices, biases
    and LayerNorm parameters a little off their initial values."""
    gen = torch.Generator("cuda").manual_seed(1234)
    out = {k: [None] * cfg.n_layer for k in W.LAYER_TENSORS}
    for name, layer, shape, kind in W._tensor_shapes(cfg):
        t = torch.randn(shape, generator=gen, device="cuda") * 0.02
        if kind == "gain":
            t += 1.0
        a = t.cpu().numpy() if cfg.dtype == "f32" else t.bfloat16().view(torch.int16).cpu().numpy().view(np.uint16)
        if layer < 0:
            out[name] = a
        else:
            out[name][layer] = a
    return out


def _weights(cfg, seed):
    w = dict(_checkpoint(cfg))
    r = seed % cfg.n_layer
    for k in W.LAYER_TENSORS:
        w[k] = w[k][r:] + w[k][:r]
    return w


# ---------------------------------------------------------------- trees and inputs

def _parents(case, seed):
    n, t = case["n"], case["tree"]
    if t == "chain":
        return W.chain_tree(n)
    if t == "binary":
        return W.complete_binary_tree(n)
    if t == "best":
        return W.best_first_tree(n, seed=3 + seed % 1000)[1]
    return W.branching_tree([int(c) for c in t], n)


def _tokens(n, vocab, seed):
    return np.random.default_rng([seed, 7]).integers(0, vocab, n).astype(np.int32)


def _cache(cfg, rows, P, seed, device="cuda"):
    """Prefix cache rows < P ~ N(0, 0.7), what this model's own K and V look like."""
    gen = torch.Generator(device).manual_seed(seed + 17)
    dt = torch.float32 if cfg.dtype == "f32" else torch.bfloat16
    out = []
    for _ in range(2):
        c = torch.zeros(W.kv_shape(cfg, rows), dtype=dt, device=device)
        c[:, :, :P] = torch.randn((cfg.n_layer, cfg.n_head, P, cfg.head_dim), generator=gen, device=device) * 0.7
        out.append(c)
    return out


def _ctx_rows(case):
    return case["P"] + case["n"] + 16


def _outs(n):
    """path[n], path_len[1], next_token[1] as views of one buffer."""
    buf = torch.zeros(n + 2, dtype=torch.int32, device="cuda")
    return buf, (buf[:n], buf[n:n + 1], buf[n + 1:])


def prepare(case, seed):
    cfg = _config(case)
    kind, n = case["kind"], case["n"]
    par = _parents(case, seed)
    st = {"case": case, "par": par}
    model = ssd.Model(cfg, _weights(cfg, seed), q8=case.get("q8", False))
    st["model"] = model
    if kind in ("accept", "cdf"):
        st["sess"] = ssd.Session(model, 0, 256)
        st.update(_sampling_inputs(case, seed, par))
        st["buf"], st["out"] = _outs(n)
        return st
    P = case["P"]
    st["toks"] = _tokens(n, cfg.vocab, seed)
    kc, vc = _cache(cfg, _ctx_rows(case), P, seed)
    if kind == "draft":
        st["view"] = model.prefix_view(4)
        st["sess"] = ssd.Session(st["view"], _ctx_rows(case), n, kc[:4].contiguous(), vc[:4].contiguous())
    else:
        st["sess"] = ssd.Session(model, _ctx_rows(case), n, kc, vc)
    st["logits"] = torch.zeros((n, cfg.vocab), dtype=torch.float32, device="cuda")
    if kind == "step":
        st["buf"], st["out"] = _outs(n)
    if kind == "prefill":
        st["path"] = torch.arange(n, dtype=torch.int32, device="cuda")
        st["plen"] = torch.tensor([n], dtype=torch.int32, device="cuda")
    if kind == "reuse":
        # the draft has run on the tree; the oracle takes every second node over with its ancestors
        st["view"] = model.prefix_view(4)
        st["draft"] = ssd.Session(st["view"], _ctx_rows(case), n, st["sess"].k_cache[:4], st["sess"].v_cache[:4])
        st["draft"].verify(P, st["toks"], par)
        st["rows"], st["sub_par"] = _endorsed(par)
        st["sub_toks"] = st["toks"][st["rows"]]
        st["sub_logits"] = torch.zeros((len(st["rows"]), cfg.vocab), dtype=torch.float32, device="cuda")
    return st


def _endorsed(par):
    """The nodes of even rank among their siblings, with their ancestors."""
    seen, keep, pos, rank = {}, [0], {0: 0}, [0]
    for i in range(1, len(par)):
        p = int(par[i])
        rank.append(seen.get(p, 0))
        seen[p] = rank[i] + 1
        if p in pos and rank[i] % 2 == 0:
            pos[i] = len(keep)
            keep.append(i)
    return (np.array(keep, np.int32), np.array([-1] + [pos[int(par[i])] for i in keep[1:]], np.int32))


def _sampling_inputs(case, seed, par):
    """Logits peaked as a trained model's, and children as the draft proposes them: drawn without
    replacement from a draft row that is half the target and half heavy-tailed
    noise (wor), the draft's top tokens (det), or its inverse-CDF picks at the
    node's own uniform and two beside it (cdf)."""
    n = case["n"]
    gen = torch.Generator("cuda").manual_seed(seed + 29)
    logits = torch.randn((n, VOCAB), generator=gen, device="cuda") * 4.5
    toks = _tokens(n, VOCAB, seed)
    kids = [[] for _ in range(n)]
    for i in range(1, n):
        kids[int(par[i])].append(i)
    most = max(1, max(len(k) for k in kids))
    out = {"logits": logits, "toks": toks, "seed": seed}
    if case["kind"] == "accept":
        if case["mode"] == "wor":
            noise = torch.rand((n, VOCAB), generator=gen, device="cuda") ** 10
            q = 0.5 * torch.softmax(logits / case["temperature"], 1) + 0.5 * noise / noise.sum(1, keepdim=True)
            out["draft"] = q.contiguous()
            g = -torch.log(-torch.log(torch.rand((n, VOCAB), generator=gen, device="cuda").clamp(1e-20, 1 - 1e-7)))
            pick = (q.log() + g).topk(most, 1).indices.cpu().numpy()
        else:
            near = logits + torch.randn((n, VOCAB), generator=gen, device="cuda") * 0.3
            pick = near.topk(most, 1).indices.cpu().numpy()
    else:
        near = logits + torch.randn((n, VOCAB), generator=gen, device="cuda") * 0.1
        out["near"] = near
        r = np.random.default_rng([seed, 11])
        out["rows"] = np.sort(r.integers(0, n, case["picks"])).astype(np.int32)
        out["us"] = r.random(case["picks"])
        cdf = torch.softmax(near.double() / case["temperature"], 1).cumsum(1)
        us = np.array([[(ssd.uniform(seed, 2, u) + o) % 1.0 for o in (0.0, 0.05, -0.05)] for u in range(n)])
        pick = torch.searchsorted(cdf, torch.from_numpy(us).to("cuda"), right=True).clamp(max=VOCAB - 1)
        pick = pick.cpu().numpy()
        most = pick.shape[1]
    for u in range(n):
        for j, c in enumerate(kids[u]):
            toks[c] = pick[u, min(j, most - 1)]
    return out


# ---------------------------------------------------------------- one pass

def run(st):
    case, s = st["case"], st["sess"]
    kind = case["kind"]
    if kind == "step":
        lg = s.verify_greedy(case["P"], st["toks"], st["par"], st["logits"], st["out"])[0]
        s.commit(case["P"], st["out"][0], st["out"][1])
        return [lg, s.k_tree, s.v_tree, s.k_cache, s.v_cache, st["buf"]]
    if kind == "verify":
        return [s.verify(case["P"], st["toks"], st["par"], st["logits"]), s.k_tree, s.v_tree]
    if kind == "prefill":
        lg = s.verify(case["P"], st["toks"], st["par"], st["logits"])
        s.commit(case["P"], st["path"], st["plen"])
        return [lg, s.k_cache, s.v_cache]
    if kind == "draft":
        lg = s.verify(case["P"], st["toks"], st["par"], st["logits"])
        idx, val, lse = s.topk(lg, case["k"])
        return [lg, val, lse, idx]
    if kind == "reuse":
        x = st["draft"].reuse_into(s, st["rows"])
        lg = s.verify_from(case["P"], st["sub_toks"], st["sub_par"], 4, x, st["sub_logits"])
        return [lg, x]
    if kind == "accept":
        mode = ssd.SAMPLE_WOR if case["mode"] == "wor" else ssd.SAMPLE_DET
        s.accept(st["toks"], st["par"], st["logits"], mode=mode, draft_probs=st.get("draft"),
                 temperature=case["temperature"], seed=st["seed"], out=st["out"], top_k=case["top_k"])
        return [st["buf"]]
    picks = s.cdf_pick(st["near"], st["rows"], st["us"], case["temperature"])
    s.accept(st["toks"], st["par"], st["logits"], mode=ssd.SAMPLE_CDF, temperature=case["temperature"],
             seed=st["seed"], out=st["out"])
    return [picks, st["buf"]]


def _layers(case):
    cfg = _config(case)
    return 4 if case["kind"] == "draft" else cfg.n_layer - 4 if case["kind"] == "reuse" else cfg.n_layer


def work(case):
    cfg, n = _config(case), case["n"]
    if case["kind"] == "accept":
        # the logits (and draft rows) of the nodes that a walk passes: the root at least
        rows = 2 if case["mode"] == "wor" else 1
        return {"bytes": rows * 4 * VOCAB, "flops": 10 * VOCAB}
    if case["kind"] == "cdf":
        return {"bytes": 4 * VOCAB * (min(n, case["picks"]) + 1), "flops": 4 * VOCAB * (case["picks"] + 1)}
    if case["kind"] == "reuse":
        n = len(_endorsed(_parents(case, 0))[0])
    d, m, V, L, P = cfg.d_model, cfg.d_mlp, cfg.vocab, _layers(case), case["P"]
    es = 4 if cfg.dtype == "f32" else 2
    wbytes = 1 if case["q8"] else es
    par = _parents(case, 0)
    depth = [0] * len(par)
    for i in range(1, len(par)):
        depth[i] = depth[par[i]] + 1
    own = sum(x + 1 for x in depth[:n])
    per_layer = 4 * d * d + 2 * d * m
    return {
        "bytes": L * (per_layer * wbytes + 2 * P * d * es + 2 * n * d * es) + V * d * wbytes + 4 * n * V,
        "flops": 2 * n * (L * per_layer + V * d) + 4 * L * d * (n * P + own),
    }


# ---------------------------------------------------------------- tolerances and 64-bit results

def tolerance(case):
    if case["kind"] in ("accept", "cdf"):
        return "exact"
    if case.get("model") == "toy":
        # float32 sums of up to 512 terms in another order (2e-7 seen against 64 bits)
        return {"rel": 1e-6}
    # float16 GEMM inputs and bfloat16 K/V, each rounded once: up to 9e-4 of
    # the logits and of K/V (a bfloat16 step is 4e-3) seen against 64 bits
    tol = {"rel": 4e-3}
    if case["kind"] == "step":
        tol["differ"] = 1.01 / (case["n"] + 2)  # the next token, where two logits tie within the rounding
    if case["kind"] == "draft":
        tol["differ"] = 0.1  # neighbours in a row's top-k that tie within the rounding
    return tol


def _bf16(x):
    return x.to(torch.bfloat16).double()


def _quantized(w):
    """Symmetric 8-bit codes and a float32 scale per row, decided in float32."""
    w = w.float()
    a = w.abs().amax(1, keepdim=True)
    top = torch.full_like(a, 127.0)  # (a tensor: torch turns scalar / tensor into a reciprocal's product)
    code = torch.clamp(torch.round(w * (top / a)), -127, 127)
    return code.double() * (a / top).double()


def _norm(x, g, b):
    mu = x.mean(1, keepdim=True)
    var = ((x - mu) ** 2).mean(1, keepdim=True)
    return (x - mu) / torch.sqrt(var + LN_EPS) * g + b


def _forward(case, seed, cfg, layers, toks, par):
    """Float64 pass over the tree: logits, the K and V of the tree and of the
    prefix, and the residual stream after layer 4 (K and V rounded to the
    cache's type, as they are stored)."""
    f32 = cfg.dtype == "f32"
    w = _weights(cfg, seed)

    def up(a, quant=False):
        t = torch.from_numpy(np.ascontiguousarray(a)).cuda() if f32 else \
            torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda().view(torch.bfloat16)
        return _quantized(t) if quant else t.double()

    q8, n, P, H, D = case["q8"], len(toks), case["P"], cfg.n_head, cfg.head_dim
    kc, vc = _cache(cfg, _ctx_rows(case), P, seed)
    depth = np.zeros(n, np.int64)
    mask = torch.zeros((n, n), dtype=torch.bool)
    for i in range(n):
        if i:
            depth[i] = depth[par[i]] + 1
            mask[i] = mask[int(par[i])]
        mask[i, i] = True
    mask = torch.cat([torch.ones((n, P), dtype=torch.bool), mask], 1).cuda()
    wte = up(w["wte"])
    x = wte[torch.from_numpy(toks.astype(np.int64)).cuda()] + up(w["wpe"])[torch.from_numpy(P + depth).cuda()]
    ks, vs, x4 = [], [], None
    rnd = (lambda t: t.float().double()) if f32 else _bf16
    for l in range(layers):
        p = {k: up(w[k][l], q8 and k.startswith("w_")) for k in W.LAYER_TENSORS}
        qkv = _norm(x, p["ln1_g"], p["ln1_b"]) @ p["w_qkv"].T + p["b_qkv"]
        q, k, v = (t.view(n, H, D).transpose(0, 1) for t in qkv.split(cfg.d_model, 1))
        k, v = rnd(k), rnd(v)
        ks.append(k)
        vs.append(v)
        ka = torch.cat([kc[l, :, :P].double(), k], 1)
        va = torch.cat([vc[l, :, :P].double(), v], 1)
        sc = torch.matmul(q, ka.transpose(1, 2)) / math.sqrt(D)
        o = torch.matmul(torch.softmax(sc.masked_fill(~mask, -math.inf), -1), va)
        x = x + o.transpose(0, 1).reshape(n, -1) @ p["w_o"].T + p["b_o"]
        h = _norm(x, p["ln2_g"], p["ln2_b"]) @ p["w_fc"].T + p["b_fc"]
        h = 0.5 * h * (1 + torch.tanh(math.sqrt(2 / math.pi) * (h + 0.044715 * h ** 3)))
        x = x + h @ p["w_pr"].T + p["b_pr"]
        if l == 3:
            x4 = x.clone()
    head = _quantized(up(w["wte"]).float()) if q8 else wte
    logits = _norm(x, up(w["lnf_g"]), up(w["lnf_b"])) @ head.T
    return logits, torch.stack(ks), torch.stack(vs), kc, vc, x4


def exact(case, seed):
    kind = case["kind"]
    if kind in ("accept", "cdf"):
        return None
    cfg = _config(case)
    par, toks = _parents(case, seed), _tokens(case["n"], cfg.vocab, seed)
    if kind == "reuse":
        rows, sub = _endorsed(par)
        lg, _, _, _, _, x4 = _forward(case, seed, cfg, cfg.n_layer, toks[rows], sub)
        return [lg, x4]
    lg, k, v, kc, vc, _ = _forward(case, seed, cfg, 4 if kind == "draft" else cfg.n_layer, toks, par)
    if kind == "verify":
        return [lg, k, v]
    P, n = case["P"], case["n"]
    if kind == "draft":
        val = lg.topk(case["k"], 1).values
        return [lg, val, torch.logsumexp(lg, 1), None]
    if kind == "prefill":
        path = list(range(n))
    else:
        best = lg.argmax(1).cpu().numpy()
        paths = {0: [0]}
        for i in range(1, n):
            if int(par[i]) in paths and int(toks[i]) == int(best[par[i]]):
                paths[i] = paths[int(par[i])] + [i]
        path = max(paths.values(), key=len)
    kc, vc = kc.double(), vc.double()
    kc[:, :, P:P + len(path)] = k[:, :, path]
    vc[:, :, P:P + len(path)] = v[:, :, path]
    return [lg, kc, vc] if kind == "prefill" else [lg, k, v, kc, vc, None]
