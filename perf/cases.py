"""The work a serving program has this library do, as measurable cases.

A case is one call of a serving iteration's GPU share on seeded random inputs:

  entry "layer"   one decoder-layer step over a prepared batch (relserve_layer_step or, with "w8a8",
                  relserve_layer_step_w8a8).  A batch is prepared once per model step and serves all its layers, so the
                  prepared batch belongs to what the program already has.
  entry "model"   one whole iteration on a short stack: prepare the batch the scheduler handed over, upload its token
                  ids, relserve_model_step, relserve_greedy_sample, fetch the next tokens, destroy the batch.

Fields of a case: "shape" (a layer shape of workloads.py), "n_layers" and "vocab" (entry "model"); the batch: "n_dec"
decode rows whose own contexts (beyond the shared template) are drawn from [dec_lo, dec_hi], "n_pre" prefill rows of
[pre_lo, pre_hi] query tokens, spread over "groups" relQueries whose templates of "prefix" tokens are cached (0: no
shared template), and one more prefill request of "chunk" tokens without a past; "lengths" seeds the drawn lengths.
"w8a8": quantised projections; "kv8": quantised cache; "packed": weights in the streaming layout (else row-major).
"""
import math
import random

import numpy as np
import torch

from paper_2601_11546_amd import binding as rs
from paper_2601_11546_amd import duration_model
from paper_2601_11546_amd import workloads as W

SHAPES = {"tiny": W.TINY, "tiny_gqa": W.TINY_GQA, "tiny_g5": W.TINY_G5, "13b": W.LLAMA_13B, "70b": W.LLAMA_70B,
          "70b_tp4": W.LLAMA_70B_TP4, "32b": W.QWEN_32B, "32b_tp2": W.QWEN_32B_TP2}
DEPTH = {"13b": 40, "70b": 80, "70b_tp4": 80, "32b": 64, "32b_tp2": 64}   # of the stack a layer is cut from (init scale)
K_SCALE, V_SCALE = 2.0 ** -4, 2.0 ** -5                                   # of the quantised pools


def _case(name, shape, **kw):
    c = {"name": name, "entry": "layer", "shape": shape, "n_layers": 1, "vocab": 0, "n_dec": 0, "dec_lo": 1, "dec_hi": 1, "n_pre": 0,
         "pre_lo": 1, "pre_hi": 1, "groups": 1, "prefix": 0, "chunk": 0, "lengths": 1, "w8a8": False, "kv8": False, "packed": True}
    c.update(kw)
    return c


def listed():
    return [
        # the tiny layer of the first benchmark configuration: six decode rows and two 64-token prefills, all launch cost
        _case("tiny_mixed", "tiny", n_dec=6, dec_lo=128, dec_hi=128, n_pre=2, pre_lo=64, pre_hi=64, packed=False),
        # the end of a relQuery: its last four rows decode behind their template; latency of a nearly idle server
        _case("decode4_13b", "13b", n_dec=4, dec_lo=31, dec_hi=136, prefix=512),
        # a serving iteration of a small decode batch, with everything the worker does for it
        _case("serve_decode24_13b", "13b", entry="model", n_layers=4, vocab=32000, n_dec=24, dec_lo=31, dec_hi=136, groups=2,
              prefix=512, packed=False),
        # the headline batch: one relQuery of 200 rows behind a 512-token template, 16 of them prefilling their suffix
        _case("relquery_13b", "13b", n_dec=184, dec_lo=31, dec_hi=136, n_pre=16, pre_lo=30, pre_hi=120, prefix=512),
        # prefill of about 8000 suffix tokens behind one cached template
        _case("prefill_13b", "13b", n_pre=65, pre_lo=50, pre_hi=200, prefix=1024),
        # the same with quantised projections, an odd half of the size
        _case("prefill_13b_w8a8", "13b", n_pre=31, pre_lo=50, pre_hi=200, prefix=1024, w8a8=True),
        # decode rows of four relQueries beside one long prefill chunk, grouped-query layer of the 70B shape
        _case("mixed_70b", "70b", n_dec=256, dec_lo=1, dec_hi=732, groups=4, prefix=768, chunk=2048),
        # the same decode rows alone: weights and matrix work about equal
        _case("decode256_70b", "70b", n_dec=256, dec_lo=1, dec_hi=732, groups=4, prefix=768),
        # decode at context 1024 without sharing: bound by the cached keys and values
        _case("decode128_13b", "13b", n_dec=128, dec_lo=1024, dec_hi=1024),
        # the same with both quantised variants
        _case("decode128_13b_w8a8_kv8", "13b", n_dec=128, dec_lo=1024, dec_hi=1024, w8a8=True, kv8=True),
        # the headline kind of batch on the 32B shape (five query heads per kv head), both quantised variants, odd sizes
        _case("relquery_32b_w8a8_kv8", "32b", n_dec=95, dec_lo=31, dec_hi=136, n_pre=9, pre_lo=30, pre_hi=120, groups=3, prefix=256,
              w8a8=True, kv8=True),
        # a serving iteration that decodes long contexts and prefills a 512-token chunk
        _case("serve_chunk512_13b", "13b", entry="model", n_layers=4, vocab=32000, n_dec=128, dec_lo=1024, dec_hi=1024, chunk=512),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng: random.Random) -> dict:
    """Batches of the same kinds at sizes spread over the range: 1-256 decode rows, 2-8000 prefill tokens, mixtures."""
    shape = rng.choice(["13b", "13b", "13b", "70b", "32b", "32b_tp2", "70b_tp4", "tiny", "tiny_gqa", "tiny_g5"])
    small = shape.startswith("tiny")
    c = _case("", shape, lengths=rng.randrange(1, 1 << 20), groups=rng.randint(1, 4),
              prefix=rng.choice([0, 16 * rng.randint(4, 16), 16 * rng.randint(16, 64)]))
    del c["name"]
    kind = rng.choice(["decode", "prefill", "mixed", "chunk"])
    if kind != "prefill":
        c["n_dec"] = _log_int(rng, 1, 256)
        c["dec_lo"] = rng.randint(1, 40)
        c["dec_hi"] = c["dec_lo"] + _log_int(rng, 8, 120 if c["prefix"] else 1400)
    if kind in ("prefill", "mixed"):
        c["n_pre"] = _log_int(rng, 1, 70 if kind == "prefill" else 24)
        c["pre_lo"] = rng.randint(2, 60)
        c["pre_hi"] = c["pre_lo"] + rng.randint(1, 140)
    if kind == "chunk":
        c["chunk"] = _log_int(rng, 16, 2048)
    if not small:
        c["w8a8"] = rng.random() < 0.3
        c["packed"] = rng.random() < 0.75
        if shape == "13b" and rng.random() < 0.35:
            c.update(entry="model", n_layers=rng.randint(1, 4), vocab=32000)
    else:
        c["packed"] = False
    c["kv8"] = rng.random() < 0.25
    c["groups"] = max(1, min(c["groups"], c["n_dec"] + c["n_pre"]))
    top = max(_cost(x) for x in listed())
    while _cost(c) > top:    # never dearer than the largest listed case
        if c["n_layers"] > 1:
            c["n_layers"] -= 1
        elif c["n_pre"] + c["chunk"] > 1:
            c["n_pre"], c["chunk"] = (c["n_pre"] + 1) // 2, c["chunk"] // 2
        else:
            c["n_dec"] = max(1, c["n_dec"] // 2)
    return c


def _lengths(case):
    """(q_len, ctx_len, prefix_id) of the batch: decided by the case alone, so that every seed does the same work."""
    rng = np.random.default_rng(case["lengths"])
    n_dec, n_pre, prefix, groups = case["n_dec"], case["n_pre"], case["prefix"], case["groups"]
    pre = rng.integers(case["pre_lo"], case["pre_hi"] + 1, n_pre)
    own = rng.integers(case["dec_lo"], case["dec_hi"] + 1, n_dec)
    q_len = np.concatenate([pre, np.ones(n_dec, np.int64)])
    ctx = prefix + np.concatenate([pre, own])
    n = n_pre + n_dec
    pid = np.arange(n) * groups // max(n, 1) if prefix else np.full(n, -1)
    if prefix and groups > 1:
        pid = rng.permutation(pid)       # rows of several relQueries interleave in a batch
    if case["chunk"]:
        q_len, ctx, pid = np.append(q_len, case["chunk"]), np.append(ctx, case["chunk"]), np.append(pid, -1)
    return q_len.astype(np.int32), ctx.astype(np.int32), pid.astype(np.int32)


def _batch(case, seed):
    q_len, ctx, pid = _lengths(case)
    return W.build_batch(SHAPES[case["shape"]], q_len, ctx, pid, [case["prefix"]] * case["groups"] if case["prefix"] else [], seed=seed)


def work(case):
    s = SHAPES[case["shape"]]
    q_len, ctx, pid = (a.astype(np.int64) for a in _lengths(case))
    T, past = int(q_len.sum()), ctx - q_len
    we, ke = (1 if case["w8a8"] else 2), (1 if case["kv8"] else 2)
    proj = s.qkv_dim * s.hidden + s.hidden * s.q_dim + 3 * s.mlp_dim * s.hidden
    visible = int((q_len * past + q_len * (q_len + 1) // 2).sum())
    flops = 2 * T * proj + 4 * s.q_dim * visible
    # every weight once, every cached key and value once (a template once for all its rows), activations in and out
    used = [p for p in np.unique(pid) if p >= 0]
    cached = int(ctx.sum()) - case["prefix"] * int((pid >= 0).sum()) + case["prefix"] * len(used)
    kv = 2 * s.kv_dim * ke
    layer = proj * we + 4 * s.hidden + cached * kv + (s.qkv_dim + 3 * s.mlp_dim + s.hidden) * 4 * (we == 1)
    if case["entry"] == "layer":
        return {"bytes": layer + 4 * T * s.hidden, "flops": flops}
    n = len(q_len)
    return {"bytes": case["n_layers"] * layer + 2 * (case["vocab"] + T) * s.hidden + 4 * n * case["vocab"],
            "flops": case["n_layers"] * flops + 2 * n * case["vocab"] * s.hidden}


def _cost(case):
    w = work(case)
    return max(w["bytes"] / 5e12, w["flops"] / (2e15 if case["w8a8"] else 1.1e15))


def prepare(case, seed):
    s, batch = SHAPES[case["shape"]], _batch(case, seed)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def randn(*size, std=1.0, mean=0.0):
        return (torch.randn(*size, generator=g, device="cuda", dtype=torch.float32) * std + mean).to(torch.bfloat16)

    H, I, depth = s.hidden, s.mlp_dim, DEPTH.get(case["shape"], 0)
    out_std = 0.02 / math.sqrt(2 * depth) if depth else 0.02

    def weights():
        w = {"w_in_norm": randn(H, std=0.02, mean=1.0), "w_qkv": randn(s.qkv_dim, H, std=0.02), "w_o": randn(H, s.q_dim, std=out_std),
             "w_post_norm": randn(H, std=0.02, mean=1.0), "w_gate_up": randn(2 * I, H, std=0.02), "w_down": randn(H, I, std=out_std)}
        if case["w8a8"]:
            w = duration_model.quantise_layer_on_device(torch, w)
            return rs.pack_layer_weights_w8a8(w) if case["packed"] else w
        return rs.pack_layer_weights(w) if case["packed"] else w

    pool = (batch.num_pages, s.page_size, s.n_kv_heads, s.head_dim)

    def cache():
        if not case["kv8"]:
            return randn(*pool), randn(*pool)

        def codes():    # magnitudes under 32 code units, random signs
            c = torch.randint(0, 96, pool, generator=g, device="cuda", dtype=torch.uint8)
            return c | (torch.randint(0, 2, pool, generator=g, device="cuda", dtype=torch.uint8) << 7)
        return rs.QuantPool(codes(), K_SCALE), rs.QuantPool(codes(), V_SCALE)

    layer = rs.relserve_layer_create(s)
    st = {"case": case, "layer": layer, "batch": batch}
    if case["entry"] == "layer":
        st.update(weights=weights(), x=randn(batch.T, H), prepared=rs.relserve_batch_prepare(layer, batch))
        st["k"], st["v"] = cache()
        st["y"] = torch.empty_like(st["x"])
        st["workspace"] = torch.empty(rs.relserve_workspace_bytes(layer, batch.T), dtype=torch.uint8, device="cuda")
        return st
    vocab = case["vocab"]
    emb = randn(vocab, H)
    # a trained output layer prefers few tokens: here the successor of the token just read, above the random rest
    head = randn(vocab, H, std=0.02) + 0.002 * torch.roll(emb, 1, 0)
    st["model"] = {"embedding": emb, "layers": [weights() for _ in range(case["n_layers"])], "caches": [cache() for _ in range(case["n_layers"])],
                   "w_final_norm": randn(H, std=0.02, mean=1.0), "w_lm_head": head}
    st["ids"] = np.random.default_rng(seed).integers(0, vocab, batch.T).astype(np.int32)
    st["workspace"] = torch.empty(rs.relserve_model_workspace_bytes(layer, batch.T, batch.num_reqs), dtype=torch.uint8, device="cuda")
    return st


def _pool(p):
    return p.codes if isinstance(p, rs.QuantPool) else p


def run(st):
    case, layer = st["case"], st["layer"]
    if case["entry"] == "layer":
        step = rs.relserve_layer_step_w8a8 if case["w8a8"] else rs.relserve_layer_step
        step(layer, st["prepared"], st["weights"], st["x"], st["y"], st["k"], st["v"], st["workspace"])
        return {"y": st["y"], "k": _pool(st["k"]), "v": _pool(st["v"])}
    batch, model = st["batch"], st["model"]
    pb = rs.relserve_batch_prepare(layer, batch)
    ids = torch.from_numpy(st["ids"]).cuda()
    logits = torch.empty(batch.num_reqs, case["vocab"], dtype=torch.float32, device="cuda")
    tokens = torch.empty(batch.num_reqs, dtype=torch.int32, device="cuda")
    rs.relserve_model_step(layer, pb, model, ids, logits, st["workspace"])
    rs.relserve_greedy_sample(logits, tokens)
    tokens = tokens.cpu()                  # the worker looks at them to see which requests have finished
    pb.close()
    return {"logits": logits, "tokens": tokens, "caches": [[_pool(k), _pool(v)] for k, v in model["caches"]]}


def tolerance(case):
    # Outputs are bf16 and every intermediate result is rounded to bf16 (or to 8-bit codes) once, so implementations differ
    # by values that round the other way.  Measured between this one and itself with other sums (other tiles and k splits,
    # every row attending to its template alone instead of with its group): a layer's output rel 1.7e-3, largest
    # difference one unit in the last place (0.0078 of the value; with quantised projections 0.029 of the RMS); four
    # layers' logits rel 4.1e-3, their caches up to 0.023 of the RMS; codes and tokens equal.  Four times these:
    if case["entry"] == "model":
        return {"rel": 1.6e-2, "max": 0.1, "differ": 1e-3}
    return {"rel": 7e-3, "max": 0.12 if case["w8a8"] else 0.032, "differ": 1e-3}
