"""Prefill rows of a group whose items walk the shared keys and then each request's own (GPU), against the CPU oracle: requests that
end inside, at and behind an item, templates of no multiple of 64 keys, decode rows and other groups beside them."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2601_11546_amd import workloads as W
from tests.gpu_harness import assert_close, dev_bf16, host_bits, host_f32

pytestmark = pytest.mark.gpu


# query tokens, own keys and template of a group whose prefill rows take joint items (test_attention_items.py): requests that share
# items and waves, some with cached keys of their own
JOINT_BATCH = (np.array([50, 50, 60, 65, 90, 70, 12]), np.array([50, 110, 63, 65, 100, 110, 12]), 80)
# the same with a decode row behind the template: over 16-bit pools the template is an item of the one launch for it
MIXED_BATCH = (np.array([300, 1]), np.array([300, 41]), 80)
# query tokens and own keys of requests with which the same group takes two passes: their cached keys, one request after the other
# in a joint item, would take too long
TWO_PASSES = (np.array([4] * 4), np.array([1500] * 4))
JOINT_SHAPES = {"group1": replace(W.TINY, n_q_heads=48, n_kv_heads=48), "group5": W.TINY_G5, "d128": W.TINY_D128, "g3d128": W.TINY_G3_D128}


@pytest.fixture(scope="module")
def rs():
    assert torch.cuda.is_available(), "GPU tests need a device"
    from paper_2601_11546_amd import binding
    return binding


@pytest.mark.parametrize("shape", [W.TINY, W.TINY_GQA, W.TINY_G5], ids=["group1", "gqa", "group5"])
@pytest.mark.parametrize("prefix", [16, 64, 80, 208])
@pytest.mark.parametrize("q_len", [[128, 128], [127, 2, 130], [64, 1, 63, 65, 1, 2], [33, 1, 200, 40, 31]], ids=str)
def test_joint_items(rs, oracle, shape, prefix, q_len):
    q = np.array(q_len + [50])                                  # the last request carries no template
    own = q + np.arange(len(q)) % 3 * 37                        # some have cached keys of their own behind the template
    pid = np.array([0] * len(q_len) + [-1])
    b = W.build_batch(shape, q, own + np.where(pid >= 0, prefix, 0), pid, [prefix], seed=prefix)
    wl = W.Workload("joint", shape, b, prefix)
    weights, x = wl.weights(), W.make_activations(b.T, shape.hidden, prefix)
    kp, vp = W.make_cache(shape, b.num_pages, prefix)
    layer = rs.relserve_layer_create(shape)
    pb = rs.relserve_batch_prepare(layer, b)
    xd = dev_bf16(x)
    y = torch.full_like(xd, float("nan"))
    ws = torch.full((rs.relserve_workspace_bytes(layer, b.T),), 0xff, dtype=torch.uint8, device="cuda")
    rs.relserve_layer_step(layer, pb, {k: dev_bf16(v) for k, v in weights.items()}, xd, y, dev_bf16(kp), dev_bf16(vp), ws)
    want = oracle.layer_step(shape, b, weights, x, kp, vp).y_f32
    assert_close(host_f32(y), want, f"joint {q_len} behind {prefix}")     # the whole step's bar


@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
@pytest.mark.parametrize("shape", JOINT_SHAPES.values(), ids=JOINT_SHAPES)
def test_a_request_spoils_its_own_rows_alone(rs, shape, fp8):
    """Requests that share an item, and waves of it, with one whose cached keys or values are not finite: the others' rows have
    the bits they have beside finite ones."""
    q, own, prefix = JOINT_BATCH
    bad_v, bad_k = [1, 3], [5]
    b = W.build_batch(shape, q, own + prefix, [0] * len(q), [prefix], seed=4)
    g = torch.Generator(device="cuda").manual_seed(5)
    size = (b.num_pages, shape.page_size, shape.n_kv_heads, shape.head_dim)
    if fp8:
        pools = [torch.randint(0, 120, size, generator=g, device="cuda", dtype=torch.uint8) for _ in "kv"]
        bad = [0x7f, 0xff]                      # the 8-bit format has NaN alone
    else:
        pools = [torch.randn(*size, generator=g, device="cuda").bfloat16() for _ in "kv"]
        bad = [float("inf"), float("nan")]
    table = np.asarray(b.block_table).reshape(len(q), -1)
    qs = torch.randn(b.T, shape.q_dim, generator=g, device="cuda").bfloat16()
    layer = rs.relserve_layer_create(shape)
    pb = rs.relserve_batch_prepare(layer, b)

    def attend(k, v):
        ws = torch.full((rs.relserve_workspace_bytes(layer, b.T),), 0xff, dtype=torch.uint8, device="cuda")
        out = torch.zeros(b.T, shape.q_dim, dtype=torch.bfloat16, device="cuda")
        rs.relserve_attention(layer, pb, qs, shape.q_dim, *((rs.QuantPool(k, 0.125), rs.QuantPool(v, 0.07)) if fp8 else (k, v)), out, ws)
        torch.cuda.synchronize()
        return out.float().cpu().numpy()

    clean = attend(*pools)
    assert np.isfinite(clean).all()
    k, v = (p.clone() for p in pools)
    for pool, requests in ((v, bad_v), (k, bad_k)):
        for i, r in enumerate(requests):
            pages = table[r, prefix // shape.page_size:(prefix + own[r] + shape.page_size - 1) // shape.page_size]
            pool[torch.from_numpy(pages.astype(np.int64)).cuda()] = bad[i]
    got = attend(k, v)
    start = np.concatenate([[0], np.cumsum(q)])
    for r in range(len(q)):
        rows = slice(start[r], start[r + 1])
        if r in bad_v + bad_k:
            assert not np.isfinite(got[rows]).all()
        else:
            assert np.array_equal(got[rows], clean[rows]), r


@pytest.mark.parametrize("batch", [JOINT_BATCH, MIXED_BATCH], ids=["joint", "mixed"])
@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
@pytest.mark.parametrize("shape", JOINT_SHAPES.values(), ids=JOINT_SHAPES)
def test_joint_items_have_the_two_passes_bits(rs, oracle, shape, fp8, batch):
    """The attention of the same requests, over the same pages, in joint items and (beside others) in two passes, and the oracle's."""
    q, own, prefix = batch
    n = len(q)
    q_all, own_all = np.concatenate([q, TWO_PASSES[0]]), np.concatenate([own, TWO_PASSES[1]])
    both = W.build_batch(shape, q_all, own_all + prefix, [0] * len(q_all), [prefix], seed=6)
    alone = both.select(range(n))
    g = torch.Generator(device="cuda").manual_seed(7)
    size = (both.num_pages, shape.page_size, shape.n_kv_heads, shape.head_dim)
    if fp8:
        kd, vd = (torch.randint(0, 96, size, generator=g, device="cuda", dtype=torch.uint8) for _ in "kv")
        pools = rs.QuantPool(kd, 0.125), rs.QuantPool(vd, 0.07)
        kp, vp = kd.cpu().numpy(), vd.cpu().numpy()
    else:
        kd, vd = pools = [torch.randn(*size, generator=g, device="cuda").bfloat16() for _ in "kv"]
        kp, vp = host_bits(kd), host_bits(vd)
    qs = torch.randn(both.T, shape.q_dim, generator=g, device="cuda").bfloat16()
    layer = rs.relserve_layer_create(shape)

    def attend(b):
        pb = rs.relserve_batch_prepare(layer, b)
        ws = torch.full((rs.relserve_workspace_bytes(layer, b.T),), 0xff, dtype=torch.uint8, device="cuda")
        out = torch.zeros(b.T, shape.q_dim, dtype=torch.bfloat16, device="cuda")
        rs.relserve_attention(layer, pb, qs, shape.q_dim, *pools, out, ws)
        return host_f32(out)

    joint, passes = attend(alone), attend(both)
    start = np.concatenate([[0], np.cumsum(q)])
    qf = host_f32(qs)
    past = np.repeat(own + prefix - q, q) + np.arange(alone.T) - np.repeat(start[:-1], q)   # position of every query token
    for r in range(n):
        rows = slice(start[r], start[r + 1])
        if q[r] > 1:
            assert np.array_equal(joint[rows], passes[rows]), r
        else:
            # a decode row's two states are merged in the one and one state runs on in the other: fp32 sums either way, but the
            # probabilities are rounded to bf16 against other reference values: 2^-9 of a weighted mean of |v| on each side, and the
            # output's own rounding, 2^-9 of it on each side
            v_max = float((vd.view(torch.float8_e4m3fn).float() * 0.07 if fp8 else vd.float()).abs().max())
            assert (np.abs(joint[rows] - passes[rows]) <= 2.0 ** -8 * (v_max + np.abs(passes[rows]))).all(), r
        for t in (start[r], start[r + 1] - 1):
            args = (shape, alone, r, int(past[t]), qf[t].reshape(shape.n_q_heads, -1), kp, vp)
            want = oracle.attention_token_fp8kv(*args, 0.125, 0.07) if fp8 else oracle.attention_token(*args)
            # the attention stage's bar
            assert_close(joint[t], want.reshape(-1), f"request {r}, token {t}", max_abs=2e-2, rel_l2=1e-2)
