"""Decode-only batches whose rows are computed in parts (chunks of the shared prefix, chunks of their own keys) that one
merge puts together: lengths around the chunk and block edges, groups and loose rows in one batch, one to 256 rows."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2601_11546_amd import workloads as W
from tests.gpu_harness import assert_close, dev_bf16, host_f32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rs():
    assert torch.cuda.is_available(), "GPU tests need a device"
    from paper_2601_11546_amd import binding
    return binding


def _check(rs, oracle, shape, b, rows, fp8=False):
    rng = np.random.default_rng(b.T)
    q_bits = W.f32_to_bf16_bits(rng.standard_normal((b.T, shape.q_dim), dtype=np.float32))
    if fp8:
        kp, vp = W.make_cache_fp8(shape, b.num_pages, 11)
        pools = rs.QuantPool(torch.from_numpy(kp).cuda(), 0.125), rs.QuantPool(torch.from_numpy(vp).cuda(), 0.07)
    else:
        kp, vp = W.make_cache(shape, b.num_pages, 11)
        pools = dev_bf16(kp), dev_bf16(vp)
    layer = rs.relserve_layer_create(shape)
    pb = rs.relserve_batch_prepare(layer, b)
    ws = torch.full((rs.relserve_workspace_bytes(layer, b.T),), 0xff, dtype=torch.uint8, device="cuda")   # NaN everywhere
    out = torch.zeros(b.T, shape.q_dim, dtype=torch.bfloat16, device="cuda")
    rs.relserve_attention(layer, pb, dev_bf16(q_bits), shape.q_dim, *pools, out, ws)
    got = host_f32(out)
    assert np.isfinite(got).all()
    qf = W.bf16_bits_to_f32(q_bits)
    for t in rows:
        q = qf[t].reshape(shape.n_q_heads, -1)
        want = (oracle.attention_token_fp8kv(shape, b, t, int(b.past[t]), q, kp, vp, 0.125, 0.07) if fp8
                else oracle.attention_token(shape, b, t, int(b.past[t]), q, kp, vp))
        assert_close(got[t], want.reshape(-1), f"row {t} of {b.T}", max_abs=2e-2, rel_l2=1e-2)   # the attention stage's bar


@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
@pytest.mark.parametrize("page", [16, 256])
@pytest.mark.parametrize("shape", [W.TINY, W.TINY_GQA, W.TINY_G5, W.TINY_G3_D128], ids=["mha", "gqa", "g5", "g3d128"])
def test_rows_in_parts(rs, oracle, shape, page, fp8):
    shape = replace(shape, page_size=page)
    long = max(page, 1040 // page * page)            # a template of several chunks, not a multiple of 64 keys with small pages
    plen = [long, page]
    own = [1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 129, 300, 700]
    pid = [0, 1, -1, 0, 0, 1, 0, -1, 0, 1, 1, 0, 0, -1]
    ctx = [o + (plen[p] if p >= 0 else 0) for o, p in zip(own, pid)]
    _check(rs, oracle, shape, W.build_batch(shape, [1] * len(own), ctx, pid, plen, seed=5), range(len(own)), fp8)


@pytest.mark.parametrize("n", [1, 2, 3, 255, 256])
def test_batch_sizes(rs, oracle, n):
    """Up to the largest batch that keeps its parts in slots; a single row has no group and is cut by its length alone."""
    shape = W.TINY_GQA
    rng = np.random.default_rng(n)
    own = rng.integers(1, 200, n)
    own[0] = 900
    b = W.build_batch(shape, [1] * n, 272 + own, [0] * n, [272], seed=6)
    _check(rs, oracle, shape, b, np.unique(np.concatenate([[0, n - 1], rng.integers(0, n, 12)])))


@pytest.mark.parametrize("members", [6, 1], ids=["template", "own"])
def test_parts_without_a_finite_score(rs, oracle, members):
    """Keys whose scores are -inf have no weight: a row whose first part holds nothing else takes its value from the rest."""
    shape = W.TINY_GQA
    b = W.build_batch(shape, [1] * members, [1040 + 100] * members, [0] * members, [1040], seed=9)
    rng = np.random.default_rng(3)
    q = np.abs(rng.standard_normal((b.T, shape.n_q_heads, shape.head_dim), dtype=np.float32))
    q_bits = W.f32_to_bf16_bits(q.reshape(b.T, -1))
    kp, vp = W.make_cache(shape, b.num_pages, 11)
    for page in np.asarray(b.block_table).reshape(members, -1)[0, :192 // shape.page_size]:   # the first 192 keys, shared by all rows
        kp[page, :, :, 0] = 0xff80                                                            # -inf
    layer = rs.relserve_layer_create(shape)
    pb = rs.relserve_batch_prepare(layer, b)
    ws = torch.full((rs.relserve_workspace_bytes(layer, b.T),), 0xff, dtype=torch.uint8, device="cuda")
    out = torch.zeros(b.T, shape.q_dim, dtype=torch.bfloat16, device="cuda")
    rs.relserve_attention(layer, pb, dev_bf16(q_bits), shape.q_dim, dev_bf16(kp), dev_bf16(vp), out, ws)
    got, qf = host_f32(out), W.bf16_bits_to_f32(q_bits)
    for t in range(members):
        want = oracle.attention_token(shape, b, t, int(b.past[t]), qf[t].reshape(shape.n_q_heads, -1), kp, vp)
        assert np.isfinite(want).all()
        assert_close(got[t], want.reshape(-1), f"row {t}", max_abs=2e-2, rel_l2=1e-2)   # the attention stage's bar
