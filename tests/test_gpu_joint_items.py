"""Prefill rows of a group whose items walk the shared keys and then each request's own (GPU), against the CPU oracle: requests that
end inside, at and behind an item, templates of no multiple of 64 keys, decode rows and other groups beside them."""
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
