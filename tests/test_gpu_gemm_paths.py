"""Launch rules of the projections at the sizes where they change over (GPU): tile edges, remainders, both ends of a range."""
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


@pytest.mark.parametrize("T", [1, 64, 65, 128, 129, 192, 193, 256])
def test_wide_output_of_few_rows(rs, oracle, T):
    """The output layer's shape: few rows, so many features (and a last tile of four) that whole tiles fill the chip."""
    N, K = 206 * 128 + 4, 192
    rng = np.random.default_rng(T)
    ab = W.f32_to_bf16_bits(rng.standard_normal((T, K), dtype=np.float32))
    wb = W.f32_to_bf16_bits(rng.standard_normal((N, K), dtype=np.float32) * 0.05)
    rows = np.unique([0, T // 2, T - 1])
    want = oracle.linear(wb, W.bf16_bits_to_f32(ab[rows]))
    a, w = dev_bf16(ab), dev_bf16(wb)
    out = torch.full((T, N), float("nan"), dtype=torch.float32, device="cuda")
    rs.relserve_linear(a, w, 1, None, out)
    scale = max(1.0, np.abs(want).max())
    assert torch.isfinite(out).all()
    # exact products, fp32 sums in another order: 192 roundings of 2^-24 each, as the other epilogue tests allow
    assert_close(host_f32(out)[rows], want, "wide", max_abs=1e-3 * scale, rel_l2=1e-4)
    resb = W.f32_to_bf16_bits(rng.standard_normal((T, N), dtype=np.float32))
    rs.relserve_linear(a, w, 1, dev_bf16(resb), out)
    assert_close(host_f32(out)[rows], want + W.bf16_bits_to_f32(resb[rows]), "wide + residual", max_abs=1e-3 * scale, rel_l2=1e-4)


@pytest.mark.parametrize("T", [129, 160, 192, 193, 255, 256])
@pytest.mark.parametrize("packed", [False, True])
def test_one_token_tile_of_192_or_256_rows(rs, oracle, T, packed):
    """Projections of 129 .. 256 tokens inside a layer step (the entry that has split scratch): k split over workgroups for
    every projection, and a gate/up projection that is wide enough to run whole."""
    for shape in (W.LayerShape(512, 4, 2, 128, 704, 16, 1e-5, 10000.0), W.LayerShape(256, 4, 4, 64, 8256, 16, 1e-5, 10000.0)):
        b = W.build_batch(shape, [T - 7] + [1] * 7, [T - 7] + [5] * 7, seed=T)
        wl = W.Workload("one_tile", shape, b, T)
        weights, x = wl.weights(), W.make_activations(b.T, shape.hidden, T)
        kp, vp = W.make_cache(shape, b.num_pages, T)
        wd = {k: dev_bf16(v) for k, v in weights.items()}
        if packed:
            wd = rs.pack_layer_weights(wd)
        layer = rs.relserve_layer_create(shape)
        pb = rs.relserve_batch_prepare(layer, b)
        ws = torch.full((rs.relserve_workspace_bytes(layer, b.T),), 0xff, dtype=torch.uint8, device="cuda")
        xd = dev_bf16(x)
        y = torch.empty_like(xd)
        rs.relserve_layer_step(layer, pb, wd, xd, y, dev_bf16(kp), dev_bf16(vp), ws)
        want = oracle.layer_step(shape, b, weights, x, kp, vp).y_f32
        assert_close(host_f32(y), want, f"step T={T}")     # the whole step's bar
