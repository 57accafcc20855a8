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
