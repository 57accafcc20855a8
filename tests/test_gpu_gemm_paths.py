"""Launch rules of the projections at the sizes where they change over (GPU): tile edges, remainders, both ends of a range."""
import numpy as np
import pytest
import torch

from paper_2601_11546_amd import duration_model
from paper_2601_11546_amd import workloads as W
from tests import host_program
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


@pytest.mark.parametrize("w8a8", [False, True], ids=["bf16", "codes"])
@pytest.mark.parametrize("T", [1, 300])
def test_whole_tiles_of_any_shape_give_the_same_bits(rs, T, w8a8):
    """The tile shape of a projection that splits nothing is a matter of time alone: one running sum over k each."""
    N, K = 1168, 640
    g = torch.Generator(device="cuda").manual_seed(T)
    if w8a8:
        def codes(*s):
            return torch.randint(0, 120, s, generator=g, device="cuda", dtype=torch.uint8) | (torch.randint(0, 2, s, generator=g, device="cuda", dtype=torch.uint8) << 7)
        a, w, sw = codes(T, K), codes(N, K), torch.rand(N, generator=g, device="cuda") * 1e-3
        run = lambda epi, res, out: rs.relserve_linear_w8a8(a, w, sw, 0.03, epi, res, out)
    else:
        a = torch.randn(T, K, generator=g, device="cuda").bfloat16()
        w = (torch.randn(N, K, generator=g, device="cuda") * 0.05).bfloat16()
        run = lambda epi, res, out: rs.relserve_linear(a, w, epi, res, out)
    rb, rf = torch.randn(T, N, generator=g, device="cuda").bfloat16(), torch.randn(T, N, generator=g, device="cuda")
    for epi, res, cols, dtype in ((0, None, N, torch.bfloat16), (1, rb, N, torch.float32), (2, rf, N, torch.bfloat16), (3, None, N // 2, torch.bfloat16)):
        outs = []
        for tile in (-1, 0, 1, 2, 3, 4):
            out = torch.empty(T, cols, dtype=dtype, device="cuda")
            rs.relserve_debug_force_gemm_plan(tile, 0)
            try:
                run(epi, res, out)
                torch.cuda.synchronize()
            finally:
                rs.relserve_debug_force_gemm_plan(-1, 0)
            outs.append(out)
        for tile, out in enumerate(outs[1:]):
            assert torch.equal(out, outs[0]), (epi, tile)


@pytest.mark.parametrize("w8a8", [False, True], ids=["bf16", "codes"])
@pytest.mark.parametrize("packed", [False, True], ids=["rows", "packed"])
@pytest.mark.parametrize("nk", [1, 2, 3, 4, 5, 7])
def test_rings_of_few_stages(rs, nk, packed, w8a8):
    """Every tile shape where k is as short as its rings of stages and shorter: what a hand-over refills ends with the matrix.  Integers
    and multiples of 1/64 (codes: 0, 1 and 2): every order of the sums is exact, so every tile has the product's own bits."""
    T, N = 257, 520
    g = torch.Generator(device="cuda").manual_seed(nk)
    if w8a8:
        K = 128 * nk
        codes = lambda *s: torch.tensor([0, 0x38, 0x40], dtype=torch.uint8, device="cuda")[torch.randint(0, 3, s, generator=g, device="cuda")]
        value = lambda c: c.view(torch.float8_e4m3fn).double()
        a, w, sw = codes(T, K), codes(N, K), torch.full((N,), 0.5, device="cuda")
        want = (value(a).cpu() @ value(w).cpu().T * 0.25).float()
        wp = rs.pack_codes(w) if packed else w
        run = lambda out: rs.relserve_linear_w8a8(a, wp, sw, 0.5, 1, None, out, n=N if packed else 0)
    else:
        K = 64 * nk
        a = torch.randint(-4, 5, (T, K), generator=g, device="cuda").bfloat16()
        w = (torch.randint(-4, 5, (N, K), generator=g, device="cuda").float() / 64).bfloat16()
        want = (a.double().cpu() @ w.double().cpu().T).float()
        if packed:
            wp = torch.empty(rs.relserve_packed_weight_elems(N, K), dtype=torch.bfloat16, device="cuda")
            rs.relserve_pack_weight(w, wp)
            run = lambda out: rs.relserve_linear_packed(a, wp, N, 1, None, out)
        else:
            run = lambda out: rs.relserve_linear(a, w, 1, None, out)
    for tile in (-1, 0, 1, 2, 3, 4):
        out = torch.full((T, N), float("nan"), dtype=torch.float32, device="cuda")
        rs.relserve_debug_force_gemm_plan(tile, 0)
        try:
            run(out)
            torch.cuda.synchronize()
        finally:
            rs.relserve_debug_force_gemm_plan(-1, 0)
        assert torch.equal(out.cpu(), want), tile


@pytest.mark.parametrize("N, shift", [(512, 0), (512, 4), (516, 0), (516, 4), (252, 4)])
def test_rows_that_end_or_begin_inside_a_group_of_8(rs, N, shift):
    """bf16 rows are stored 8 features at a time where whole groups begin at 16-byte boundaries: rows of no multiple of 8, and rows that
    begin 8 bytes further on, are stored 4 by 4.  Exact sums, as above; nothing behind the last row is touched."""
    T, K = 259, 128
    g = torch.Generator(device="cuda").manual_seed(N + shift)
    a = torch.randint(-4, 5, (T, K), generator=g, device="cuda").bfloat16()
    w = (torch.randint(-4, 5, (N, K), generator=g, device="cuda").float() / 64).bfloat16()
    res = torch.randint(-8, 9, (T, N), generator=g, device="cuda").float()
    sums = (a.double().cpu() @ w.double().cpu().T).float()
    for epi, want in ((0, sums.bfloat16()), (2, (sums + res.cpu()).bfloat16())):
        for tile in (0, 1, 2, 3, 4):
            buf = torch.full((shift + T * N + 64,), 7.0, dtype=torch.bfloat16, device="cuda")
            out = buf[shift:shift + T * N].view(T, N)
            rs.relserve_debug_force_gemm_plan(tile, 0)
            try:
                rs.relserve_linear(a, w, epi, res if epi == 2 else None, out)
                torch.cuda.synchronize()
            finally:
                rs.relserve_debug_force_gemm_plan(-1, 0)
            assert torch.equal(out.cpu(), want), (epi, tile)
            assert (buf[:shift] == 7).all() and (buf[shift + T * N:] == 7).all(), (epi, tile)


@pytest.mark.parametrize("w8a8", [False, True], ids=["bf16", "codes"])
@pytest.mark.parametrize("T", [1, 63, 259])
@pytest.mark.parametrize("N", [4, 60, 68, 132, 512, 516])
def test_fp32_rows_that_end_inside_a_group_of_64(rs, N, T, w8a8):
    """Rows of fp32 are stored 64 features at a time by 16 lanes, four tokens by four: rows of features that end inside a group and
    tokens that end inside four, on every tile shape and on the kernel for k of no multiple of 64.  Exact sums, as above; nothing behind
    the last row is touched."""
    g = torch.Generator(device="cuda").manual_seed(N + T)
    res = torch.randint(-8, 9, (T, N), generator=g, device="cuda").bfloat16()
    for K in (128, 384) if w8a8 else (64, 72, 320):
        if w8a8:
            codes = lambda *s: torch.tensor([0, 0x38, 0x40], dtype=torch.uint8, device="cuda")[torch.randint(0, 3, s, generator=g, device="cuda")]
            value = lambda c: c.view(torch.float8_e4m3fn).double().cpu()
            a, w = codes(T, K), codes(N, K)
            sw = 2.0 ** torch.randint(-3, 4, (N,), generator=g, device="cuda").float()
            sums = ((value(a) @ value(w).T) * (0.5 * sw.double().cpu())).float()
            run = lambda r, out: rs.relserve_linear_w8a8(a, w, sw, 0.5, 1, r, out)
        else:
            a = torch.randint(-4, 5, (T, K), generator=g, device="cuda").bfloat16()
            w = (torch.randint(-4, 5, (N, K), generator=g, device="cuda").float() / 64).bfloat16()
            sums = (a.double().cpu() @ w.double().cpu().T).float()
            run = lambda r, out: rs.relserve_linear(a, w, 1, r, out)
        for r, want in ((None, sums), (res, sums + res.float().cpu())):
            for tile in (-1, 0, 1, 2, 3, 4):
                buf = torch.full((T * N + 64,), 7.0, dtype=torch.float32, device="cuda")
                rs.relserve_debug_force_gemm_plan(tile, 0)
                try:
                    run(r, buf[:T * N].view(T, N))
                    torch.cuda.synchronize()
                finally:
                    rs.relserve_debug_force_gemm_plan(-1, 0)
                assert torch.equal(buf[:T * N].view(T, N).cpu(), want), (K, tile)
                assert (buf[T * N:] == 7).all(), (K, tile)


@pytest.mark.parametrize("T", [5, 64, 67, 128, 140, 192, 250, 256, 300])
def test_slabs_of_rows_that_end_inside_a_group_of_64(rs, oracle, T):
    """Split projections onto 520 features (W_o of k = 512, W_down of k = 704) beside unsplit ones of k = 520, on one row of tiles of
    every height and on two."""
    shape = W.LayerShape(520, 4, 2, 128, 704, 16, 1e-5, 10000.0)
    b = W.build_batch(shape, [T - 4] + [1] * 4, [T - 4] + [5] * 4, seed=T)
    wl = W.Workload("ragged_rows", shape, b, T)
    weights, x = wl.weights(), W.make_activations(b.T, shape.hidden, T)
    kp, vp = W.make_cache(shape, b.num_pages, T)
    layer = rs.relserve_layer_create(shape)
    pb = rs.relserve_batch_prepare(layer, b)
    ws = torch.full((rs.relserve_workspace_bytes(layer, b.T),), 0xff, dtype=torch.uint8, device="cuda")
    xd = dev_bf16(x)
    y = torch.empty_like(xd)
    rs.relserve_layer_step(layer, pb, {k: dev_bf16(v) for k, v in weights.items()}, xd, y, dev_bf16(kp), dev_bf16(vp), ws)
    torch.cuda.synchronize()
    assert_close(host_f32(y), oracle.layer_step(shape, b, weights, x, kp, vp).y_f32, f"step T={T}")     # the whole step's bar


@pytest.mark.parametrize("T", [257, 482, 1308])
@pytest.mark.parametrize("hidden", [192, 256, 448, 512])
def test_short_k_takes_whole_tiles_at_mid_size(rs, T, hidden):
    """Narrow layers at a few hundred tokens: k below 512 is not cut and runs as whole tiles, 512 is cut in two; both agree
    with forced whole tiles as sums in another order do."""
    shape = W.LayerShape(hidden, 4, 4, 64, 704, 16, 1e-5, 10000.0)
    b = W.build_batch(shape, [T - 7] + [1] * 7, [T - 7] + [5] * 7, seed=T)
    g = torch.Generator(device="cuda").manual_seed(hidden)
    randn = lambda *s, std=0.05: torch.empty(*s, dtype=torch.float32, device="cuda").normal_(0, std, generator=g).bfloat16()
    wd = {"w_in_norm": randn(hidden, std=1.0), "w_qkv": randn(shape.qkv_dim, hidden), "w_o": randn(hidden, shape.q_dim), "w_post_norm": randn(hidden, std=1.0),
          "w_gate_up": randn(2 * 704, hidden), "w_down": randn(hidden, 704)}
    x = randn(b.T, hidden, std=1.0)
    pool = (b.num_pages, shape.page_size, shape.n_kv_heads, shape.head_dim)
    k, v = randn(*pool, std=1.0), randn(*pool, std=1.0)
    layer = rs.relserve_layer_create(shape)
    pb = rs.relserve_batch_prepare(layer, b)
    ws = torch.empty(rs.relserve_workspace_bytes(layer, b.T), dtype=torch.uint8, device="cuda")
    outs = []
    for tile in (-1, 3):
        y = torch.empty_like(x)
        rs.relserve_debug_force_gemm_plan(tile, 0)
        try:
            rs.relserve_layer_step(layer, pb, wd, x, y, k.clone(), v.clone(), ws)
            torch.cuda.synchronize()
        finally:
            rs.relserve_debug_force_gemm_plan(-1, 0)
        outs.append(y.float().cpu().numpy())
    # W_down (k = 704) is cut in two on one side: rounded once to bf16, so a value in some thousands lies one unit apart
    assert_close(outs[0], outs[1], f"T={T} hidden={hidden}", max_abs=2e-2 * max(1.0, np.abs(outs[1]).max()), rel_l2=2e-3)


@pytest.mark.parametrize("w8a8", [False, True], ids=["bf16", "codes"])
@pytest.mark.parametrize("T", [385, 577, 640, 806, 1409])
@pytest.mark.parametrize("epi, N", [(1, 11012), (3, 27648), (0, 7176)])
def test_columns_of_two_tile_shapes_give_the_same_bits(rs, T, epi, N, w8a8):
    """Sizes whose whole tiles fill their last round badly run as two launches, each its own columns and tile shape: the bits of one shape,
    every column written once.  (1409 tokens of the last two and 385 of the first keep one launch.)"""
    K = 5120 if w8a8 else 2560
    g = torch.Generator(device="cuda").manual_seed(T + N)
    if w8a8:
        codes = lambda *s: (torch.randn(s, generator=g, device="cuda") * 60).to(torch.float8_e4m3fn).view(torch.uint8)
        a, w, sw = codes(T, K), codes(N, K), torch.rand(N, generator=g, device="cuda") * 1e-4
        run = lambda res, out: rs.relserve_linear_w8a8(a, w, sw, 0.03, epi, res, out)
    else:
        a = torch.randn(T, K, generator=g, device="cuda").bfloat16()
        w = (torch.randn(N, K, generator=g, device="cuda") * 0.02).bfloat16()
        run = lambda res, out: rs.relserve_linear(a, w, epi, res, out)
    res = torch.randn(T, N, generator=g, device="cuda").bfloat16() if epi == 1 else None
    outs = []
    for tile in (-1, 0):
        out = torch.full((T, N // 2 if epi == 3 else N), float("nan"), dtype=torch.float32 if epi == 1 else torch.bfloat16, device="cuda")
        rs.relserve_debug_force_gemm_plan(tile, 0)
        try:
            run(res, out)
            torch.cuda.synchronize()
        finally:
            rs.relserve_debug_force_gemm_plan(-1, 0)
        outs.append(out)
    assert torch.isfinite(outs[1]).all() and torch.equal(outs[0], outs[1])


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    exe = host_program.build(tmp_path_factory.mktemp("launches"), "gemm_launches")
    return lambda *row: host_program.run(exe, "%d %d %d %d %d %d\n" % row)[0]


def _one_shape_or_two(rs, launches, row, run, outs):
    """outs: what run() writes; on the automatic choice, which has to be two launches, and on one shape of 256 x 256."""
    assert launches(*row)[4] > 0, "the size is meant to run as two launches"
    got = []
    for tile in (-1, 0):
        for o in outs:
            o.fill_(float("nan"))
        rs.relserve_debug_force_gemm_plan(tile, 0)
        try:
            run()
            torch.cuda.synchronize()
        finally:
            rs.relserve_debug_force_gemm_plan(-1, 0)
        got.append([o.clone() for o in outs])
    for two, one in zip(*got):
        assert torch.isfinite(one).all() and torch.equal(two, one)


@pytest.mark.parametrize("w8a8", [False, True], ids=["bf16", "codes"])
@pytest.mark.parametrize("T, epi, N", [(1409, 0, 11012), (3300, 0, 5524), (1409, 1, 11012), (1500, 1, 11012), (1409, 2, 11012),
                                       (806, 3, 27664), (2000, 3, 13840)])
def test_two_launches_write_every_column_once(rs, launches, T, epi, N, w8a8):
    """Sizes that do run as two launches (the plan is asked), with tokens and features that end inside a tile: the bits of one shape."""
    K = 5120 if w8a8 else 2560
    g = torch.Generator(device="cuda").manual_seed(T + N)
    res = None if epi in (0, 3) else torch.randn(T, N, generator=g, device="cuda", dtype=torch.bfloat16 if epi == 1 else torch.float32)
    out = torch.empty((T, N // 2 if epi == 3 else N), dtype=torch.float32 if epi == 1 else torch.bfloat16, device="cuda")
    if w8a8:
        codes = lambda *s: (torch.randn(s, generator=g, device="cuda") * 60).to(torch.float8_e4m3fn).view(torch.uint8)
        a, w, sw = codes(T, K), codes(N, K), torch.rand(N, generator=g, device="cuda") * 1e-4
        run = lambda: rs.relserve_linear_w8a8(a, w, sw, 0.03, epi, res, out)
    else:
        a = torch.randn(T, K, generator=g, device="cuda").bfloat16()
        w = (torch.randn(N, K, generator=g, device="cuda") * 0.02).bfloat16()
        run = lambda: rs.relserve_linear(a, w, epi, res, out)
    _one_shape_or_two(rs, launches, (T, N, 2560, 0, int(epi == 3), 0), run, [out])


@pytest.mark.parametrize("n_q, n_kv, d", [(75, 5, 128), (150, 10, 64)])
def test_two_launches_of_the_qkv_projection(rs, launches, n_q, n_kv, d):
    """The same where the epilogue rotates and appends: queries, keys and values, the last tile half a column."""
    T, K = 1409, 2560
    shape = W.LayerShape(K, n_q, n_kv, d, 704, 16, 1e-5, 10000.0)
    g = torch.Generator(device="cuda").manual_seed(d)
    b = W.build_batch(shape, [T - 9] + [1] * 9, [T - 9] + [40] * 9, seed=3)
    layer = rs.relserve_layer_create(shape)
    pb = rs.relserve_batch_prepare(layer, b)
    h = torch.randn(T, K, generator=g, device="cuda").bfloat16()
    w = (torch.randn(shape.qkv_dim, K, generator=g, device="cuda") * 0.02).bfloat16()
    q = torch.empty(T, n_q * d, dtype=torch.bfloat16, device="cuda")
    kd, vd = (torch.zeros(b.num_pages, 16, n_kv, d, dtype=torch.bfloat16, device="cuda") for _ in range(2))

    def run():   # slots that no token of the batch takes keep what they hold
        kd.zero_()
        vd.zero_()
        rs.relserve_qkv_rope_append(layer, pb, h, w, q, kd, vd)
    _one_shape_or_two(rs, launches, (T, shape.qkv_dim, K, 1, 0, 0), run, [q, kd, vd])


@pytest.mark.parametrize("T, shape, w8a8", [
    # tiles of 256 and of 192 rows are all tail (13 x 9 and 17 or 18 x 9), two ranges each; k of 36, 32 and 17 slices, of 35, 16 and 18
    (3132, W.LayerShape(2304, 16, 1, 128, 1088, 16, 1e-5, 10000.0), False), (3272, W.LayerShape(2304, 16, 1, 128, 1088, 16, 1e-5, 10000.0), False),
    (3132, W.LayerShape(2304, 32, 2, 64, 1088, 16, 1e-5, 10000.0), False), (3272, W.LayerShape(2240, 8, 8, 128, 1152, 16, 1e-5, 10000.0), False),
    # tails of two tiles beside 256 whole ones (gate/up); W_down of k = 16448
    (300, W.LayerShape(1024, 8, 8, 128, 16448, 16, 1e-5, 10000.0), False),
    (3132, W.LayerShape(2304, 16, 1, 128, 1152, 16, 1e-5, 10000.0), True), (300, W.LayerShape(2048, 16, 4, 128, 2176, 16, 1e-5, 10000.0), True),
])
def test_two_k_ranges_on_either_tile_give_the_same_bits(rs, T, shape, w8a8):
    """256-row tiles of two k ranges, as halves (16-bit, where the rule says so) or through slabs and their finish kernel, against slabs and
    finish of 192-row tiles: the same ranges, the same order of additions.  The last 256 rows hold 60, 200 or 44: halves with and without a lower one."""
    b = W.build_batch(shape, [100] * (T // 100) + ([T % 100] if T % 100 else []), [100] * (T // 100) + ([T % 100] if T % 100 else []), seed=T)
    g = torch.Generator(device="cuda").manual_seed(T)
    randn = lambda *s, std=0.05: torch.empty(*s, dtype=torch.float32, device="cuda").normal_(0, std, generator=g).bfloat16()
    H, I = shape.hidden, shape.mlp_dim
    wd = {"w_in_norm": randn(H, std=1.0), "w_qkv": randn(shape.qkv_dim, H), "w_o": randn(H, shape.q_dim), "w_post_norm": randn(H, std=1.0),
          "w_gate_up": randn(2 * I, H), "w_down": randn(H, I)}
    step = rs.relserve_layer_step
    if w8a8:
        wd, step = duration_model.quantise_layer_on_device(torch, wd), rs.relserve_layer_step_w8a8
    x = randn(b.T, H, std=1.0)
    pool = (b.num_pages, shape.page_size, shape.n_kv_heads, shape.head_dim)
    layer = rs.relserve_layer_create(shape)
    pb = rs.relserve_batch_prepare(layer, b)
    ws = torch.empty(rs.relserve_workspace_bytes(layer, b.T), dtype=torch.uint8, device="cuda")
    outs = []
    for tile in (0, 1):
        y, k, v = torch.empty_like(x), torch.zeros(pool, dtype=torch.bfloat16, device="cuda"), torch.zeros(pool, dtype=torch.bfloat16, device="cuda")
        rs.relserve_debug_force_gemm_plan(tile, 2)
        try:
            step(layer, pb, wd, x, y, k, v, ws)
            torch.cuda.synchronize()
        finally:
            rs.relserve_debug_force_gemm_plan(-1, 0)
        outs.append((y, k, v))
    assert torch.isfinite(outs[0][0]).all()
    for name, got, want in zip("ykv", *outs):
        assert torch.equal(got.view(torch.int16), want.view(torch.int16)), name


def test_iteration_of_640_tokens_keeps_its_sums_whole(rs):
    """The q/k/v projection of a 13B layer at T = 640 (128 decode rows and a 512-token chunk) fills its rounds well enough to
    split nothing: the appended keys and values carry the bits of whole tiles, as its gate/up projection's sums do."""
    shape = W.LLAMA_13B
    b = W.build_batch(shape, [512] + [1] * 128, [512] + [40] * 128, seed=1)
    g = torch.Generator(device="cuda").manual_seed(2)
    randn = lambda *s, std=0.02: torch.empty(*s, dtype=torch.float32, device="cuda").normal_(0, std, generator=g).bfloat16()
    H, I = shape.hidden, shape.mlp_dim
    wd = {"w_in_norm": randn(H, std=1.0), "w_qkv": randn(shape.qkv_dim, H), "w_o": randn(H, shape.q_dim), "w_post_norm": randn(H, std=1.0),
          "w_gate_up": randn(2 * I, H), "w_down": randn(H, I)}
    x = randn(b.T, H, std=1.0)
    pool = (b.num_pages, shape.page_size, shape.n_kv_heads, shape.head_dim)
    cached = randn(*pool, std=1.0), randn(*pool, std=1.0)
    layer = rs.relserve_layer_create(shape)
    pb = rs.relserve_batch_prepare(layer, b)
    ws = torch.empty(rs.relserve_workspace_bytes(layer, b.T), dtype=torch.uint8, device="cuda")
    pools = []
    for tile in (-1, 0, 1, 2):
        k, v, y = cached[0].clone(), cached[1].clone(), torch.empty_like(x)
        rs.relserve_debug_force_gemm_plan(tile, 0)
        try:
            rs.relserve_layer_step(layer, pb, wd, x, y, k, v, ws)
            torch.cuda.synchronize()
        finally:
            rs.relserve_debug_force_gemm_plan(-1, 0)
        pools.append((k, v))
    for tile, (k, v) in enumerate(pools[1:]):
        assert torch.equal(k, pools[0][0]) and torch.equal(v, pools[0][1]), tile


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
def test_rotation_rounds_the_same_on_every_path(rs, d, fp8):
    """Activations of +-1 and weights that are multiples of 1/64: every order of a sum is exact, so the appended keys and values of
    a token differ between the paths (k split over workgroups, split tail, whole tiles) only if the rotation rounds differently."""
    shape = W.LayerShape(4096, 2048 // d, 1024 // d, d, 512, 16, 1e-5, 10000.0)    # q/k/v at 300 tokens: 32 tiles split 4 ways
    g = torch.Generator(device="cuda").manual_seed(d)
    H, I = shape.hidden, shape.mlp_dim
    ones = torch.ones(H, device="cuda", dtype=torch.bfloat16)
    ints = lambda *s: (torch.randint(-4, 5, s, generator=g, device="cuda").float() / 64).bfloat16()
    wd = {"w_in_norm": ones, "w_qkv": ints(shape.qkv_dim, H), "w_o": ints(H, shape.q_dim), "w_post_norm": ones, "w_gate_up": ints(2 * I, H),
          "w_down": ints(H, I)}
    x = (torch.randint(0, 2, (300, H), generator=g, device="cuda") * 2 - 1).to(torch.bfloat16)
    layer = rs.relserve_layer_create(shape)
    want = None
    for T, tile in ((60, -1), (100, -1), (200, -1), (300, -1), (300, 0), (300, 1), (300, 2)):
        b = W.build_batch(shape, [T], [T], seed=0)
        b.block_table[:] = np.arange(b.block_table.size).reshape(b.block_table.shape)        # token t in slot t
        pb = rs.relserve_batch_prepare(layer, b)
        pool = lambda: torch.zeros(b.num_pages, 16, shape.n_kv_heads, d, device="cuda", dtype=torch.uint8 if fp8 else torch.bfloat16)
        k, v = pool(), pool()
        ws = torch.empty(rs.relserve_workspace_bytes(layer, T), dtype=torch.uint8, device="cuda")
        rs.relserve_debug_force_gemm_plan(tile, 0)
        try:
            rs.relserve_layer_step(layer, pb, wd, x[:T], torch.empty_like(x[:T]), *((rs.QuantPool(k, 0.05), rs.QuantPool(v, 0.05)) if fp8 else (k, v)), ws)
            torch.cuda.synchronize()
        finally:
            rs.relserve_debug_force_gemm_plan(-1, 0)
        got = [p.view(torch.uint8).reshape(-1, shape.kv_dim * (1 if fp8 else 2))[:60] for p in (k, v)]
        want = want or got
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), (T, tile)


@pytest.mark.parametrize("kind", ["rows", "packed", "codes", "packed codes"])
@pytest.mark.parametrize("T", [1, 64, 65, 129, 192, 193, 256])
def test_wide_output_of_other_operands(rs, oracle, T, kind):
    """test_wide_output_of_few_rows with a k long enough for the deep ring (1024 bytes a row), in both weight layouts and on 8-bit
    codes."""
    N, K = 206 * 128 + 4, 1024 if "codes" in kind else 512
    rng = np.random.default_rng(T)
    rows = np.unique([0, T // 2, T - 1])
    resb = W.f32_to_bf16_bits(rng.standard_normal((T, N), dtype=np.float32))
    out = torch.full((T, N), float("nan"), dtype=torch.float32, device="cuda")
    if "codes" not in kind:
        ab = W.f32_to_bf16_bits(rng.standard_normal((T, K), dtype=np.float32))
        wb = W.f32_to_bf16_bits(rng.standard_normal((N, K), dtype=np.float32) * 0.05)
        want = oracle.linear(wb, W.bf16_bits_to_f32(ab[rows]))
        if kind == "rows":
            rs.relserve_linear(dev_bf16(ab), dev_bf16(wb), 1, dev_bf16(resb), out)
        else:
            w = torch.empty(rs.relserve_packed_weight_elems(N, K), dtype=torch.bfloat16, device="cuda")
            rs.relserve_pack_weight(dev_bf16(wb), w)
            rs.relserve_linear_packed(dev_bf16(ab), w, N, 1, dev_bf16(resb), out)
    else:
        codes = lambda *s: W.nearest_e4m3_codes(rng.standard_normal(s).astype(np.float32) * np.float32(60))
        a, w = codes(T, K), codes(N, K)
        s_w = ((0.5 + rng.random(N)) * 1e-5).astype(np.float32)
        want = oracle.linear_w8a8(w, s_w, a[rows], 0.03)
        a, w, s_w = (torch.from_numpy(t).cuda() for t in (a, w, s_w))
        if kind == "codes":
            rs.relserve_linear_w8a8(a, w, s_w, 0.03, 1, dev_bf16(resb), out)
        else:
            rs.relserve_linear_w8a8(a, rs.pack_codes(w), s_w, 0.03, 1, dev_bf16(resb), out, n=N)
    scale = max(1.0, np.abs(want).max())
    assert torch.isfinite(out).all()
    # exact products, fp32 sums of 512 or 1024 in another order (the matrix unit's adder on codes), then one fp32 addition
    assert_close(host_f32(out)[rows], want + W.bf16_bits_to_f32(resb[rows]), f"wide {kind}", max_abs=1e-3 * scale, rel_l2=1e-4)


@pytest.mark.parametrize("w8a8", [False, True], ids=["bf16", "codes"])
@pytest.mark.parametrize("stages", [1, 2, 3, 4, 5, 8])
def test_ring_with_a_further_stage_of_weights(rs, stages, w8a8):
    """Tiles of 192 and 256 rows keep one stage more of the weights than of the activations: k of fewer stages than either ring
    holds, of just as many, and of more, against the tile whose rings are alike."""
    T, N, K = 70, 264, stages * (128 if w8a8 else 64)
    g = torch.Generator(device="cuda").manual_seed(stages)
    if w8a8:
        codes = lambda *s: torch.randint(0, 120, s, generator=g, device="cuda", dtype=torch.uint8) | (torch.randint(0, 2, s, generator=g, device="cuda", dtype=torch.uint8) << 7)
        a, w, sw = codes(T, K), codes(N, K), torch.rand(N, generator=g, device="cuda") * 1e-3
        run = lambda out: rs.relserve_linear_w8a8(a, w, sw, 0.03, 1, None, out)
        value = lambda c: c.view(torch.float8_e4m3fn).double()
        want = (value(a) @ value(w).T) * sw.double() * 0.03
    else:
        a = torch.randn(T, K, generator=g, device="cuda").bfloat16()
        w = (torch.randn(N, K, generator=g, device="cuda") * 0.05).bfloat16()
        run = lambda out: rs.relserve_linear(a, w, 1, None, out)
        want = a.double() @ w.double().T
    outs = []
    for tile in (3, 0, 1):
        outs.append(torch.full((T, N), float("nan"), dtype=torch.float32, device="cuda"))
        rs.relserve_debug_force_gemm_plan(tile, 0)
        try:
            run(outs[-1])
            torch.cuda.synchronize()
        finally:
            rs.relserve_debug_force_gemm_plan(-1, 0)
    # exact products; at most 1024 roundings of 2^-24 of partial sums that stay of the order of the result
    assert float((outs[0].double() - want).norm() / want.norm()) <= 1e-4
    for tile, out in zip((0, 1), outs[1:]):
        assert torch.equal(out, outs[0]), tile
