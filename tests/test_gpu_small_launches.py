"""The kernels between the projections at a few tokens (GPU): row lengths and numbers of k ranges where their code changes."""
import numpy as np
import pytest
import torch

from paper_2601_11546_amd import workloads as W
from tests.gpu_harness import dev_bf16, host_f32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rs():
    assert torch.cuda.is_available(), "GPU tests need a device"
    from paper_2601_11546_amd import binding
    return binding


@pytest.mark.parametrize("H", [8, 2040, 2048, 2056, 4104, 6144, 8192, 8200, 16384])
@pytest.mark.parametrize("f32", [False, True])
def test_rmsnorm_row_lengths(rs, H, f32):
    """1 .. 4 chunks per thread in registers, and the loop beyond; the last chunk of a row in every place."""
    g = torch.Generator(device="cuda").manual_seed(H)
    x = torch.randn(3, H, generator=g, device="cuda")
    x = x if f32 else x.bfloat16()
    w = (1 + 0.02 * torch.randn(H, generator=g, device="cuda")).bfloat16()
    out = torch.full((3, H), float("nan"), dtype=torch.bfloat16, device="cuda")
    rs.relserve_rmsnorm(x, w, 1e-5, out)
    xd = x.double()
    want = xd * w.double() / torch.sqrt((xd * xd).mean(1, keepdim=True) + 1e-5)
    # one bf16 rounding (2^-8 relative) on top of fp32 arithmetic (below 1e-5 relative)
    assert ((out.double() - want).abs() <= want.abs() * (2.0 ** -8 + 1e-5)).all()


@pytest.mark.parametrize("hidden, mlp", [(256, 64), (256, 512), (256, 1152), (256, 2112), (256, 2304), (256, 4352),   # k ranges of W_down
                                         (264, 64), (2048, 64), (8184, 64), (8192, 64), (8200, 64)])                # row of the fused norm
@pytest.mark.parametrize("T", [1, 5, 70])
def test_k_ranges_and_rows(rs, oracle, T, hidden, mlp):
    """W_down over 1 .. 17 k ranges: the sums of one, of up to eight and of more than eight slabs.  W_o's rows of 33 .. 1024
    chunks of eight, normed by the kernel that adds its slabs, and the first row too long for that."""
    shape = W.LayerShape(hidden, 4, 2, 64, mlp, 16, 1e-5, 10000.0)
    n_dec = max(1, T - 4)
    q = [T - n_dec] * (T > n_dec) + [1] * n_dec
    b = W.build_batch(shape, q, [n + 3 for n in q], seed=T + mlp)
    wl = W.Workload("k_ranges", shape, b, mlp)
    weights, x = wl.weights(), W.make_activations(b.T, shape.hidden, mlp)
    kp, vp = W.make_cache(shape, b.num_pages, mlp)
    layer = rs.relserve_layer_create(shape)
    pb = rs.relserve_batch_prepare(layer, b)
    ws = torch.full((rs.relserve_workspace_bytes(layer, b.T),), 0xff, dtype=torch.uint8, device="cuda")
    xd = dev_bf16(x)
    y = torch.empty_like(xd)
    rs.relserve_layer_step(layer, pb, {k: dev_bf16(v) for k, v in weights.items()}, xd, y, dev_bf16(kp), dev_bf16(vp), ws)
    want = oracle.layer_step(shape, b, weights, x, kp, vp).y_f32
    # the whole step's bar, plus the rounding of an output as large as these wide layers' (|y| up to 8): half a bf16 unit, 2^-9 |y|
    got = host_f32(y)
    assert np.linalg.norm(got - want) <= 1e-2 * np.linalg.norm(want)
    assert (np.abs(got - want) <= 2e-2 + np.abs(want) * 2.0 ** -9).all()


@pytest.mark.parametrize("T", [1, 31, 32, 33, 100])
@pytest.mark.parametrize("N, K", [(4, 16), (36, 48), (64, 128), (96, 144), (40, 688), (32, 1024)])
def test_small_projection_has_the_tiled_kernels_bits(rs, T, N, K):
    """One wave per tile of 32 x 32 (a forced tile takes the general path): remainders of tokens and features, one k step to the
    last allowed, whole and partial batches of eight steps."""
    g = torch.Generator(device="cuda").manual_seed(T * 1000 + K)
    a = torch.randn(T, K, generator=g, device="cuda").bfloat16()
    for epi, n, dtype in ((0, N, torch.bfloat16), (1, N, torch.float32), (2, N, torch.bfloat16), (3, 4 * N, torch.bfloat16)):
        w = (torch.randn(n, K, generator=g, device="cuda") * 0.05).bfloat16()
        res = torch.randn(T, n, generator=g, device="cuda")
        for r in {1: (None, res.bfloat16()), 2: (res,)}.get(epi, (None,)):
            outs = []
            for tile in (-1, 0):
                rs.relserve_debug_force_gemm_plan(tile, 0)
                try:
                    outs.append(torch.full((T, n // 2 if epi == 3 else n), float("nan"), dtype=dtype, device="cuda"))
                    rs.relserve_linear(a, w, epi, r, outs[-1])
                finally:
                    rs.relserve_debug_force_gemm_plan(-1, 0)
            assert torch.isfinite(outs[0]).all()
            assert torch.equal(outs[0].view(torch.uint8), outs[1].view(torch.uint8)), (epi, r is None)


@pytest.mark.parametrize("shape", [W.LayerShape(256, 3, 1, 64, 704, 16, 1e-5, 10000.0), W.LayerShape(192, 3, 1, 128, 704, 16, 1e-5, 10000.0)],
                         ids=["d64", "d128"])
@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("kv8", [False, True])
def test_small_layer_step_has_the_tiled_kernels_bits(rs, shape, packed, kv8):
    """q/k/v with rotation and append on both pool formats, and every projection that takes the small kernel, on both weight layouts."""
    b = W.build_batch(shape, [37, 1, 1, 24], [37, 9, 20, 30], seed=3)
    weights = {k: dev_bf16(v) for k, v in W.Workload("small", shape, b, 5).weights().items()}
    if packed:
        weights = rs.pack_layer_weights(weights)
    layer = rs.relserve_layer_create(shape)
    pb = rs.relserve_batch_prepare(layer, b)
    x = dev_bf16(W.make_activations(b.T, shape.hidden, 5))
    ws = torch.empty(rs.relserve_workspace_bytes(layer, b.T), dtype=torch.uint8, device="cuda")
    pools = (b.num_pages, shape.page_size, shape.n_kv_heads, shape.head_dim)
    outs = []
    for tile in (-1, 0):
        g = torch.Generator(device="cuda").manual_seed(1)
        if kv8:
            k, v = (torch.randint(0, 96, pools, generator=g, device="cuda", dtype=torch.uint8) for _ in range(2))
        else:
            k, v = (torch.randn(*pools, generator=g, device="cuda").bfloat16() for _ in range(2))
        y = torch.full_like(x, float("nan"))
        rs.relserve_debug_force_gemm_plan(tile, 0)
        try:
            rs.relserve_layer_step(layer, pb, weights, x, y, rs.QuantPool(k, 2.0 ** -4) if kv8 else k, rs.QuantPool(v, 2.0 ** -5) if kv8 else v, ws)
        finally:
            rs.relserve_debug_force_gemm_plan(-1, 0)
        outs.append((y, k, v))
    assert torch.isfinite(outs[0][0]).all()
    for name, got, want in zip("ykv", *outs):
        assert torch.equal(got.view(torch.uint8), want.view(torch.uint8)), name


@pytest.mark.parametrize("other_stream", [False, True], ids=["default", "other"])
def test_batches_destroyed_behind_their_work(rs, other_stream):
    """A destroyed batch's device allocation serves later ones: batches of different sizes prepared, stepped and destroyed one behind the
    other, with nothing waited for, give what each gives alone; on another stream than the default one they do so too."""
    shape = W.TINY_GQA
    g = torch.Generator(device="cuda").manual_seed(3)
    randn = lambda *s, std=0.05: torch.empty(*s, dtype=torch.float32, device="cuda").normal_(0, std, generator=g).bfloat16()
    H, I = shape.hidden, shape.mlp_dim
    wd = {"w_in_norm": randn(H, std=1.0), "w_qkv": randn(shape.qkv_dim, H), "w_o": randn(H, shape.q_dim), "w_post_norm": randn(H, std=1.0),
          "w_gate_up": randn(2 * I, H), "w_down": randn(H, I)}
    layer = rs.relserve_layer_create(shape)
    cases = []
    for T in (9, 64, 150, 333):
        b = W.build_batch(shape, [T - 7] + [1] * 7, [T - 7] + [5 + T // 8] * 7, seed=T)
        pool = (b.num_pages, shape.page_size, shape.n_kv_heads, shape.head_dim)
        cases.append((b, randn(b.T, H, std=1.0), randn(*pool, std=1.0), randn(*pool, std=1.0)))
    ws = torch.empty(max(rs.relserve_workspace_bytes(layer, c[0].T) for c in cases), dtype=torch.uint8, device="cuda")

    def step(c, stream=None):
        b, x, k, v = c
        y = torch.empty_like(x)
        pb = rs.relserve_batch_prepare(layer, b, stream=stream)
        rs.relserve_layer_step(layer, pb, wd, x, y, k, v, ws, stream=stream)
        pb.close()
        return y

    want = []
    for c in cases:
        want.append(step(c))
        torch.cuda.synchronize()
    s = torch.cuda.Stream() if other_stream else None
    if s:
        s.wait_stream(torch.cuda.current_stream())
    got = []
    for i in range(48):   # the keys and values a step appends are the same every time
        c = cases[(i * 7 + i // 4) % 4]
        got.append(((i * 7 + i // 4) % 4, step(c, s)))
    torch.cuda.synchronize()
    for i, y in got:
        assert torch.equal(y, want[i]), i


def _tiny_steps(rs, n):
    """n prepared-elsewhere batches of one size class and other contents: (layer, weights, [(batch, x, k, v, what its step gives)])."""
    shape = W.TINY_GQA
    g = torch.Generator(device="cuda").manual_seed(5)
    randn = lambda *s, std=0.05: torch.empty(*s, dtype=torch.float32, device="cuda").normal_(0, std, generator=g).bfloat16()
    H, I = shape.hidden, shape.mlp_dim
    wd = {"w_in_norm": randn(H, std=1.0), "w_qkv": randn(shape.qkv_dim, H), "w_o": randn(H, shape.q_dim), "w_post_norm": randn(H, std=1.0),
          "w_gate_up": randn(2 * I, H), "w_down": randn(H, I)}
    layer = rs.relserve_layer_create(shape)
    cases = []
    for i in range(n):
        b = W.build_batch(shape, [60 - 4 * i] + [1] * (4 * i + 6), [60 - 4 * i] + [9 + i] * (4 * i + 6), seed=40 + i)
        pool = (b.num_pages, shape.page_size, shape.n_kv_heads, shape.head_dim)
        x, k, v = randn(b.T, H, std=1.0), randn(*pool, std=1.0), randn(*pool, std=1.0)
        y = torch.empty_like(x)
        pb = rs.relserve_batch_prepare(layer, b)
        rs.relserve_layer_step(layer, pb, wd, x, y, k, v, torch.empty(rs.relserve_workspace_bytes(layer, b.T), dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        pb.close()
        cases.append((b, x, k, v, y))
    return layer, wd, cases


@pytest.mark.parametrize("first", ["default", "other"])
def test_allocation_of_a_batch_whose_work_is_outstanding(rs, first):
    """A batch's step waits behind long work on one stream, the batch is destroyed, and another stream prepares and steps the next one,
    whose tables differ: neither sees the other's."""
    layer, wd, cases = _tiny_steps(rs, 6)
    other = torch.cuda.Stream()
    streams = [torch.cuda.default_stream(), other] if first == "default" else [other, torch.cuda.default_stream()]
    got = []
    torch.cuda.synchronize()
    for i in range(0, 6, 2):
        for s, (b, x, k, v, _) in zip(streams, cases[i:i + 2]):
            with torch.cuda.stream(s):
                y = torch.full_like(x, float("nan"))
                ws = torch.empty(rs.relserve_workspace_bytes(layer, b.T), dtype=torch.uint8, device="cuda")
                pb = rs.relserve_batch_prepare(layer, b, stream=s)
                if s is streams[0]:
                    torch.cuda._sleep(20_000_000)   # some ms; prepare itself waits for its stream
                rs.relserve_layer_step(layer, pb, wd, x, y, k, v, ws, stream=s)
                pb.close()
                got.append((y, ws))
    torch.cuda.synchronize()
    for (y, _), case in zip(got, cases):
        assert torch.equal(y, case[4])


def test_handles_destroyed_inside_a_capture(rs):
    """A program that captures may let go of old handles meanwhile: the capture goes on, and its graph gives the eager results."""
    layer, wd, cases = _tiny_steps(rs, 3)
    b, x, k, v, want = cases[0]
    keep = rs.relserve_batch_prepare(layer, b)
    ws = torch.empty(rs.relserve_workspace_bytes(layer, b.T), dtype=torch.uint8, device="cuda")
    ws2 = torch.empty(rs.relserve_workspace_bytes(layer, cases[1][0].T), dtype=torch.uint8, device="cuda")
    y = torch.empty_like(x)
    side = torch.cuda.Stream()
    old_layer = rs.relserve_layer_create(W.TINY_GQA)
    old = [rs.relserve_batch_prepare(old_layer, cases[1][0]), rs.relserve_batch_prepare(old_layer, cases[2][0], stream=side)]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        old[0].close()
        rs.relserve_layer_step(layer, keep, wd, x, y, k, v, ws)
        old[1].close()
        old_layer.close()
    for _ in range(3):
        y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)
        again = rs.relserve_batch_prepare(layer, cases[1][0])   # takes what was kept
        y2 = torch.empty_like(cases[1][1])
        rs.relserve_layer_step(layer, again, wd, cases[1][1], y2, cases[1][2], cases[1][3], ws2)
        torch.cuda.synchronize()
        assert torch.equal(y2, cases[1][4])
        again.close()
