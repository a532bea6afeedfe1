"""GPU parity at the edges: the library's maximum expert count and fan-out, degenerate routings (every token
to one expert, k = 1), and the empty batch."""
import numpy as np
import pytest
import torch

from workloads import MoEConfig
from test_gpu_parity import _run_and_check_layer

pytestmark = pytest.mark.gpu


def test_maximum_experts_and_fanout(gpu_lib):
    """E = 256 and k = 16 are the library's limits; most experts get a handful of rows."""
    _run_and_check_layer(gpu_lib, MoEConfig("max", T=70, d=256, E=256, k=16, F=128, modes=("routed",), seed=31), "routed")
    _run_and_check_layer(gpu_lib, MoEConfig("maxk", T=50, d=128, E=16, k=16, F=256, modes=("routed",), seed=32), "routed")


def test_every_token_to_the_same_experts(gpu_lib):
    """Replay logs that send all tokens to one expert (k = 1, weight 1) or to the same pair: every other expert
    is empty and the busy ones span several row tiles with a ragged last one."""
    cfg = MoEConfig("one_hot", T=700, d=256, E=8, k=1, F=256, modes=("replay",), seed=33)
    ids = np.full((cfg.T, 1), 5, dtype=np.int32)
    w = np.ones((cfg.T, 1), dtype=np.float32)
    _run_and_check_layer(gpu_lib, cfg, "replay", log=(ids, w))
    cfg = MoEConfig("pair", T=530, d=128, E=6, k=2, F=384, modes=("replay",), seed=34)
    ids = np.tile(np.array([[4, 1]], dtype=np.int32), (cfg.T, 1))
    rng = np.random.default_rng(34)
    w = rng.dirichlet(np.ones(2), cfg.T).astype(np.float32)
    _run_and_check_layer(gpu_lib, cfg, "replay", log=(ids, w))


def test_k1_routed_weight_is_exactly_one(gpu_lib):
    cfg = MoEConfig("k1", T=300, d=256, E=12, k=1, F=128, modes=("routed",), seed=35)
    _run_and_check_layer(gpu_lib, cfg, "routed")
    from workloads import make_inputs
    inp = make_inputs(cfg, with_experts=False)
    layer = gpu_lib.MoELayer(cfg.T, cfg.d, cfg.E, cfg.k, cfg.F)
    try:
        layer.route(inp["x"].cuda(), inp["W_r"].cuda(), None)
        assert torch.all(layer.topk_w == 1.0)
    finally:
        layer.close()


def test_empty_batch(gpu_lib):
    """T = 0: every call succeeds, nothing is launched, offsets come back as zeros."""
    E, d, F, k = 8, 256, 128, 2
    ctx = gpu_lib.moe_create(0, d, E, k, F)
    try:
        dev = "cuda"
        x = torch.empty((0, d), dtype=torch.bfloat16, device=dev)
        W_r = torch.randn((E, d), dtype=torch.float32, device=dev)
        idx = torch.empty((0, k), dtype=torch.int32, device=dev)
        w = torch.empty((0, k), dtype=torch.float32, device=dev)
        perm = torch.empty(0, dtype=torch.int32, device=dev)
        inv = torch.empty(0, dtype=torch.int32, device=dev)
        for call in ("route", "replay", "replay_ids"):
            offsets = torch.full((E + 1,), 7, dtype=torch.int32, device=dev)
            if call == "route":
                gpu_lib.moe_route(ctx, x, W_r, None, k, idx, w, offsets, perm, inv)
            elif call == "replay":
                gpu_lib.moe_route_replay(ctx, x, idx, w, idx, w, offsets, perm, inv)
            else:
                gpu_lib.moe_route_replay_ids(ctx, x, W_r, idx, idx, w, offsets, perm, inv)
            torch.cuda.synchronize()
            assert torch.all(offsets == 0)
        assert gpu_lib.moe_check_ids(ctx) == 0
        xq = torch.empty((0, d), dtype=torch.uint8, device=dev)
        xs = torch.empty((d // 128, 0), dtype=torch.float32, device=dev)
        gpu_lib.moe_quantize_fp8(ctx, x, 0, d, 128, None, 1, xq, xs)
        W = torch.zeros((E, F, d), dtype=torch.uint8, device=dev)
        W2 = torch.zeros((E, d, F), dtype=torch.uint8, device=dev)
        s13 = torch.ones((E, F // 128, d // 128), dtype=torch.float32, device=dev)
        s2 = torch.ones((E, d // 128, F // 128), dtype=torch.float32, device=dev)
        y_perm = torch.empty((0, d), dtype=torch.float32, device=dev)
        gpu_lib.moe_expert_ffn_fp8(ctx, xq, xs, offsets, W, W, W2, s13, s13, s2, y_perm)
        gpu_lib.moe_expert_ffn_fp8_gather(ctx, xq, xs, perm, offsets, W, W, W2, s13, s13, s2, y_perm)
        y = torch.empty((0, d), dtype=torch.bfloat16, device=dev)
        gpu_lib.moe_combine(ctx, y_perm, inv, w, y, None)
        torch.cuda.synchronize()
    finally:
        gpu_lib.moe_destroy(ctx)


@pytest.mark.parametrize("T,d,E,k", [(16500, 256, 16, 2), (20000, 128, 200, 4), (33000, 128, 40, 3)])
def test_route_token_tile_variants(gpu_lib, T, d, E, k):
    """Routing only, at batch sizes that select the 64-token tile (16384 <= T < 32768) and the 128-token tile with a
    ragged last block; ids, weights and the permutation against the oracle."""
    from workloads import make_inputs
    from test_gpu_parity import _compare_routing, _check_permutation, _host
    cfg = MoEConfig("tiles", T=T, d=d, E=E, k=k, F=128, modes=("routed",), seed=T % 97)
    inp = make_inputs(cfg, with_experts=False)
    h = _host(inp)
    layer = gpu_lib.MoELayer(cfg.T, cfg.d, cfg.E, cfg.k, cfg.F)
    try:
        layer.route(inp["x"].cuda(), inp["W_r"].cuda(), None)
        torch.cuda.synchronize()
        _compare_routing(h, layer, None)
        _check_permutation(layer.topk_idx.cpu().numpy(), cfg.E, layer)
        # ids-only replay of the router's own ids reproduces its weights bit for bit
        idx, w = layer.topk_idx.clone(), layer.topk_w.clone()
        layer.route_replay_ids(inp["x"].cuda(), inp["W_r"].cuda(), idx)
        torch.cuda.synchronize()
        assert torch.equal(layer.topk_idx, idx) and torch.equal(layer.topk_w.view(torch.int32), w.view(torch.int32))
    finally:
        layer.close()


def _random_shape(i):
    """A seeded random shape with at least 2^17 hidden activations: the 2e-3 bar is a statement about large tensors
    (one e4m3 step the other way in the hidden activations moves a row of a d = F = 128 layer by half a percent, and a
    few dozen of them are expected whatever the size), so shapes too small for the law of large numbers are drawn again."""
    rng = np.random.default_rng(2024 + i)
    while True:
        E = int(rng.choice([1, 2, 3, 5, 8, 17, 40, 64, 130, 256]))
        k = int(min(E, rng.choice([1, 2, 3, 6, 8, 16])))
        T = int(rng.choice([1, 7, 33, 64, 65, 129, 300, 700, 1500, 2500]))
        d, F = 128 * int(rng.integers(1, 7)), 128 * int(rng.integers(1, 5))
        if T * k * F >= 1 << 17:
            return MoEConfig(f"rand{i}", T=T, d=d, E=E, k=k, F=F, modes=("routed", "replay"), seed=100 + i)


@pytest.mark.parametrize("i", range(10))
def test_random_small_shapes(gpu_lib, i):
    """Seeded random shapes (1 to 2500 tokens, 1 to 256 experts, any fan-out, one to six K blocks) through the whole
    layer against the oracle, stage by stage: between them they take the split and the single-pass router, the
    single-block and the chunked permutation, narrow, ragged and full GEMM tiles."""
    cfg = _random_shape(i)
    _run_and_check_layer(gpu_lib, cfg, "routed" if i % 3 else "replay")


@pytest.mark.parametrize("mode", ["routed", "replay"])
def test_layer_under_hip_graph_capture(gpu_lib, mode):
    """The whole layer recorded into a HIP graph (decode-sized batch, where launches are a visible share of the step) and
    replayed several times with eager work and synchronisations in between: every replay must reproduce the eager result
    bit for bit, also after the inputs have changed in place.  The library enqueues kernels only (no memsets, no
    allocations, no synchronisation) in these calls, which is what makes them capturable."""
    from workloads import make_inputs
    cfg = MoEConfig("graph", T=192, d=512, E=16, k=4, F=384, modes=("routed", "replay"), seed=77)
    inp = make_inputs(cfg)
    dv = {n: (v.cuda() if isinstance(v, torch.Tensor) else v) for n, v in inp.items()}
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        layer = gpu_lib.MoELayer(cfg.T, cfg.d, cfg.E, cfg.k, cfg.F, stream=stream)
        try:
            x = dv["x"].clone()
            layer.forward_routed(x, dv["W_r"], None, dv)              # eager warm-up: one-time attribute calls happen here
            stream.synchronize()
            log_idx, log_w = layer.topk_idx.clone(), layer.topk_w.clone()

            def step():
                if mode == "routed":
                    layer.forward_routed(x, dv["W_r"], None, dv)
                else:
                    layer.forward_replay(x, log_idx, log_w, dv)

            step()
            stream.synchronize()
            want = layer.y.clone()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                step()
            for rep in range(3):
                layer.y.zero_()
                layer.y_perm.zero_()
                graph.replay()
                stream.synchronize()
                assert torch.equal(layer.y.view(torch.int16), want.view(torch.int16)), f"replay {rep}"
                _ = (dv["W_r"] * 2).sum().item()                     # the program's own eager work between replays
            # other activations in the same buffers: the graph reads them, and the eager path agrees
            x.copy_(torch.roll(dv["x"], 5, dims=0))
            graph.replay()
            stream.synchronize()
            got = layer.y.clone()
            step()
            stream.synchronize()
            assert torch.equal(got.view(torch.int16), layer.y.view(torch.int16))
            if mode == "routed":
                assert not torch.equal(got.view(torch.int16), want.view(torch.int16))
        finally:
            layer.close()


# Row counts around every size that the big tiles of the grouped GEMMs distinguish: the narrow tile's limit, each number of 32-row
# groups, one row over a full tile, splits of two and three tiles.  The launch's tile height depends on all counts and on the shape;
# tests/test_tile_rules_host.py asks the rule which heights and tiles these layers get: in both projections every height, every number
# of groups an expert's only tile or one of several can have, with one and with more K blocks, also in half-empty feature tiles.
HEIGHT_COUNTS = [0, 1, 31, 32, 33, 64, 65, 95, 97, 128, 129, 160, 161, 192, 193, 223, 225, 255, 256, 257, 289, 320, 511, 513, 600]
HEIGHT_SHAPES = [(128, 128), (384, 256), (256, 640)]
_MIXED = [150, 185, 215, 250, 80, 40, 300, 420, 520, 700]
HEIGHT_LAYERS = [([189, 189, 191, 20], 128, 128), ([226, 217, 194], 384, 128), ([247, 249, 247], 128, 384),
                 (_MIXED * 5, 128, 128), (_MIXED * 7, 384, 256)]


def _heights_log(counts, d, F):
    cfg = MoEConfig("heights", T=sum(counts), d=d, E=len(counts), k=1, F=F, modes=("replay",), seed=d + F)
    rng = np.random.default_rng(cfg.seed)
    ids = rng.permutation(np.repeat(np.arange(cfg.E, dtype=np.int32), counts)).reshape(cfg.T, 1)
    return cfg, (np.ascontiguousarray(ids), np.ones((cfg.T, 1), dtype=np.float32))


def _run_heights(gpu_lib, counts, d, F):
    cfg, log = _heights_log(counts, d, F)
    _run_and_check_layer(gpu_lib, cfg, "replay", log=log)


@pytest.mark.parametrize("d,F", HEIGHT_SHAPES)
def test_tile_heights(gpu_lib, d, F):
    """Replay logs (k = 1) that give the experts all of HEIGHT_COUNTS; one, two, three and five K blocks; output feature tiles that are
    half empty."""
    _run_heights(gpu_lib, HEIGHT_COUNTS, d, F)


@pytest.mark.parametrize("counts,d,F", HEIGHT_LAYERS, ids=lambda v: f"{len(v)}experts" if isinstance(v, list) else str(v))
def test_chosen_tile_heights(gpu_lib, counts, d, F):
    """Loads that make the launch take the other heights."""
    _run_heights(gpu_lib, counts, d, F)


@pytest.mark.parametrize("d,F", [(128, 128), (384, 256), (640, 384)])
def test_narrow_tiles_of_two_and_three_groups(gpu_lib, d, F):
    """Experts on both sides of every row count at which a narrow tile changes: two or three groups of 32 rows, the copies of 8 rows
    that are left out, and the first count that is no narrow tile any more; output feature tiles that are half empty."""
    _run_heights(gpu_lib, [63, 64, 65, 72, 73, 80, 81, 88, 89, 95, 96, 97, 104, 90, 70], d, F)


# Lists that are dealt to the XCDs in parts of equal numbers and of equal cost, with and without units left to whoever is free, and with
# so uneven parts that every block has to look (which of them: tests/test_tile_rules_host.py).
DEALT_LAYERS = [([8 + i % 33 for i in range(64)], 128, 4096), ([270, 22, 18, 16, 16, 8, 7, 2], 128, 4096),
                ([150, 137, 59, 50, 45, 45] + [41] * 3 + [39, 37, 37, 26, 25, 24, 23, 20] + [19] * 3 + [17, 16, 16, 13, 10, 10, 10, 9, 8, 7]
                 + [6] * 4 + [5] * 3 + [3, 2], 128, 1024),
                ([18, 17, 552, 133, 70, 15, 36, 7, 26, 39, 2, 28, 11, 77, 17, 45, 3, 8, 12, 23, 14, 30, 88, 31], 6144, 128)]


@pytest.mark.parametrize("counts,d,F", DEALT_LAYERS, ids=lambda v: f"{len(v)}experts" if isinstance(v, list) else str(v))
def test_dealt_lists(gpu_lib, counts, d, F):
    """Against the oracle, and further passes over the same context, which find the counts of the last one's shared units."""
    from workloads import make_inputs
    _run_heights(gpu_lib, counts, d, F)
    cfg, (ids, w) = _heights_log(counts, d, F)
    inp = {n: (v.cuda() if isinstance(v, torch.Tensor) else v) for n, v in make_inputs(cfg).items()}
    layer = gpu_lib.MoELayer(cfg.T, cfg.d, cfg.E, cfg.k, cfg.F)
    try:
        want = None
        for _ in range(3):
            layer.y_perm.fill_(float("nan"))
            layer.forward_replay(inp["x"], torch.from_numpy(ids).cuda(), torch.from_numpy(w).cuda(), inp)
            torch.cuda.synchronize()
            want = layer.y_perm.clone() if want is None else want
            assert not torch.isnan(layer.y_perm).any() and torch.equal(layer.y_perm, want)
    finally:
        layer.close()


# Layers of so few units that both projections stream whatever their rows per expert, or the down projection alone (which of them:
# tests/test_tile_rules_host.py): no rows to five tiles of them, feature tiles that are half empty.
ROUND_COUNTS = [0, 1, 63, 64, 65, 129, 200, 300]
ROUND_SHAPES = [(512, 640), (640, 512), (512, 2048)]


@pytest.mark.parametrize("d,F", ROUND_SHAPES)
def test_layers_of_one_round(gpu_lib, d, F):
    _run_heights(gpu_lib, ROUND_COUNTS, d, F)


@pytest.mark.parametrize("rows", [1, 15, 16, 17, 31, 32, 33, 48, 65])
def test_activation_codes_at_block_edges(gpu_lib, rows):
    """Row counts around the quantisation kernel's 32-row blocks, plain and fanned out, with the values its short quotient has
    to get right: groups at both ends of the scale range, where the division itself is taken, negative zeros, and quotients
    that land on rounding boundaries (every bf16 significand under one scale).  Codes and scales are exact."""
    from oracle import fp_formats as ff, moe_layer as om
    d, fan = 384, 2
    g = torch.Generator().manual_seed(rows)
    x = torch.randn((rows, d), generator=g)
    bits = torch.arange(128, dtype=torch.int32) + (126 << 7)                # 0.5 .. 1: every significand
    x[0, :128] = (bits << 16).view(torch.float32)
    x[0, 128:256] *= 1e-36
    x[0, 256:] *= 1e36
    x[rows - 1, ::3] = -0.0
    xb = x.to(torch.bfloat16)
    xb_bits = xb.view(torch.int16).numpy().view(np.uint16)
    q_o, s_o = om.quantize_rows(ff.bf16_bits_to_f64(xb_bits))
    neg_zero = (xb_bits & 0x8000) != 0                                      # zeros keep their sign (the oracle's coder may not)
    dst = torch.randperm(rows * fan, generator=g).to(torch.int32)
    ctx = gpu_lib.moe_create(0, 128, 1, 1, 128)
    try:
        for dst_rows, f in ((None, 1), (dst.cuda(), fan)):
            q = torch.full((rows * f, d), 0x55, dtype=torch.uint8, device="cuda")
            s = torch.full((d // 128, rows * f), -1.0, device="cuda")
            gpu_lib.moe_quantize_fp8(ctx, xb.cuda(), rows, d, 128, dst_rows, f, q, s)
            torch.cuda.synchronize()
            src = np.arange(rows)
            if dst_rows is not None:
                src = np.empty(rows * fan, dtype=np.int64)
                src[dst.numpy()] = np.arange(rows * fan) // fan
            got = q.cpu().numpy()
            assert np.array_equal(s.cpu().numpy().T, s_o[src])
            assert np.array_equal(got & 0x7F, (q_o & 0x7F)[src])
            assert np.array_equal((got & 0x80) != 0, neg_zero[src])
    finally:
        gpu_lib.moe_destroy(ctx)


@pytest.mark.parametrize("k", [1, 2, 3, 5, 7, 8, 9, 16])
@pytest.mark.parametrize("d", [128, 1024, 1152])
def test_combine_at_every_fan_out(gpu_lib, k, d):
    """One, exactly one and two blocks of columns per token; compiled and run-time fan-outs; slots without a row.  The fp32
    sums are the slot-order multiply-add chain: k roundings of at most half an ulp of a partial sum each."""
    T = 5
    g = torch.Generator().manual_seed(k * 31 + d)
    y_perm, w = torch.randn((T * k, d), generator=g), torch.rand((T, k), generator=g)
    inv = torch.randperm(T * k, generator=g).to(torch.int32).view(T, k)
    inv[2, k // 2] = -1
    layer = gpu_lib.MoELayer(T, d, 16, k, 128)
    try:
        layer.y_perm.copy_(y_perm)
        layer.inv_perm.copy_(inv.view(-1))
        layer.topk_w.copy_(w)
        sums = torch.empty((T, d), device="cuda")
        layer.combine(sums)
        torch.cuda.synchronize()
        rows = torch.where(inv[..., None] >= 0, y_perm[inv.clamp(min=0).long()], torch.zeros(()))
        terms = w[..., None].double() * rows.double()
        err = (sums.cpu().double() - terms.sum(1)).abs()
        assert torch.all(err <= k * 2.0 ** -24 * terms.abs().sum(1) + 1e-30)
        assert torch.equal(layer.y.cpu(), sums.cpu().to(torch.bfloat16))
    finally:
        layer.close()


@pytest.mark.parametrize("d,F", [(384, 384), (8320, 256), (128, 1152), (640, 384)])
def test_weight_streaming_tiles(gpu_lib, d, F):
    """Few rows per expert (a replay log with k = 1): experts of one to three streaming tiles, row counts around one and two
    groups of 32 columns and around a tile; one to 65 K blocks (fewer than the ring's stages; one more than a wave keeps
    weight scales for); odd output feature tiles; a hidden size above d."""
    E = 70 if d <= 640 else 20
    counts = [1, 2, 31, 32, 33, 63, 64, 65, 96, 129] + [0] * (E - 10)
    cfg = MoEConfig("stream", T=sum(counts), d=d, E=E, k=1, F=F, modes=("replay",), seed=d + F)
    rng = np.random.default_rng(cfg.seed)
    ids = rng.permutation(np.repeat(rng.permutation(cfg.E).astype(np.int32), counts)).reshape(cfg.T, 1)
    _run_and_check_layer(gpu_lib, cfg, "replay", log=(np.ascontiguousarray(ids), np.ones((cfg.T, 1), dtype=np.float32)))


# in small blocks, and streaming
SMALL_LINEARS = [(1, 128, 128), (33, 256, 384), (64, 8320, 640), (65, 384, 256), (300, 1280, 1152),
                 (33, 256, 65 * 128), (64, 8320, 65 * 128), (300, 1280, 13 * 128)]


@pytest.mark.parametrize("rows,K,NOUT", SMALL_LINEARS)
def test_small_linears_equal_the_big_tile_kernel(gpu_lib, rows, K, NOUT):
    """Dense products small enough for the small-block or the streaming kernel against the same rows inside a product that takes the
    big tiles: the same products in the same order, so the same bits."""
    big = 256 * 200                                                     # rows of the large product: over 256 streaming units
    g = torch.Generator(device="cuda").manual_seed(rows + K)
    codes = lambda *s: (torch.randn(s, generator=g, device="cuda") * 60).to(torch.float8_e4m3fn).view(torch.uint8)
    xq, wq = codes(big, K), codes(NOUT, K)
    xs = torch.rand((K // 128, big), generator=g, device="cuda") + 0.5
    ws = torch.rand((NOUT // 128, K // 128), generator=g, device="cuda") + 0.5
    ctx = gpu_lib.moe_create(big, K, 1, 1, max(NOUT, 128 * 8))
    try:
        y_big = torch.empty((big, NOUT), device="cuda")
        gpu_lib.moe_linear_fp8(ctx, xq, xs, big, K, wq, ws, NOUT, y_big)
        y = torch.full((rows, NOUT), float("nan"), device="cuda")
        gpu_lib.moe_linear_fp8(ctx, xq[:rows].contiguous(), xs[:, :rows].contiguous(), rows, K, wq, ws, NOUT, y)
        torch.cuda.synchronize()
        assert torch.equal(y, y_big[:rows])
        exact = xq[:4].view(torch.float8_e4m3fn).double().view(-1, K // 128, 128) * xs.T[:4, :, None].double()
        w = wq.view(torch.float8_e4m3fn).double().view(NOUT // 128, 128, K // 128, 128) * ws[:, None, :, None].double()
        exact = exact.reshape(-1, K) @ w.reshape(NOUT, K).T
        assert float((y[:4].double() - exact[:rows]).norm() / exact[:rows].norm()) < 1e-4
    finally:
        gpu_lib.moe_destroy(ctx)


@pytest.mark.parametrize("T,d,E,k", [(1, 128, 1, 1), (7, 1024, 5, 3), (8, 1152, 100, 8), (9, 2176, 256, 16), (32, 640, 128, 4),
                                     (33, 640, 129, 4), (2, 16384, 60, 6), (3, 16512, 60, 6)])
def test_router_of_small_batches(gpu_lib, T, d, E, k):
    """Routing at the edges of the small-batch router: one token, token groups of eight and the last size it takes; one column
    slice, a ragged last slice, as many slices as it takes and one more (the matrix-core form); with a selection bias;
    ids-only replay of the router's own ids gives its weights bit for bit."""
    from workloads import make_inputs
    from test_gpu_parity import _compare_routing, _check_permutation, _host
    cfg = MoEConfig("rows", T=T, d=d, E=E, k=k, F=128, modes=("routed",), seed=T + E)
    inp = make_inputs(cfg, with_experts=False)
    h = _host(inp)
    layer = gpu_lib.MoELayer(cfg.T, cfg.d, cfg.E, cfg.k, cfg.F)
    try:
        for bias in (None, np.linspace(-1.0, 1.0, E).astype(np.float32)):
            layer.route(inp["x"].cuda(), inp["W_r"].cuda(), None if bias is None else torch.from_numpy(bias).cuda())
            torch.cuda.synchronize()
            _compare_routing(h, layer, bias)
            _check_permutation(layer.topk_idx.cpu().numpy(), cfg.E, layer)
            idx, w = layer.topk_idx.clone(), layer.topk_w.clone()
            layer.route_replay_ids(inp["x"].cuda(), inp["W_r"].cuda(), idx)
            torch.cuda.synchronize()
            assert torch.equal(layer.topk_idx, idx) and torch.equal(layer.topk_w.view(torch.int32), w.view(torch.int32))
    finally:
        layer.close()


@pytest.mark.parametrize("T,k", [(1, 1), (63, 16), (1024, 1), (1025, 1), (683, 3), (4096, 1), (4097, 1), (1024, 8), (8193, 1)])
def test_permutation_at_block_edges(gpu_lib, T, k):
    """Assignment counts around every size the one-block permutation is compiled for, and one beyond it; a few ids are
    outside [0, E), which leaves their slots without a row."""
    E = 37
    rng = np.random.default_rng(T * k)
    ids = np.argsort(rng.random((T, E)), axis=1)[:, :k].astype(np.int32)
    w = rng.random((T, k), dtype=np.float32)
    layer = gpu_lib.MoELayer(T, 128, E, k, 128)
    try:
        for bad in (False, True):
            if bad:
                ids[rng.integers(0, T, 3), rng.integers(0, k, 3)] = [E, -1, 1 << 20]
            layer.route_replay(torch.empty((T, 128), dtype=torch.bfloat16, device="cuda"), torch.from_numpy(ids).cuda(),
                               torch.from_numpy(w).cuda())
            torch.cuda.synchronize()
            flat = ids.reshape(-1)
            ok = (flat >= 0) & (flat < E)
            order = np.flatnonzero(ok)[np.argsort(flat[ok], kind="stable")]
            inv = np.full(T * k, -1, dtype=np.int32)
            inv[order] = np.arange(order.size)
            assert np.array_equal(layer.perm.cpu().numpy()[:order.size], order)
            assert np.array_equal(layer.inv_perm.cpu().numpy(), inv)
            assert np.array_equal(layer.offsets.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(flat[ok], minlength=E))]))
            assert np.array_equal(layer.topk_idx.cpu().numpy(), ids) and np.array_equal(layer.topk_w.cpu().numpy(), w)
            assert (gpu_lib.moe_check_ids(layer.ctx) != 0) == bool((~ok).any())
    finally:
        layer.close()


@pytest.mark.parametrize("T,k", [(1366, 3), (4097, 1), (1024, 8), (8193, 1), (512, 8), (513, 8), (256, 16), (257, 16),
                                 (640, 8), (641, 8), (320, 16), (321, 16)])
def test_permutation_either_side_of_the_one_block_form(gpu_lib, T, k):
    """Assignment counts around the sizes up to which one block permutes a batch: the router's own ids (no search for repeats:
    up to 8192) and logged ids (up to 5120, with one slot a token up to 8192), the latter also with an id repeated in the
    last token."""
    from workloads import make_inputs
    from test_gpu_parity import _check_permutation
    E = 37
    cfg = MoEConfig("perm", T=T, d=128, E=E, k=k, F=128, modes=("routed",), seed=T + k)
    inp = make_inputs(cfg, with_experts=False)
    layer = gpu_lib.MoELayer(T, 128, E, k, 128)
    try:
        layer.route(inp["x"].cuda(), inp["W_r"].cuda(), None)
        torch.cuda.synchronize()
        _check_permutation(layer.topk_idx.cpu().numpy(), E, layer)
        assert gpu_lib.moe_check_ids(layer.ctx) == 0
        ids, w = layer.topk_idx.clone(), layer.topk_w.clone()
        for repeated in (False, True):
            if repeated:
                if k == 1:
                    break
                ids[T - 1, k - 1] = ids[T - 1, 0]
            layer.route_replay(inp["x"].cuda(), ids, w)
            torch.cuda.synchronize()
            _check_permutation(ids.cpu().numpy(), E, layer)
            assert torch.equal(layer.topk_idx, ids) and torch.equal(layer.topk_w, w)
            assert (gpu_lib.moe_check_ids(layer.ctx) != 0) == repeated
    finally:
        layer.close()


@pytest.mark.parametrize("rows,cols,fan", [(1, 128, 16), (15, 256, 5), (33, 384, 17), (100, 1152, 8), (47, 128, 33), (8192 * 32 + 5, 128, 1),
                                           (4097, 8192, 2)])
def test_fanned_out_quantisation(gpu_lib, rows, cols, fan):
    """Fan-outs below, at and above the sixteen indices a row's lanes hold, in groups of four and not; row counts around the
    blocks of 16; the sizes from which blocks of 32 rows are taken; slots without an output row.  Every output row has the
    bits of the plain form's row, and skipped rows stay untouched."""
    g = torch.Generator(device="cuda").manual_seed(rows + fan)
    x = torch.randn((rows, cols), generator=g, device="cuda").to(torch.bfloat16)
    dst = torch.randperm(rows * fan, generator=g, device="cuda").to(torch.int32)
    skipped = torch.zeros(rows * fan, dtype=torch.bool, device="cuda")
    skipped[torch.randperm(rows * fan, generator=g, device="cuda")[:rows * fan // 7]] = True       # by slot
    ctx = gpu_lib.moe_create(0, 128, 1, 1, 128)
    try:
        q1, s1 = torch.empty((rows, cols), dtype=torch.uint8, device="cuda"), torch.empty((cols // 128, rows), device="cuda")
        gpu_lib.moe_quantize_fp8(ctx, x, rows, cols, 128, None, 1, q1, s1)
        q = torch.full((rows * fan, cols), 0x55, dtype=torch.uint8, device="cuda")
        s = torch.full((cols // 128, rows * fan), -1.0, device="cuda")
        gpu_lib.moe_quantize_fp8(ctx, x, rows, cols, 128, torch.where(skipped, -1, dst), fan, q, s)
        torch.cuda.synchronize()
        src = torch.empty(rows * fan, dtype=torch.int64, device="cuda")
        src[dst.long()] = torch.arange(rows * fan, device="cuda") // fan
        written = torch.ones(rows * fan, dtype=torch.bool, device="cuda")
        written[dst.long()[skipped]] = False
        assert torch.equal(q, torch.where(written[:, None], q1[src], torch.full_like(q, 0x55)))
        assert torch.equal(s, torch.where(written, s1[:, src], torch.full_like(s, -1.0)))
    finally:
        gpu_lib.moe_destroy(ctx)


@pytest.mark.parametrize("T,d,k", [(3, 1280, 3), (2, 2176, 8), (5, 4992, 1), (4, 3200, 11), (3, 1152, 2), (2, 1920, 4), (3, 1408, 5),
                                   (2, 1536, 6), (1, 1664, 7)])
def test_combine_of_widths_that_split_unevenly(gpu_lib, T, d, k):
    """Two to five blocks of columns per token whose common width is not a multiple of the columns left: the slot-order
    multiply-add chain as in the test of the fan-outs, k roundings of at most half an ulp of a partial sum."""
    g = torch.Generator().manual_seed(d + k)
    y_perm, w = torch.randn((T * k, d), generator=g), torch.rand((T, k), generator=g)
    inv = torch.randperm(T * k, generator=g).to(torch.int32).view(T, k)
    layer = gpu_lib.MoELayer(T, d, 16, k, 128)
    try:
        layer.y_perm.copy_(y_perm)
        layer.inv_perm.copy_(inv.view(-1))
        layer.topk_w.copy_(w)
        layer.y.fill_(float("nan"))
        sums = torch.full((T, d), float("nan"), device="cuda")
        layer.combine(sums)
        torch.cuda.synchronize()
        terms = w[..., None].double() * y_perm[inv.long()].double()
        err = (sums.cpu().double() - terms.sum(1)).abs()
        assert torch.all(err <= k * 2.0 ** -24 * terms.abs().sum(1) + 1e-30)
        assert torch.equal(layer.y.cpu(), sums.cpu().to(torch.bfloat16))
    finally:
        layer.close()


def _concentrated_log(T, E, k, cold):
    """Every token goes to experts 0..k-1, but for `cold` slots of the last tokens that name one other expert each; None: an
    even load."""
    ids = np.tile(np.arange(k, dtype=np.int32), (T, 1))
    if cold is None:
        ids = (np.arange(T * k).reshape(T, k) % E).astype(np.int32)
    else:
        ids.reshape(-1)[T * k - cold:] = np.arange(k, k + cold, dtype=np.int32)
    return ids, np.full((T, k), 1.0 / k, dtype=np.float32)


@pytest.mark.parametrize("cold", [0, 23, 24, None])
def test_concentrated_loads_either_side_of_the_choice(gpu_lib, cold):
    """A batch with few rows per expert on average, large enough that the down projection's kernel is chosen from the loads on
    the device: big tiles where there are more than twice as many 64-row tiles as 256-row ones (72 + cold against 24 + cold
    here), otherwise the streaming kernel."""
    cfg = MoEConfig("conc", T=520, d=2048, E=90, k=8, F=128, modes=("replay",), seed=900 + (cold or 0))
    ids, w = _concentrated_log(cfg.T, cfg.E, cfg.k, cold)
    n = np.bincount(ids.reshape(-1), minlength=cfg.E)
    assert (((n + 63) // 64).sum() > 2 * ((n + 255) // 256).sum()) == (cold in (0, 23))
    _run_and_check_layer(gpu_lib, cfg, "replay", log=(ids, w))


def test_one_context_takes_concentrated_and_even_loads_in_turn(gpu_lib):
    """The same context with loads on both sides of that choice, other activations each time: every call equals a fresh
    context's (lists, counts and workspaces of the call before must not show)."""
    from workloads import make_inputs
    cfg = MoEConfig("turns", T=520, d=2048, E=90, k=8, F=256, modes=("replay",), seed=55)
    dv = {n: (v.cuda() if isinstance(v, torch.Tensor) else v) for n, v in make_inputs(cfg).items()}
    kept = gpu_lib.MoELayer(cfg.T, cfg.d, cfg.E, cfg.k, cfg.F)
    try:
        for step, cold in enumerate((0, None, 23, 24, 0)):
            x = torch.roll(dv["x"], step, dims=0)
            ids, w = (torch.from_numpy(a).cuda() for a in _concentrated_log(cfg.T, cfg.E, cfg.k, cold))
            got = kept.forward_replay(x, ids, w, dv).clone()
            fresh = gpu_lib.MoELayer(cfg.T, cfg.d, cfg.E, cfg.k, cfg.F)
            try:
                want = fresh.forward_replay(x, ids, w, dv, fused=False)
                torch.cuda.synchronize()
                assert torch.isfinite(want.float()).all() and float(want.float().abs().max()) > 0
                assert torch.equal(got.view(torch.int16), want.view(torch.int16)), step
            finally:
                fresh.close()
    finally:
        kept.close()
