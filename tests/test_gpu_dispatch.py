"""GPU: the instances and the rules between them that the layers of the other files do not reach: the dense product on the big
tiles at ragged sizes, the gathering form of the streaming kernel, sizes either side of every rule that chooses between
streaming and big tiles, graph replay of such layers, values that are not finite in the quantisers."""
import numpy as np
import pytest
import torch

from workloads import MoEConfig, make_inputs
from test_gpu_parity import _check_permutation, _compare_routing, _host, _run_and_check_layer

pytestmark = pytest.mark.gpu


# --------------------------------------------------------------------------- dense products on the big tiles
def _codes(g, *shape):
    return (torch.randn(shape, generator=g, device="cuda") * 60).to(torch.float8_e4m3fn).view(torch.uint8)


# all above 256 streaming units, so that none streams (which tiles they get: tests/test_tile_rules_host.py): one ragged row tile, two and
# four, many with a last one of five rows, and 2 to 8 groups of 32 rows in a tile, odd and even
BIG_LINEARS = [(70, 384, 259 * 128), (129, 128, 257 * 128), (193, 256, 258 * 128), (257, 256, 131 * 128), (300, 1280, 131 * 128),
               (777, 128, 67 * 128), (130 * 256 + 5, 256, 128), (9000, 640, 9 * 128),
               (130, 640, 172 * 128), (150, 1024, 181 * 128), (160, 384, 176 * 128), (3000, 256, 42 * 128)]


@pytest.mark.parametrize("rows,K,NOUT", BIG_LINEARS)
def test_big_tile_linear_at_ragged_sizes(gpu_lib, rows, K, NOUT):
    """Every row of the product: against the same rows in calls of 64, which stream (the same instructions in the same order, so
    the same bits), and against a 64-bit evaluation (bar 1e-4: the matrix pipe's own rounding is 1.3e-5)."""
    assert (rows + 63) // 64 * ((NOUT + 255) // 256) > 256
    g = torch.Generator(device="cuda").manual_seed(rows + K)
    xq, wq = _codes(g, rows, K), _codes(g, NOUT, K)
    xs = torch.rand((K // 128, rows), generator=g, device="cuda") + 0.5
    ws = torch.rand((NOUT // 128, K // 128), generator=g, device="cuda") + 0.5
    ctx = gpu_lib.moe_create(rows, K, 1, 1, NOUT)
    try:
        y = torch.full((rows, NOUT), float("nan"), device="cuda")
        gpu_lib.moe_linear_fp8(ctx, xq, xs, rows, K, wq, ws, NOUT, y)
        part = torch.empty((64, NOUT), device="cuda")
        wd = wq.view(torch.float8_e4m3fn).double().view(NOUT // 128, 128, K // 128, 128) * ws[:, None, :, None].double()
        wd = wd.view(NOUT, K).T.contiguous()
        err = ref = 0.0
        for r in range(0, rows, 64):
            n = min(64, rows - r)
            part.fill_(float("nan"))
            xs_r = xs[:, r:r + n].contiguous()
            gpu_lib.moe_linear_fp8(ctx, xq[r:r + n], xs_r, n, K, wq, ws, NOUT, part)
            assert torch.equal(y[r:r + n], part[:n]), r
            xd = xq[r:r + n].view(torch.float8_e4m3fn).double().view(n, K // 128, 128) * xs_r.T[:, :, None].double()
            exact = xd.view(n, K) @ wd
            err += float((part[:n].double() - exact).square().sum())
            ref += float(exact.square().sum())
        assert (err / ref) ** 0.5 < 1e-4
    finally:
        gpu_lib.moe_destroy(ctx)


@pytest.mark.parametrize("K", [128, 1024])
def test_big_tile_linear_of_small_integers_is_exact(gpu_lib, K):
    """Unit scales and codes that decode to multiples of 0.5 up to 4: every partial sum is a multiple of 0.25 below 2^22, so fp32
    accumulation loses nothing and the product must be exact."""
    rows, NOUT = 333, 131 * 128
    g = torch.Generator(device="cuda").manual_seed(K)
    small = lambda *s: (torch.randint(-8, 9, s, generator=g, device="cuda") * 0.5).to(torch.float8_e4m3fn).view(torch.uint8)
    xq, wq = small(rows, K), small(NOUT, K)
    ctx = gpu_lib.moe_create(rows, K, 1, 1, NOUT)
    try:
        y = torch.full((rows, NOUT), float("nan"), device="cuda")
        gpu_lib.moe_linear_fp8(ctx, xq, torch.ones((K // 128, rows), device="cuda"), rows, K, wq,
                               torch.ones((NOUT // 128, K // 128), device="cuda"), NOUT, y)
        exact = xq.view(torch.float8_e4m3fn).double() @ wq.view(torch.float8_e4m3fn).double().T.contiguous()
        assert torch.equal(y.double(), exact)
    finally:
        gpu_lib.moe_destroy(ctx)


# --------------------------------------------------------------------------- the gathering form of the streaming kernel
def _skewed_log(T, E, hot0, hot1, step):
    """k = 2 distinct ids a token: expert 0 gets the first `hot0` tokens, expert 1 the last `hot1`, the other slots go round."""
    t = np.arange(T)
    ids = np.stack([2 + (t + step) % (E - 2), 2 + (t + step + 1) % (E - 2)], axis=1).astype(np.int32)
    ids[:hot0, 0] = 0
    ids[T - hot1:, 1] = 1
    return np.roll(ids, step, axis=0).copy(), np.random.default_rng(T + step).dirichlet(np.ones(2), T).astype(np.float32)


@pytest.mark.parametrize("T,d,E,F,hot0,hot1", [(150, 256, 16, 384, 130, 40), (100, 384, 16, 128, 65, 64), (150, 640, 16, 640, 129, 33),
                                               (90, 8320, 12, 256, 70, 33), (1, 384, 16, 384, 0, 0), (33, 1152, 24, 256, 33, 32)])
def test_gathering_streaming_form(gpu_lib, T, d, E, F, hot0, hot1):
    """Two experts a token, so that gathered rows, token planes and sorted rows differ: two to 65 K blocks, experts of one to three
    streaming tiles, odd feature tiles.  Three calls on one context with other activations and routing each time, the
    gathered form against a fresh context's expert-ordered one bit for bit; that one against the oracle."""
    cfg = MoEConfig("gather", T=T, d=d, E=E, k=2, F=F, modes=("replay",), seed=T + d)
    assert T * 2 <= 32 * E and E * (F // 128) < 256                      # streams
    dv = {n: (v.cuda() if isinstance(v, torch.Tensor) else v) for n, v in make_inputs(cfg).items()}
    _run_and_check_layer(gpu_lib, cfg, "replay", log=_skewed_log(T, E, hot0, hot1, 0))
    kept = gpu_lib.MoELayer(T, d, E, 2, F)
    try:
        for step in (0, 1, 2):
            x = (torch.roll(dv["x"].float(), step, dims=1) * (1.0 + step)).to(torch.bfloat16)
            ids, w = (torch.from_numpy(a).cuda() for a in _skewed_log(T, E, hot0, hot1, step))
            kept.y_perm.fill_(float("nan"))
            got = kept.forward_replay(x, ids, w, dv, fused=True).clone()
            hq, hs = kept.hidden()
            fresh = gpu_lib.MoELayer(T, d, E, 2, F)
            try:
                want = fresh.forward_replay(x, ids, w, dv, fused=False)
                hq_w, hs_w = fresh.hidden()
                torch.cuda.synchronize()
                assert torch.equal(hq, hq_w) and torch.equal(hs.view(torch.int32), hs_w.view(torch.int32)), step
                assert torch.equal(kept.y_perm.view(torch.int32), fresh.y_perm.view(torch.int32)), step
                assert torch.equal(got.view(torch.int16), want.view(torch.int16)), step
            finally:
                fresh.close()
    finally:
        kept.close()


# --------------------------------------------------------------------------- either side of every rule
@pytest.mark.parametrize("T,d,E,k,F", [
    (800, 128, 100, 1, 384), (801, 128, 100, 1, 384),       # gate/up: 8 rows per expert, no idle units
    (1280, 128, 40, 1, 768), (1281, 128, 40, 1, 768),       #   32 rows, units expected just below 256
    (1280, 128, 40, 1, 896),                                #   and above
    (480, 256, 10, 1, 256), (481, 256, 10, 1, 256),         # down: 48 rows per expert
    (128, 128, 130, 8, 1408), (129, 128, 130, 8, 1408),     # gate/up units of the most concentrated log: 176 and 264
    (512, 2048, 90, 8, 128), (513, 2048, 90, 8, 128),       # down units of it: 512 and 576
    (64, 8448, 22, 16, 256), (65, 8448, 22, 16, 256),       #   528 in one row tile, where no weight passes twice; 1056
], ids=str)
def test_layers_either_side_of_the_streaming_rules(gpu_lib, T, d, E, k, F):
    """The last size of one kernel and the first of the other, stage by stage against the oracle.  Equal gate weights: the k rows
    of a token and their errors are independent, so the layer's relative error is then that of its rows (y_perm, held to the
    same bar).  With drawn weights few rows carry a token, and with F = 128, one scale block a row, a single hidden code
    that is steps off moved one of 513 tokens by 3e-2 of its norm, which is 1.3e-3 of the whole tensor's (3e-2 / sqrt(513))."""
    cfg = MoEConfig("rule", T=T, d=d, E=E, k=k, F=F, modes=("replay",), seed=T + F)
    rng = np.random.default_rng(T + d)
    ids = np.argsort(rng.random((T, E)), axis=1)[:, :k].astype(np.int32)
    _run_and_check_layer(gpu_lib, cfg, "replay", log=(np.ascontiguousarray(ids), np.full((T, k), 1.0 / k, dtype=np.float32)))


@pytest.mark.parametrize("T,E,k", [(16, 8, 2), (17, 8, 2), (32, 128, 8), (17, 129, 8), (32, 256, 8)])
def test_router_of_one_chunk_either_side_of_its_rule(gpu_lib, T, E, k):
    """d = 128: the vector-ALU router up to 16 tokens (up to 32 above 128 experts), the matrix-core one beyond; ids-only replay
    of the router's own ids gives its weights bit for bit."""
    cfg = MoEConfig("chunk", T=T, d=128, E=E, k=k, F=128, modes=("routed",), seed=T + E)
    inp = make_inputs(cfg, with_experts=False)
    layer = gpu_lib.MoELayer(T, 128, E, k, 128)
    try:
        layer.route(inp["x"].cuda(), inp["W_r"].cuda(), None)
        torch.cuda.synchronize()
        _compare_routing(_host(inp), layer)
        _check_permutation(layer.topk_idx.cpu().numpy(), E, layer)
        idx, w = layer.topk_idx.clone(), layer.topk_w.clone()
        layer.route_replay_ids(inp["x"].cuda(), inp["W_r"].cuda(), idx)
        torch.cuda.synchronize()
        assert torch.equal(layer.topk_idx, idx) and torch.equal(layer.topk_w.view(torch.int32), w.view(torch.int32))
    finally:
        layer.close()


# --------------------------------------------------------------------------- graph replay
GRAPH_LAYERS = {"streaming": (24, 640, 16, 2, 384), "chosen-on-device": (520, 2048, 90, 8, 128), "persistent-blocks": (400, 512, 60, 2, 512),
                "persistent-blocks-down": (1000, 512, 36, 2, 640)}


@pytest.mark.parametrize("T,d,E,k,F", GRAPH_LAYERS.values(), ids=GRAPH_LAYERS)
def test_graph_replay_with_other_logs_and_activations(gpu_lib, T, d, E, k, F):
    """A replayed layer recorded into a graph; between replays its inputs change in place, from an even log to one that sends
    every token to the same experts and back, with eager work in between.  Every replay equals the eager result."""
    cfg = MoEConfig("graph", T=T, d=d, E=E, k=k, F=F, modes=("replay",), seed=T)
    dv = {n: (v.cuda() if isinstance(v, torch.Tensor) else v) for n, v in make_inputs(cfg).items()}
    even = (torch.arange(T * k, device="cuda").view(T, k) % E).to(torch.int32).contiguous()
    same = torch.arange(k, device="cuda", dtype=torch.int32).repeat(T, 1)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        layer, eager = (gpu_lib.MoELayer(T, d, E, k, F, stream=stream) for _ in range(2))
        try:
            x, ids, w = dv["x"].clone(), even.clone(), torch.full((T, k), 1.0 / k, device="cuda")
            layer.forward_replay(x, ids, w, dv)
            stream.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                layer.forward_replay(x, ids, w, dv)
            seen = []
            for rep, log in enumerate((even, same, even, same, same)):
                ids.copy_(log)
                x.copy_(torch.roll(dv["x"], rep, dims=0))
                layer.y.zero_()
                layer.y_perm.zero_()
                graph.replay()
                want = eager.forward_replay(x, ids, w, dv)
                stream.synchronize()
                assert torch.equal(layer.y.view(torch.int16), want.view(torch.int16)), rep
                seen.append(layer.y.clone())
                _ = (dv["W_r"] * 2).sum().item()
            assert not torch.equal(seen[0], seen[1]) and not torch.equal(seen[3], seen[4])
        finally:
            layer.close()
            eager.close()


# --------------------------------------------------------------------------- values that are not finite
def test_quantisers_of_values_that_are_not_finite(gpu_lib):
    """A NaN does not count towards the scale and becomes -448; an infinity makes the scale infinite, all finite values of its
    group zeros and infinities -448 (infinity over infinity); a group of NaNs has scale 1.  The other groups are untouched."""
    rows, cols = 256, 512
    g = torch.Generator().manual_seed(7)
    x = torch.randn((rows, cols), generator=g)
    x[3, 5] = x[3, 130] = x[200, 511] = float("nan")
    x[9, 128:256] = float("nan")
    x[17, 260] = float("inf")
    x[18, 261] = -float("inf")
    x[19, 262], x[19, 263] = float("inf"), float("nan")
    xb = x.to(torch.bfloat16)
    ctx = gpu_lib.moe_create(0, 128, 1, 1, 128)

    def expected(groups):                                              # [..., 128 or 128 x 128 values of a group as the last axis]
        v = groups.float()
        amax = torch.where(v.isnan(), torch.zeros(()), v.abs()).amax(-1, keepdim=True)
        s = torch.where(amax == 0, torch.ones(()), amax / 448.0)
        q = v / s
        q = torch.where(q.isnan(), torch.full((), -448.0), q.clamp(-448.0, 448.0))
        return q.to(torch.float8_e4m3fn).view(torch.uint8), s.squeeze(-1)

    try:
        q, s = torch.empty((rows, cols), dtype=torch.uint8, device="cuda"), torch.empty((cols // 128, rows), device="cuda")
        gpu_lib.moe_quantize_fp8(ctx, xb.cuda(), rows, cols, 128, None, 1, q, s)
        q_e, s_e = expected(xb.view(rows, cols // 128, 128))
        assert torch.equal(q.cpu().view(rows, cols // 128, 128), q_e) and torch.equal(s.cpu().T, s_e)
        qw, sw = torch.empty((rows, cols), dtype=torch.uint8, device="cuda"), torch.empty((rows // 128, cols // 128), device="cuda")
        gpu_lib.moe_quantize_weights_fp8(ctx, xb.cuda(), rows, cols, qw, sw)
        blocks = lambda t: t.view(rows // 128, 128, cols // 128, 128).transpose(1, 2).reshape(rows // 128, cols // 128, -1)
        q_e, s_e = expected(blocks(xb))
        assert torch.equal(blocks(qw.cpu()), q_e) and torch.equal(sw.cpu(), s_e)
    finally:
        gpu_lib.moe_destroy(ctx)


# --------------------------------------------------------------------------- products that do not fill the chip
# either side of every tile height (16, 32, 64 rows) and of a round's four K blocks; one, two and three row tiles
@pytest.mark.parametrize("rows", [1, 15, 16, 17, 32, 33, 48, 49, 64, 65, 130])
@pytest.mark.parametrize("K,NOUT", [(128, 256), (384, 128), (512, 1024), (640, 2688), (1152, 128), (66 * 128, 384)])
def test_linear_of_few_blocks(gpu_lib, rows, K, NOUT):
    """At most 256 blocks of 32 features: the same bits as the first NOUT features of a product that is wide enough for the streaming
    kernel or the big tiles (every kernel folds the K blocks in order), whose own tests hold it to a 64-bit evaluation."""
    WIDE = 131 * 128
    assert (rows + 63) // 64 * NOUT // 32 <= 256 < (rows + 63) // 64 * WIDE // 32
    g = torch.Generator(device="cuda").manual_seed(rows + K + NOUT)
    xq, wq = _codes(g, rows, K), _codes(g, WIDE, K)
    xs = torch.rand((K // 128, rows), generator=g, device="cuda") + 0.5
    ws = torch.rand((WIDE // 128, K // 128), generator=g, device="cuda") + 0.5
    ctx = gpu_lib.moe_create(rows, K, 1, 1, WIDE)
    try:
        wide = torch.full((rows, WIDE), float("nan"), device="cuda")
        gpu_lib.moe_linear_fp8(ctx, xq, xs, rows, K, wq, ws, WIDE, wide)
        y = torch.full((rows + 1, NOUT), float("nan"), device="cuda")
        gpu_lib.moe_linear_fp8(ctx, xq, xs, rows, K, wq[:NOUT], ws[:NOUT // 128].contiguous(), NOUT, y)
        assert torch.equal(y[:rows], wide[:, :NOUT])
        assert torch.isnan(y[rows]).all()                    # nothing past the last row
    finally:
        gpu_lib.moe_destroy(ctx)


# 200 and 400 tokens on one set of experts: one and two full tiles an expert, whose weights go past the caches
@pytest.mark.parametrize("T", [1, 2, 5, 16, 200, 400])
@pytest.mark.parametrize("d,E,k,F", [(640, 16, 2, 384), (128, 8, 3, 128), (1152, 5, 1, 1280)])
@pytest.mark.parametrize("hot", [False, True], ids=["spread", "one-set"])
def test_layer_of_a_small_batch_has_the_bits_of_a_large_one(gpu_lib, T, d, E, k, F, hot):
    """The same tokens and log as the first T of 1500, which take the big tiles: the replayed layer's outputs, hidden codes and scales."""
    assert 1500 * k > 48 * E
    g = torch.Generator(device="cuda").manual_seed(T + d + E)
    big = 1500
    x = torch.randn((big, d), generator=g, device="cuda").to(torch.bfloat16)
    ids = torch.rand((big, E), generator=g, device="cuda").topk(k, dim=1).indices.to(torch.int32)
    if hot:
        ids[:T] = ids[0].clone()                               # a tile of T rows for each of k experts
    gates = torch.rand((big, k), generator=g, device="cuda")
    w = {}
    for q, s, r, c in (("W1q", "s1", F, d), ("W3q", "s3", F, d), ("W2q", "s2", d, F)):
        w[q] = _codes(g, E, r, c)
        w[s] = (torch.rand((E, r // 128, c // 128), generator=g, device="cuda") + 0.5) * 1e-3
    out = []
    for n in (big, T):
        layer = gpu_lib.MoELayer(n, d, E, k, F)
        for _ in range(2):                                   # (twice: the tickets of the first call are back at zero)
            layer.forward_replay(x[:n].contiguous(), ids[:n].contiguous(), gates[:n].contiguous(), w)
        hq, hs = layer.hidden()
        at = layer.inv_perm.view(n, k)[:T].long().flatten()
        out.append((layer.y[:T].clone().view(torch.int16), layer.y_perm[at].clone(), hq[at], hs[:, at]))
        layer.close()
    for a, b in zip(*out):
        assert torch.equal(a, b)


# --------------------------------------------------------------------------- quantisation in the permutation's launches
# one block beside the router's last step (T <= 16), one block of its own, three launches; a row more and less than 32
@pytest.mark.parametrize("T,d,E,k", [(1, 128, 8, 2), (16, 1152, 200, 16), (16, 128, 130, 3), (17, 640, 16, 4), (31, 2176, 60, 5),
                                     (33, 128, 5, 1), (700, 384, 256, 6), (2100, 896, 64, 8)])
def test_routing_with_quantisation_is_the_two_calls(gpu_lib, T, d, E, k):
    """Routed and replayed: ids, weights, permutation, codes and scales of the joint call against the separate ones, bit for bit; the
    quantised arrays are written to their ends and not beyond."""
    g = torch.Generator(device="cuda").manual_seed(T + d)
    x = torch.randn((T, d), generator=g, device="cuda").to(torch.bfloat16)
    W_r = torch.randn((E, d), generator=g, device="cuda") * d ** -0.5
    bias = torch.randn((E,), generator=g, device="cuda")
    log = torch.rand((T, E), generator=g, device="cuda").topk(k, dim=1).indices.to(torch.int32).contiguous()
    log_w = torch.rand((T, k), generator=g, device="cuda")
    log[T // 2, 0] = E + 3                                    # reported by both, skipped by both
    ctx = gpu_lib.moe_create(T, d, E, k, 128)

    def outputs():
        i32 = dict(dtype=torch.int32, device="cuda")
        return [torch.full((T, k), -7, **i32), torch.full((T, k), -7.0, device="cuda"), torch.full((E + 1,), -7, **i32),
                torch.full((T * k,), -7, **i32), torch.full((T * k,), -7, **i32)]

    def codes():
        return torch.full((T * d + 64,), 0x55, dtype=torch.uint8, device="cuda"), torch.full((T * d // 128 + 16,), -7.0, device="cuda")
    try:
        for routed in (True, False):
            a, b, (qa, sa), (qb, sb) = outputs(), outputs(), codes(), codes()
            if routed:
                gpu_lib.moe_route(ctx, x, W_r, bias, k, *a)
                gpu_lib.moe_quantize_fp8(ctx, x, T, d, 128, None, 1, qa, sa)
                gpu_lib.moe_route_quantize(ctx, x, W_r, bias, k, *b, qb, sb)
                assert gpu_lib.moe_check_ids(ctx) == 0
            else:
                gpu_lib.moe_route_replay(ctx, x, log, log_w, *a)
                assert gpu_lib.moe_check_ids(ctx) != 0
                gpu_lib.moe_quantize_fp8(ctx, x, T, d, 128, None, 1, qa, sa)
                gpu_lib.moe_route_replay_quantize(ctx, x, log, log_w, *b, qb, sb)
                assert gpu_lib.moe_check_ids(ctx) != 0
            for u, v in zip(a + [qa, sa], b + [qb, sb]):
                assert torch.equal(u, v)
            assert (qb[T * d:] == 0x55).all() and (sb[T * d // 128:] == -7.0).all()
    finally:
        gpu_lib.moe_destroy(ctx)


@pytest.mark.parametrize("T,d,E,k", [(1, 256, 8, 2), (16, 640, 256, 16), (13, 1152, 60, 5)])
def test_one_block_router_permutes_as_the_log_does(gpu_lib, T, d, E, k):
    """Up to 16 tokens the router's last block permutes: against the replay of its own log, which permutes in a launch of its own; ids-only
    replay of that log gives the same weights, and a repeated id is reported."""
    g = torch.Generator(device="cuda").manual_seed(T + d)
    x = torch.randn((T, d), generator=g, device="cuda").to(torch.bfloat16)
    W_r = torch.randn((E, d), generator=g, device="cuda") * d ** -0.5
    ctx = gpu_lib.moe_create(T, d, E, k, 128)
    new = lambda: [torch.empty((T, k), dtype=torch.int32, device="cuda"), torch.empty((T, k), device="cuda"),
                   *(torch.full((n,), -7, dtype=torch.int32, device="cuda") for n in (E + 1, T * k, T * k))]
    try:
        a, b, c = new(), new(), new()
        gpu_lib.moe_route(ctx, x, W_r, None, k, *a)
        gpu_lib.moe_route_replay(ctx, x, a[0], a[1], *b)
        gpu_lib.moe_route_replay_ids(ctx, x, W_r, a[0], *c)
        assert gpu_lib.moe_check_ids(ctx) == 0
        for u, v, w in zip(a, b, c):
            assert torch.equal(u, v) and torch.equal(u, w)
        twice = a[0].clone()
        twice[T - 1, k - 1] = twice[T - 1, 0]
        gpu_lib.moe_route_replay_ids(ctx, x, W_r, twice, *c)
        assert gpu_lib.moe_check_ids(ctx) != 0
    finally:
        gpu_lib.moe_destroy(ctx)


# 255 and 260 units of 64 rows x 256 features: the streaming kernel, and big tiles of the height that fills a round; one short row tile
@pytest.mark.parametrize("rows,K,NOUT", [(300, 384, 51 * 256), (300, 384, 52 * 256), (300, 640, 52 * 256 - 128), (65, 256, 131 * 256)])
def test_linear_either_side_of_the_streaming_line(gpu_lib, rows, K, NOUT):
    """The same bits as in calls of 64 rows, which stream."""
    g = torch.Generator(device="cuda").manual_seed(rows + NOUT)
    xq, wq = _codes(g, rows, K), _codes(g, NOUT, K)
    xs = torch.rand((K // 128, rows), generator=g, device="cuda") + 0.5
    ws = torch.rand((NOUT // 128, K // 128), generator=g, device="cuda") + 0.5
    ctx = gpu_lib.moe_create(rows, K, 1, 1, NOUT)
    try:
        y = torch.full((rows + 1, NOUT), float("nan"), device="cuda")
        gpu_lib.moe_linear_fp8(ctx, xq, xs, rows, K, wq, ws, NOUT, y)
        part = torch.empty((64, NOUT), device="cuda")
        for r in range(0, rows, 64):
            n = min(64, rows - r)
            gpu_lib.moe_linear_fp8(ctx, xq[r:r + n], xs[:, r:r + n].contiguous(), n, K, wq, ws, NOUT, part)
            assert torch.equal(y[r:r + n], part[:n]), r
        assert torch.isnan(y[rows]).all()
    finally:
        gpu_lib.moe_destroy(ctx)


# --------------------------------------------------------------------------- the order of a sum
def _cancelling_rows(g, n, K):
    """Codes [n, K] for activations of 256 in even and 2^-9 in odd columns: in every K block a product of 2^16, one of -2^16 and one of
    2^-18, each in a 16-column piece of its own.  The matrix instructions add such pieces one after another and keep some 24 bits, so
    whether the small one is in the result depends on their order, and only the order that all kernels promise gives the same bits."""
    w = torch.zeros((n, K // 128, 8, 16), dtype=torch.uint8, device="cuda")
    piece = torch.rand((n, K // 128, 8), generator=g, device="cuda").argsort(dim=2)
    at = torch.randint(0, 8, (n, K // 128, 3), generator=g, device="cuda") * 2
    for j, code in enumerate((0x78, 0xF8, 0x01)):
        p, col = piece[..., j], at[..., j] + (j == 2)
        w.view(n, K // 128, 128).scatter_(2, (p * 16 + col)[..., None], code)
    return w.view(n, K)


def _alternating(*shape):
    x = torch.full(shape, 0x78, dtype=torch.uint8, device="cuda")
    x[..., 1::2] = 0x01
    return x


@pytest.mark.parametrize("rows", [1, 17, 40, 64, 300])
@pytest.mark.parametrize("K", [128, 640])
def test_linear_sums_in_one_order(gpu_lib, rows, K):
    """Tiles of 16, 32 and 64 rows in small blocks, the streaming kernel and the big tiles: one order of a row's products."""
    WIDE = 131 * 256
    g = torch.Generator(device="cuda").manual_seed(rows + K)
    wq, xq = _cancelling_rows(g, WIDE, K), _alternating(rows, K)
    xs, ws = torch.ones((K // 128, rows), device="cuda"), torch.ones((WIDE // 128, K // 128), device="cuda")
    ctx = gpu_lib.moe_create(rows, K, 1, 1, WIDE)
    try:
        out = []
        for n in (WIDE, 4096, 1024):                          # big tiles or streaming, then smaller forms
            y = torch.full((rows, n), float("nan"), device="cuda")
            gpu_lib.moe_linear_fp8(ctx, xq, xs, rows, K, wq[:n], ws[:n // 128].contiguous(), n, y)
            out.append(y[:, :1024].clone())
        kept = out[0][0] * 2.0 ** 18                          # K blocks whose small product is in the sum
        assert (kept == 0).any() and (kept == K // 128).any()
        for y in out[1:]:
            assert torch.equal(y, out[0])
        assert (out[0] == out[0][0]).all()                    # nor does a row's place in its tile matter
    finally:
        gpu_lib.moe_destroy(ctx)


@pytest.mark.parametrize("T", [1, 5, 16, 200, 400])
@pytest.mark.parametrize("which", ["gate_up", "down"])
def test_layer_sums_in_one_order(gpu_lib, T, which):
    """The first T of 1500 tokens, which take the big tiles, in small blocks, the streaming kernel and narrow tiles."""
    d, E, k, F, big = 640, 16, 2, 384, 1500
    g = torch.Generator(device="cuda").manual_seed(T)
    ids = torch.rand((big, E), generator=g, device="cuda").topk(k, dim=1).indices.to(torch.int32)
    gates = torch.rand((big, k), generator=g, device="cuda")
    one = lambda r, c: torch.ones((E, r // 128, c // 128), device="cuda")
    w = {"s1": one(F, d), "s3": one(F, d), "s2": one(d, F)}
    if which == "gate_up":                                    # codes of scale 1: 256 and 2^-9, a maximum of 448 in every group
        x = _alternating(big, d).view(torch.float8_e4m3fn).to(torch.bfloat16)
        x.view(big, d // 128, 128)[:, :, 126] = 448.0
        for n in ("W1q", "W3q"):
            w[n] = _cancelling_rows(g, E * F, d).view(E, F, d)
            w[n].view(E, F, d // 128, 128)[..., 126] = 0
        w["s1"] *= 2.0 ** 18
        w["s3"] *= 2.0 ** 18
        w["W2q"] = _codes(g, E, d, F)
    else:                                                     # one column of x decides: h is 448^3 and 448^2 * 2^-9 in turn
        x = torch.zeros((big, d), device="cuda", dtype=torch.bfloat16)
        x[:, 0] = 448.0
        w["W1q"] = torch.zeros((E, F, d), dtype=torch.uint8, device="cuda")
        w["W3q"] = w["W1q"].clone()
        w["W1q"][:, :, 0] = 0x38
        w["W3q"][:, :, 0] = 0x7E
        w["W3q"][:, 1::2, 0] = 0x01
        w["W2q"] = _cancelling_rows(g, E * d, F).view(E, d, F)
    out = []
    for n in (big, T):
        layer = gpu_lib.MoELayer(n, d, E, k, F)
        layer.forward_replay(x[:n].contiguous(), ids[:n].contiguous(), gates[:n].contiguous(), w)
        hq, hs = layer.hidden()
        at = layer.inv_perm.view(n, k)[:T].long().flatten()
        out.append((hq[at], hs[:, at], layer.y_perm[at].clone(), layer.y[:T].clone().view(torch.int16)))
        layer.close()
    if which == "gate_up":
        h = out[0][0][0]
        assert (h == 0).any() and (h != 0).any()
    else:
        small = out[0][2][0].abs()
        assert out[0][0][0].unique().numel() == 2 and small.unique().numel() > 1
    for a, b in zip(*out):
        assert torch.equal(a, b)
