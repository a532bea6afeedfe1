"""GPU: the weight-streaming GEMMs in persistent blocks (csrc/ffn_flow.hip), at the edges of their tiles and of what they accept."""
import numpy as np
import pytest
import torch

from test_flow_rules_host import EDGE_ROWS, LAYERS

pytestmark = pytest.mark.gpu


def _log(counts, k, extra, g):
    """k ids a token so that expert e has counts[e] rows; behind them `extra` tokens of k further experts."""
    E = len(counts)
    slots = [np.repeat(np.arange(E, dtype=np.int32), c) for c in (counts if k == 1 else (counts + 1) // 2, counts // 2)][:k]
    T = max(len(s) for s in slots)
    ids = np.stack([np.resize(s, T) for s in slots], axis=1)
    if k == 2:
        ids[:, 1] = (ids[:, 0] + 1 + np.arange(T) % (E - 1)) % E
    ids = ids[g.permutation(T)]
    return np.concatenate([ids, np.tile(np.arange(E, E + k, dtype=np.int32), (extra, 1))]), T


@pytest.mark.parametrize("name", sorted(LAYERS))
def test_persistent_blocks_have_the_bits_of_the_big_tiles(gpu_lib, name):
    """Hidden codes, their scales and the expert outputs of a layer that streams in persistent blocks, gathered and expert-ordered: the
    bits that its rows get in a batch with so many further rows that the big tiles take it (which the other files compare with the
    oracle).  Tiles of 1 to 96 rows in steps of 16 and either side of them, experts of no row, of one row and of several tiles."""
    d, E, k, F, scale = LAYERS[name]
    g = np.random.default_rng(d + E + k)
    counts = np.maximum(np.resize(EDGE_ROWS, E) * scale // 4, 0)
    extra = 97 * (E + k)                                       # more than 96 rows per expert
    ids, T = _log(counts, k, extra, g)
    gen = torch.Generator(device="cuda").manual_seed(d + F)
    code = lambda *s: (torch.randn(s, generator=gen, device="cuda") * 60).to(torch.float8_e4m3fn).view(torch.uint8)
    scales = lambda *s: torch.rand(s, generator=gen, device="cuda") * 2e-4 + 1e-4
    w = {"W1q": code(E + k, F, d), "W3q": code(E + k, F, d), "W2q": code(E + k, d, F), "s1": scales(E + k, F // 128, d // 128),
         "s3": scales(E + k, F // 128, d // 128), "s2": scales(E + k, d // 128, F // 128)}
    few = {n: v[:E].contiguous() for n, v in w.items()}
    x = torch.randn((T + extra, d), generator=gen, device="cuda").to(torch.bfloat16)
    gates = torch.rand((T + extra, k), generator=gen, device="cuda")
    ids = torch.from_numpy(ids).cuda()
    big, layer = gpu_lib.MoELayer(T + extra, d, E + k, k, F), gpu_lib.MoELayer(T, d, E, k, F)
    try:
        big.forward_replay(x, ids, gates, w)
        hq_w, hs_w = big.hidden()
        N = T * k
        assert int(big.offsets[E]) == N
        for fused in (True, False):
            layer.y_perm.fill_(float("nan"))
            y = layer.forward_replay(x[:T].contiguous(), ids[:T].contiguous(), gates[:T].contiguous(), few, fused=fused)
            hq, hs = layer.hidden()
            assert torch.equal(layer.offsets, big.offsets[:E + 1])
            assert torch.equal(hs.view(torch.int32), hs_w[:, :N].contiguous().view(torch.int32)), fused
            assert torch.equal(hq, hq_w[:N]), fused
            assert torch.equal(layer.y_perm.view(torch.int32), big.y_perm[:N].view(torch.int32)), fused
            assert torch.equal(y.view(torch.int16), big.y[:T].view(torch.int16)), fused
    finally:
        big.close()
        layer.close()


def test_values_and_ids_that_are_not_valid(gpu_lib):
    """Slots of ids outside [0, E) have no row; activations that are not finite, weight codes of NaN and scales of infinity reach the rows
    that multiply them and no others: hidden codes, scales and outputs are those of the big tiles, a NaN for a NaN."""
    d, E, k, F, scale = LAYERS["two-a-token"]
    g = np.random.default_rng(5)
    extra = 97 * (E + k)
    ids, T = _log(np.resize(EDGE_ROWS, E) * scale // 4, k, extra, g)
    assert T > 40
    for n, bad in enumerate((-1, E + k, 1 << 20, -(1 << 31))):
        ids[7 * n + 3, n % 2] = bad
    ids[30] = -1                                               # a token without any row
    gen = torch.Generator(device="cuda").manual_seed(d)
    code = lambda *s: (torch.randn(s, generator=gen, device="cuda") * 60).to(torch.float8_e4m3fn).view(torch.uint8)
    scales = lambda *s: torch.rand(s, generator=gen, device="cuda") * 2e-4 + 1e-4
    w = {"W1q": code(E + k, F, d), "W3q": code(E + k, F, d), "W2q": code(E + k, d, F), "s1": scales(E + k, F // 128, d // 128),
         "s3": scales(E + k, F // 128, d // 128), "s2": scales(E + k, d // 128, F // 128)}
    w["W1q"][3, 5, 7], w["W3q"][20, 130, 0], w["W2q"][6, 200, 300] = 0x7F, 0xFF, 0x7F
    w["s1"][9, 1, 2], w["s2"][12, 0, 3] = float("inf"), float("nan")
    x = torch.randn((T + extra, d), generator=gen, device="cuda").to(torch.bfloat16)
    x[11, 130], x[12, 0], x[13, 700], x[14] = float("nan"), float("inf"), -float("inf"), float("nan")
    gates = torch.rand((T + extra, k), generator=gen, device="cuda")
    ids = torch.from_numpy(ids).cuda()
    big, layer = gpu_lib.MoELayer(T + extra, d, E + k, k, F), gpu_lib.MoELayer(T, d, E, k, F)
    same = lambda a, b: torch.equal(a.isnan(), b.isnan()) and torch.equal(a.nan_to_num(0.0), b.nan_to_num(0.0))
    try:
        big.y_perm.zero_()
        y_w = big.forward_replay(x, ids, gates, w)[:T].clone()
        hq_w, hs_w = big.hidden()
        N = int(big.offsets[E])
        assert N == T * k - 6 and gpu_lib.moe_check_ids(big.ctx) != 0
        for fused in (True, False):
            layer.y_perm.zero_()
            y = layer.forward_replay(x[:T].contiguous(), ids[:T].contiguous(), gates[:T].contiguous(),
                                     {n: v[:E].contiguous() for n, v in w.items()}, fused=fused)
            assert gpu_lib.moe_check_ids(layer.ctx) != 0
            hq, hs = layer.hidden()
            assert torch.equal(layer.offsets, big.offsets[:E + 1])
            assert same(hs[:, :N], hs_w[:, :N]) and torch.equal(hq[:N], hq_w[:N]), fused
            assert same(layer.y_perm[:N], big.y_perm[:N]) and not layer.y_perm[N:].any(), fused
            assert same(y, y_w), fused
        assert y_w[30].eq(0).all() and 0 < int(y_w.isnan().any(dim=1).sum()) < T // 2
    finally:
        big.close()
        layer.close()
