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
