"""GPU: the split router either side of the line up to which its waves split the fp32 weights themselves (route_splits_weights in csrc/route.hip),
against a 64-bit evaluation: the selected experts wherever their scores are not close, their weights to the tolerance of the other files."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E,k,chunks", [(33, 2048, 5, 3, 1), (64, 4096, 64, 6, 2), (129, 7168, 130, 8, 4), (500, 2176, 256, 16, 2),
                                            (1000, 4096, 33, 2, 4), (1000, 4352, 33, 2, 5), (2049, 1024, 96, 4, 3), (4096, 1152, 128, 1, 5),
                                            (2049, 1024, 160, 4, 3), (1000, 2048, 256, 8, 2), (2560, 384, 256, 8, 1), (2624, 384, 256, 8, 1)])
def test_either_side_of_the_line(gpu_lib, T, d, E, k, chunks):
    splits = max(1, min(16, 256 // ((T + 31) // 32)))
    assert (d // 128 + splits - 1) // splits == chunks
    g = torch.Generator(device="cuda").manual_seed(T + d)
    x = torch.randn((T, d), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn((E, d), generator=g, device="cuda") * d ** -0.5
    W[:, ::5] *= 2.0 ** -9                                               # magnitudes far apart: all three planes of a weight count
    bias = torch.randn((E,), generator=g, device="cuda")
    logits = x.double() @ W.double().T.contiguous()
    layer = gpu_lib.MoELayer(T, d, E, k, 128)
    try:
        for b in (None, bias):
            layer.route(x, W, b)
            score = logits if b is None else logits + b.double()
            top = torch.sort(score, dim=1, descending=True)
            gaps = (top.values[:, :-1] - top.values[:, 1:])[:, :k] if E > k else top.values[:, :-1] - top.values[:, 1:]
            clear = (gaps > 1e-4).all(dim=1)
            assert clear.float().mean() > 0.9
            ids = layer.topk_idx.long()
            assert torch.equal(ids[clear], top.indices[clear][:, :k])
            w = torch.softmax(logits.gather(1, ids), dim=1)
            assert ((layer.topk_w.double() - w).abs() <= 1e-6 + 1e-5 * w).all()
            routed = layer.topk_w.clone()
            layer.route_replay_ids(x, W, layer.topk_idx.clone())         # the same logits again
            assert torch.equal(layer.topk_w.view(torch.int32), routed.view(torch.int32))
    finally:
        layer.close()


@pytest.mark.parametrize("E,k", [(33, 16), (150, 16)])
@pytest.mark.parametrize("chunks", [1, 2, 3, 4])
def test_weights_split_by_the_waves_give_the_bits_of_the_planes(gpu_lib, chunks, E, k):
    """1000 tokens take eight blocks a token tile.  With up to four chunks of 128 columns to a block the waves split the weights; five are
    multiplied from planes.  The same columns of every block, in the second batch with zeros of x behind them, have to give the same partial
    logits: the same ids and the same bits of their weights.  Every 7th column is of weights whose last planes are subnormal."""
    T, blocks = 1000, 8
    assert min(16, 256 // ((T + 31) // 32)) == blocks and chunks * 32 * E <= 20480
    g = torch.Generator(device="cuda").manual_seed(chunks + E)
    W = torch.randn((E, blocks, chunks * 128), generator=g, device="cuda") * (blocks * chunks * 128) ** -0.5
    x = torch.randn((T, blocks, chunks * 128), generator=g, device="cuda").to(torch.bfloat16)
    W[:, :, ::5] *= 2.0 ** -9
    W[:, :, 3::7] *= 2.0 ** -112
    x[:, :, 3::7] *= 2.0 ** 112
    pad = (5 - chunks) * 128
    W_5 = torch.cat([W, torch.randn((E, blocks, pad), generator=g, device="cuda")], dim=2).reshape(E, -1).contiguous()
    x_5 = torch.cat([x, torch.zeros((T, blocks, pad), dtype=torch.bfloat16, device="cuda")], dim=2).reshape(T, -1).contiguous()
    raw, planes = gpu_lib.MoELayer(T, blocks * chunks * 128, E, k, 128), gpu_lib.MoELayer(T, blocks * 640, E, k, 128)
    try:
        for bias in (None, torch.randn((E,), generator=g, device="cuda")):
            raw.route(x.reshape(T, -1), W.reshape(E, -1), bias)
            planes.route(x_5, W_5, bias)
            assert torch.equal(raw.topk_idx, planes.topk_idx)
            assert torch.equal(raw.topk_w.view(torch.int32), planes.topk_w.view(torch.int32))
        logits = x.reshape(T, -1).double() @ W.reshape(E, -1).double().T.contiguous()
        w = torch.softmax(logits.gather(1, raw.topk_idx.long()), dim=1)
        assert ((raw.topk_w.double() - w).abs() <= 1e-6 + 1e-5 * w).all()
    finally:
        raw.close()
        planes.close()
