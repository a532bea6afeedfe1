"""GPU: the split router either side of the line up to which its waves split the fp32 weights themselves (ROUTE_RAW_CHUNKS in csrc/route.hip),
against a 64-bit evaluation: the selected experts wherever their scores are not close, their weights to the tolerance of the other files."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,E,k,chunks", [(33, 2048, 5, 3, 1), (64, 4096, 64, 6, 2), (129, 7168, 130, 8, 4), (500, 2176, 256, 16, 2),
                                            (1000, 4096, 33, 2, 4), (1000, 4352, 33, 2, 5), (2049, 1024, 96, 4, 3), (4096, 1152, 128, 1, 5)])
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
