"""GPU: repeated ids inside a token are found wherever the token lies among the 64 assignments that a wave of the one-block permutation looks at
together, in the two launches as well, and nothing else is reported."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,k", [(3, 8, 2), (40, 60, 5), (65, 256, 16), (300, 17, 7), (819, 60, 5), (640, 64, 8), (1000, 64, 6), (1707, 9, 3)])
def test_repeats(gpu_lib, T, E, k):
    g = torch.Generator(device="cuda").manual_seed(T + k)
    ids = torch.topk(torch.rand((T, E), generator=g, device="cuda"), k, dim=1).indices.to(torch.int32).contiguous()
    w = torch.rand((T, k), generator=g, device="cuda")
    x = torch.zeros((T, 128), dtype=torch.bfloat16, device="cuda")
    layer = gpu_lib.MoELayer(T, 128, E, k, 128)
    try:
        layer.route_replay(x, ids, w)
        assert gpu_lib.moe_check_ids(layer.ctx) == 0
        offsets = layer.offsets.clone()
        across = [t for t in range(T) if t * k // 64 != (t * k + k - 1) // 64]          # tokens that two groups of 64 share
        for t in sorted({0, T // 2, T - 1, *across[:2], *across[-2:]}):
            for first, again in {(0, k - 1), (0, 1), (k - 2, k - 1)}:
                bad = ids.clone()
                bad[t, again] = bad[t, first]
                layer.route_replay(x, bad, w)
                assert gpu_lib.moe_check_ids(layer.ctx) != 0, (t, first, again)
                flat = bad.flatten().long()
                order = torch.sort(flat, stable=True).indices
                assert torch.equal(layer.perm.long(), order)
                assert torch.equal(layer.inv_perm.long()[order], torch.arange(T * k, device="cuda"))
                assert torch.equal(layer.topk_idx, bad) and torch.equal(layer.topk_w, w)
        layer.route_replay(x, ids, w)
        assert gpu_lib.moe_check_ids(layer.ctx) == 0 and torch.equal(layer.offsets, offsets)
    finally:
        layer.close()
