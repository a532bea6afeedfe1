"""GPU: the router of one to four tokens in one launch (route_tiny in csrc/route.hip): the bits that the same tokens get in a batch of
sixteen, which takes the launches it replaces; the permutation of the replayed log; ids that are not valid."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,E,k", [(128, 1, 1), (1024, 4, 4), (1152, 5, 3), (4096, 64, 6), (4224, 48, 16), (640, 256, 16)])
@pytest.mark.parametrize("T", [1, 2, 3, 4])
def test_tokens_of_a_tiny_batch(gpu_lib, T, d, E, k):
    assert (E + 3) // 4 * ((d + 1023) // 1024) <= 64
    g = torch.Generator(device="cuda").manual_seed(d + E + T)
    x = torch.randn((16, d), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn((E, d), generator=g, device="cuda") * d ** -0.5
    bias = torch.randn((E,), generator=g, device="cuda")
    tiny, large = gpu_lib.MoELayer(T, d, E, k, 128), gpu_lib.MoELayer(16, d, E, k, 128)
    log = gpu_lib.MoELayer(T, d, E, k, 128)
    try:
        for step, b in enumerate((None, bias, None)):                    # calls in a row: the ticket starts at zero each time
            xs = torch.roll(x, step, 0)
            tiny.perm.fill_(-7), tiny.inv_perm.fill_(-7), tiny.offsets.fill_(-7)
            gpu_lib.moe_route_quantize(tiny.ctx, xs[:T].contiguous(), W, b, k, tiny.topk_idx, tiny.topk_w, tiny.offsets, tiny.perm,
                                       tiny.inv_perm, tiny.xq_tok, tiny.xs_tok)
            large.route(xs, W, b)
            large.quantize_tokens(xs)
            log.route_replay(xs[:T].contiguous(), tiny.topk_idx, tiny.topk_w)
            assert torch.equal(tiny.topk_idx, large.topk_idx[:T])
            assert torch.equal(tiny.topk_w.view(torch.int32), large.topk_w[:T].view(torch.int32))
            assert torch.equal(tiny.xq_tok, large.xq_tok[:T]) and torch.equal(tiny.xs_tok, large.xs_tok[:, :T])
            for name in ("offsets", "perm", "inv_perm"):
                assert torch.equal(getattr(tiny, name), getattr(log, name)), name
            w = tiny.topk_w.clone()
            if b is None:                                                # ids given: the router's own weights again
                tiny.route_replay_ids(xs[:T].contiguous(), W, log.topk_idx)
                assert torch.equal(tiny.topk_w.view(torch.int32), w.view(torch.int32))
                assert torch.equal(tiny.inv_perm, log.inv_perm) and torch.equal(tiny.offsets, log.offsets)
        assert gpu_lib.moe_check_ids(tiny.ctx) == 0
    finally:
        for layer in (tiny, large, log):
            layer.close()


def test_ids_that_are_not_valid_are_reported(gpu_lib):
    T, d, E, k = 4, 256, 8, 3
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn((T, d), generator=g, device="cuda").to(torch.bfloat16)
    W = torch.randn((E, d), generator=g, device="cuda")
    good = torch.tensor([[0, 1, 2], [2, 1, 0], [7, 0, 3], [2, 4, 6]], dtype=torch.int32, device="cuda")
    layer, log = gpu_lib.MoELayer(T, d, E, k, 128), gpu_lib.MoELayer(T, d, E, k, 128)
    try:
        for bad in (None, (1, 1, 8), (3, 0, -1), (2, 2, 7), (0, 1, 0)):  # (token, slot, id): outside [0, E), or a repeat
            ids = good.clone()
            if bad:
                ids[bad[0], bad[1]] = bad[2]
            layer.route_replay_ids(x, W, ids)
            log.route_replay(x, ids, layer.topk_w)
            for name in ("offsets", "inv_perm"):
                assert torch.equal(getattr(layer, name), getattr(log, name)), (bad, name)
            n = int(layer.offsets[E])
            assert torch.equal(layer.perm[:n], log.perm[:n])
            for c in (layer.ctx, log.ctx):
                assert (gpu_lib.moe_check_ids(c) != 0) == bool(bad), bad
    finally:
        layer.close()
        log.close()
