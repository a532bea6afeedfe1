"""GPU: the weight quantisation in pairs of blocks, which large matrices of an even number of them take, against the same rows in calls
below that size, bit for bit (those are compared with the oracle in the other files)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols", [(128 * 4099, 256), (128 * 129, 8448)])
def test_pairs_of_blocks(gpu_lib, rows, cols):
    assert cols % 256 == 0 and rows * cols * 2 >= 256 << 20
    g = torch.Generator(device="cuda").manual_seed(rows)
    w = torch.randn((rows, cols), generator=g, device="cuda").to(torch.bfloat16)
    w[:128, :128] = 0                                                    # a block of zeros beside one that is not
    w[-128:, -128:] *= 1000.0
    ctx = gpu_lib.moe_create(0, 128, 1, 1, 128)

    def quantize(a, b):
        q = torch.full((b - a, cols), 0x7F, dtype=torch.uint8, device="cuda")
        s = torch.full(((b - a) // 128, cols // 128), float("nan"), device="cuda")
        gpu_lib.moe_quantize_weights_fp8(ctx, w[a:b].contiguous(), b - a, cols, q, s)
        return q, s
    try:
        q, s = quantize(0, rows)
        step = rows // 128 // 3 * 128
        for a in range(0, rows, step):
            b = min(a + step, rows)
            assert (b - a) * cols * 2 < 256 << 20
            q_p, s_p = quantize(a, b)
            assert torch.equal(q[a:b], q_p) and torch.equal(s[a // 128:b // 128], s_p)
    finally:
        gpu_lib.moe_destroy(ctx)
