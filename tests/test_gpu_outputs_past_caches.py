"""GPU: products whose output rows go past the caches (csrc/ffn_rules.hpp, from 256 MB of a linear's y and 768 MB of a layer's rows)
against the same rows in calls below those lines, bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _codes(g, *shape):
    return (torch.randn(shape, generator=g, device="cuda") * 60).to(torch.float8_e4m3fn).view(torch.uint8)


@pytest.mark.parametrize("rows,K,NOUT", [(8200, 2048, 8320), (65536 + 37, 2048, 1152)])
def test_linear(gpu_lib, rows, K, NOUT):
    assert rows * NOUT * 4 >= 256 << 20 > (rows + 1) // 2 * NOUT * 4
    g = torch.Generator(device="cuda").manual_seed(rows)
    xq, wq = _codes(g, rows, K), _codes(g, NOUT, K)
    xs = torch.rand((K // 128, rows), generator=g, device="cuda") + 0.5
    ws = torch.rand((NOUT // 128, K // 128), generator=g, device="cuda") + 0.5
    ctx = gpu_lib.moe_create(rows, K, 1, 1, NOUT)
    try:
        y = torch.full((rows, NOUT), float("nan"), device="cuda")
        gpu_lib.moe_linear_fp8(ctx, xq, xs, rows, K, wq, ws, NOUT, y)
        for r in (0, rows // 2):
            n = (rows - r) if r else rows // 2
            part = torch.full((n, NOUT), float("nan"), device="cuda")
            gpu_lib.moe_linear_fp8(ctx, xq[r:r + n], xs[:, r:r + n].contiguous(), n, K, wq, ws, NOUT, part)
            assert torch.equal(y[r:r + n], part)
    finally:
        gpu_lib.moe_destroy(ctx)


def test_layer(gpu_lib):
    """Experts of full and ragged tiles and one whose rows make a narrow tile; an odd number of feature blocks."""
    T, d, E, F = 24700, 8320, 8, 128
    assert T * d * 4 >= 768 << 20 > (T - T // 2) * d * 4
    g = torch.Generator(device="cuda").manual_seed(T)
    ids = torch.randint(0, E - 1, (T, 1), generator=g, device="cuda", dtype=torch.int32)
    ids[100:150] = E - 1
    x = torch.randn((T, d), generator=g, device="cuda").to(torch.bfloat16)
    gates = torch.rand((T, 1), generator=g, device="cuda")
    scales = lambda *s: torch.rand(s, generator=g, device="cuda") * 2e-4 + 1e-4
    w = {"W1q": _codes(g, E, F, d), "W3q": _codes(g, E, F, d), "W2q": _codes(g, E, d, F), "s1": scales(E, F // 128, d // 128),
         "s3": scales(E, F // 128, d // 128), "s2": scales(E, d // 128, F // 128)}

    def layer(a, b):
        out = gpu_lib.MoELayer(b - a, d, E, 1, F)
        try:
            out.y_perm.fill_(float("nan"))
            out.forward_replay(x[a:b].contiguous(), ids[a:b].contiguous(), gates[a:b].contiguous(), w)
            return out.y.clone(), out.y_perm[out.inv_perm.long()]            # rows in token order
        finally:
            out.close()
    y, rows = layer(0, T)
    for a, b in ((0, T // 2), (T // 2, T)):
        y_p, rows_p = layer(a, b)
        assert torch.equal(rows[a:b], rows_p) and torch.equal(y[a:b].view(torch.int16), y_p.view(torch.int16))
