"""3x3 convolution on 16x16x32 MFMAs (tiles of 4 or 8 rows x 16 pixels): every instantiation at ragged tile edges against nine shifted
products in 64 bits, without and with residual and moments, at one type's rounding of the result."""
import pytest
import torch

from paper_2602_00608_amd import synth, wmdec
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


# 64 x 128 tiles; 128 x 128 with moments per four rows, short and whole ring of weights; 128 x 128, both rings, and of 256 channels; 128 x 256, one and two chunks
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("n,cin,cout,h,w", [(1, 32, 128, 5, 17), (5, 32, 256, 37, 50), (16, 32, 256, 37, 50), (1, 96, 128, 121, 67),
                                            (1, 32, 128, 127, 530), (1, 32, 256, 257, 259), (1, 64, 256, 182, 367),
                                            (1, 32, 256, 100, 203), (2, 64, 256, 91, 130)])
def test_tile_edges(dtype, n, cin, cout, h, w):
    g = torch.Generator(device="cuda")
    g.manual_seed(synth.SEED_BASE + 60)

    def draw(*shape):
        return torch.randn(shape, generator=g, device="cuda")
    x, res, bias = draw(n, h, w, cin).to(G.TORCH[dtype]), draw(n, h, w, cout).to(G.TORCH[dtype]), draw(cout)
    wt = (draw(cout, cin, 3, 3) / (9 * cin) ** 0.5).bfloat16()
    packed = G.pack(wt.float().cpu().numpy(), dtype)
    pad = torch.zeros((n, h + 2, w + 2, cin), dtype=torch.float64, device="cuda")
    pad[:, 1:-1, 1:-1] = x.double()
    conv = bias.double().expand(n * h * w, cout).clone()
    for ky in range(3):
        for kx in range(3):
            conv += pad[:, ky:ky + h, kx:kx + w].reshape(-1, cin) @ wt[:, :, ky, kx].double().t().contiguous()
    conv = conv.view(n, h, w, cout)
    groups, ulp = 32, 2.0 ** -8 if dtype == "bf16" else 2.0 ** -11
    ws = torch.zeros(wmdec.conv_stats_workspace_bytes(G.ENUM[dtype], G.ENUM[dtype], n, h, w, cin, cout, groups), dtype=torch.uint8, device="cuda")
    mean, rstd = torch.empty(n * groups, device="cuda"), torch.empty(n * groups, device="cuda")
    for residual, ydtype, stats in ((None, "f32", False), (None, dtype, False), (None, dtype, True), (res, dtype, False), (res, dtype, True)):
        y, check = G.canaried((n, h, w, cout), G.TORCH[ydtype])
        if stats:
            wmdec.gn_silu_conv3x3_stats(x, None, None, None, None, 1, False, packed, bias, residual, y, groups, 1e-6, mean, rstd, ws)
        else:
            wmdec.gn_silu_conv3x3(x, None, None, None, None, 1, False, packed, bias, residual, y)
        torch.cuda.synchronize()
        check()
        want = conv if residual is None else conv + res.double()
        # operands are exact: fp32 sums of 9 * cin products, and half an ulp of a 16-bit output's own size
        tol = 2e-5 * want.pow(2).mean().sqrt() + (0.0 if ydtype == "f32" else ulp) * want.abs()
        assert bool(((y.double() - want).abs() <= tol).all()), (residual is not None, ydtype, stats, float(((y.double() - want).abs() - tol).max()))
        if stats:   # of the stored values
            v = y.double().view(n, h * w, groups, cout // groups)
            m, r = v.mean((1, 3)).flatten(), (v.var((1, 3), unbiased=False) + 1e-6).rsqrt().flatten()
            assert float((mean.double() - m).abs().max()) <= 2e-5 and float((rstd.double() / r - 1).abs().max()) <= 2e-5


# 91 tiles of 8 x 16 pixels a sample and 256 channels: 128-channel tiles for one or three samples, 256-channel tiles for two or five
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("cin2", [0, 96])
def test_a_sample_keeps_its_bits_where_the_batch_chooses_the_width(dtype, cin2):
    n, h, w, cin, cout, groups = 5, 100, 100, 64, 256, 32
    g = torch.Generator(device="cuda")
    g.manual_seed(synth.SEED_BASE + 61)

    def draw(*shape):
        return torch.randn(shape, generator=g, device="cuda")
    x, res, bias = draw(n, h, w, cin).to(G.TORCH[dtype]), draw(n, h, w, cout).to(G.TORCH[dtype]), draw(cout)
    mean, rstd, gamma, beta = draw(n, groups), draw(n, groups).abs() + 0.5, draw(cin), draw(cin)
    packed = G.pack((draw(cout, cin, 3, 3) / (9 * cin) ** 0.5).bfloat16().float().cpu().numpy(), dtype)
    if cin2:
        x2, bias2 = draw(n, h, w, cin2).to(G.TORCH[dtype]), draw(cout)
        packed2 = G.pack((draw(cout, cin2, 1, 1) / cin2 ** 0.5).bfloat16().float().cpu().numpy(), dtype)

    def run(k):
        y = torch.empty((k, h, w, cout), dtype=G.TORCH[dtype], device="cuda")
        head = (x[:k], mean[:k].reshape(-1), rstd[:k].reshape(-1), gamma, beta, groups, True, packed, bias)
        if cin2:
            wmdec.gn_silu_conv3x3_shortcut(*head, x2[:k], packed2, bias2, y)
            return (y,)
        ws = torch.zeros(wmdec.conv_stats_workspace_bytes(G.ENUM[dtype], G.ENUM[dtype], k, h, w, cin, cout, groups), dtype=torch.uint8, device="cuda")
        m, r = torch.empty((k, groups), device="cuda"), torch.empty((k, groups), device="cuda")
        wmdec.gn_silu_conv3x3_stats(*head, res[:k], y, groups, 1e-6, m, r, ws)
        return y, m, r
    alone = run(1)
    for k in (2, 3, 5):
        batch = run(k)
        torch.cuda.synchronize()
        assert all(torch.equal(a[:1], b[:1]) for a, b in zip(alone, batch)), k
