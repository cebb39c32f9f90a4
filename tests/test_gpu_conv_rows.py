"""3x3 convolution on 16x16x32 MFMAs (tiles of 4 or 8 rows x 16 pixels): every tile and activation at ragged edges against nine shifted
products in 64 bits, without and with residual and moments, at one type's rounding of the result."""
import pytest
import torch

from paper_2602_00608_amd import synth, wmdec
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


# 64 x 128 tiles; 128 x 128 with moments per four rows, whole and short ring of weights (also with one chunk of channels); 128 x 128, whole ring and short;
# 128 x 256, one to nine chunks.  Without normalisation, with scale and shift, with SiLU.
@pytest.mark.parametrize("act", [None, "affine", "silu"])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("n,cin,cout,h,w", [(1, 32, 128, 5, 17), (5, 32, 256, 37, 50), (16, 32, 256, 37, 50), (1, 96, 128, 121, 67),
                                            (1, 32, 128, 127, 530), (1, 32, 256, 257, 259), (1, 64, 256, 182, 367),
                                            (1, 32, 256, 100, 203), (2, 64, 256, 91, 130), (1, 288, 256, 202, 263)])
def test_tile_edges(dtype, n, cin, cout, h, w, act):
    g = torch.Generator(device="cuda")
    g.manual_seed(synth.SEED_BASE + 60)

    def draw(*shape):
        return torch.randn(shape, generator=g, device="cuda")
    x, res, bias = (draw(n, h, w, cin) * 8).round().clamp(-24, 24).div(8).to(G.TORCH[dtype]), draw(n, h, w, cout).to(G.TORCH[dtype]), draw(cout)
    wt = (draw(cout, cin, 3, 3) / (9 * cin) ** 0.5).bfloat16()
    packed = G.pack(wt.float().cpu().numpy(), dtype)
    groups, ulp = 32, 2.0 ** -8 if dtype == "bf16" else 2.0 ** -11
    head, operand = (x, None, None, None, None, 1, False, packed, bias), x.double()
    if act:   # eighths, means in eighths, scales that are powers of two: the scaled value is exact in either type
        mean, rstd = (draw(n, groups) * 4).round().clamp(-8, 8) / 8, 2.0 ** draw(n, groups).round().clamp(-2, 2)
        gamma, beta = 2.0 ** draw(cin).round().clamp(-1, 1), torch.zeros(cin, device="cuda")
        head = (x, mean.flatten(), rstd.flatten(), gamma, beta, groups, act == "silu", packed, bias)
        t = (x - mean.repeat_interleave(cin // groups, 1)[:, None, None]).double() * (gamma * rstd.repeat_interleave(cin // groups, 1))[:, None, None].double()
        operand = (t * torch.sigmoid(t) if act == "silu" else t).to(G.TORCH[dtype]).double()

    def contract(v, weights):
        pad = torch.zeros((n, h + 2, w + 2, cin), dtype=torch.float64, device="cuda")
        pad[:, 1:-1, 1:-1] = v
        out = torch.zeros((n * h * w, cout), dtype=torch.float64, device="cuda")
        for ky in range(3):
            for kx in range(3):
                out += pad[:, ky:ky + h, kx:kx + w].reshape(-1, cin) @ weights[:, :, ky, kx].double().t().contiguous()
        return out.view(n, h, w, cout)
    conv = contract(operand, wt) + bias.double()
    slack = 2 * ulp * contract(operand.abs(), wt.abs()) if act == "silu" else 0.0   # an activated value near a rounding boundary may be the next one
    mean_out, rstd_out = torch.empty(n * groups, device="cuda"), torch.empty(n * groups, device="cuda")
    for residual, ydtype, stats in ((None, "f32", False), (res, "f32", True), (None, "f32", True), (None, dtype, False), (None, dtype, True), (res, dtype, False), (res, dtype, True)):
        y, check = G.canaried((n, h, w, cout), G.TORCH[ydtype])
        if stats:
            ws = torch.zeros(wmdec.conv_stats_workspace_bytes(G.ENUM[dtype], G.ENUM[ydtype], n, h, w, cin, cout, groups), dtype=torch.uint8, device="cuda")
            wmdec.gn_silu_conv3x3_stats(*head, residual, y, groups, 1e-6, mean_out, rstd_out, ws)
        else:
            wmdec.gn_silu_conv3x3(*head, residual, y)
        torch.cuda.synchronize()
        check()
        want = conv if residual is None else conv + res.double()
        # operands are exact: fp32 sums of 9 * cin products, and half an ulp of a 16-bit output's own size
        tol = 2e-5 * want.pow(2).mean().sqrt() + slack + (0.0 if ydtype == "f32" else ulp) * (want.abs() + slack)
        assert bool(((y.double() - want).abs() <= tol).all()), (residual is not None, ydtype, stats, float(((y.double() - want).abs() - tol).max()))
        if stats:   # of the stored values
            v = y.double().view(n, h * w, groups, cout // groups)
            m, r = v.mean((1, 3)).flatten(), (v.var((1, 3), unbiased=False) + 1e-6).rsqrt().flatten()
            assert float((mean_out.double() - m).abs().max()) <= 2e-5 and float((rstd_out.double() / r - 1).abs().max()) <= 2e-5


# groups of 1 to 32 channels: a lane holds two of them, the others of a group are up to 16 lanes of it
@pytest.mark.parametrize("groups", [8, 16, 64, 128, 256])
@pytest.mark.parametrize("n,cin,cout,h,w", [(1, 32, 256, 37, 50), (16, 32, 256, 37, 50), (1, 96, 256, 121, 131), (1, 288, 256, 202, 263)])
def test_moments_of_groups_of_any_size(groups, n, cin, cout, h, w):
    g = torch.Generator(device="cuda")
    g.manual_seed(synth.SEED_BASE + 62)
    x, bias = torch.randn((n, h, w, cin), generator=g, device="cuda").half(), torch.randn(cout, generator=g, device="cuda") * 3
    packed = G.pack((torch.randn((cout, cin, 3, 3), generator=g, device="cuda") / (9 * cin) ** 0.5).bfloat16().float().cpu().numpy(), "f16")
    y = torch.empty((n, h, w, cout), dtype=torch.float16, device="cuda")
    ws = torch.full((wmdec.conv_stats_workspace_bytes(wmdec.F16, wmdec.F16, n, h, w, cin, cout, groups),), 0xA5, dtype=torch.uint8, device="cuda")
    mean, rstd = torch.empty(n * groups, device="cuda"), torch.empty(n * groups, device="cuda")
    wmdec.gn_silu_conv3x3_stats(x, None, None, None, None, 1, False, packed, bias, None, y, groups, 1e-6, mean, rstd, ws)
    v = y.double().view(n, h * w, groups, cout // groups)
    m, sd = v.mean((1, 3)).flatten(), v.var((1, 3), unbiased=False).flatten().sqrt()
    # fp32 sums shifted by a value of the block: a few 2^-24 of the values, which are up to some 5 standard deviations
    assert float(((mean.double() - m) / sd).abs().max()) <= 4e-6 and float((rstd.double() * (sd ** 2 + 1e-6).sqrt() - 1).abs().max()) <= 4e-6


# 91 tiles of 8 x 16 pixels a sample and 256 channels: 128-channel tiles for one or three samples, 256-channel tiles for two or five (beside a residual
# from 128 input channels on)
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("cin,cin2", [(64, 0), (64, 96), (128, 0)])
def test_a_sample_keeps_its_bits_where_the_batch_chooses_the_width(dtype, cin, cin2):
    n, h, w, cout, groups = 5, 100, 100, 256, 32
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


# tiles of six rows and the eight-row tiles that share their moments: 96 x 128 (one or two samples of 128 channels, one of 256), 96 x 256 (two of 256
# channels), 128 x 128 (three of 128, with a short ring of weights and a whole one; seven of 256) and 128 x 256 (five)
PAIR = [(1, 128, 128, 131, 145), (3, 128, 128, 131, 145), (3, 256, 128, 131, 145), (1, 256, 256, 101, 99), (2, 256, 256, 101, 99), (5, 256, 256, 101, 99), (7, 256, 256, 101, 99)]


@pytest.mark.parametrize("act", [None, "affine", "silu"])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("n,cin,cout,h,w", PAIR)
def test_tile_edges_where_the_height_is_chosen(dtype, n, cin, cout, h, w, act):
    test_tile_edges(dtype, n, cin, cout, h, w, act)


def _same_bits_in_batches(dtype, sizes, cin, cin2, cout, h, w, groups):
    n, g = max(sizes), torch.Generator(device="cuda")
    g.manual_seed(synth.SEED_BASE + 63)

    def draw(*shape):
        return torch.randn(shape, generator=g, device="cuda")
    x, res, bias = draw(n, h, w, cin).to(G.TORCH[dtype]), draw(n, h, w, cout).to(G.TORCH[dtype]), draw(cout)
    mean, rstd, gamma, beta = draw(n, 32), draw(n, 32).abs() + 0.5, draw(cin), draw(cin)
    packed = G.pack((draw(cout, cin, 3, 3) / (9 * cin) ** 0.5).bfloat16().float().cpu().numpy(), dtype)
    if cin2:
        x2, bias2 = draw(n, h, w, cin2).to(G.TORCH[dtype]), draw(cout)
        packed2 = G.pack((draw(cout, cin2, 1, 1) / cin2 ** 0.5).bfloat16().float().cpu().numpy(), dtype)

    def run(k):
        y = torch.empty((k, h, w, cout), dtype=G.TORCH[dtype], device="cuda")
        head = (x[:k], mean[:k].reshape(-1), rstd[:k].reshape(-1), gamma, beta, 32, True, packed, bias)
        if cin2:
            wmdec.gn_silu_conv3x3_shortcut(*head, x2[:k], packed2, bias2, y)
            return (y,)
        ws = torch.full((wmdec.conv_stats_workspace_bytes(G.ENUM[dtype], G.ENUM[dtype], k, h, w, cin, cout, groups),), 0xA5, dtype=torch.uint8, device="cuda")
        m, r = torch.empty((k, groups), device="cuda"), torch.empty((k, groups), device="cuda")
        wmdec.gn_silu_conv3x3_stats(*head, res[:k], y, groups, 1e-6, m, r, ws)
        return y, m, r
    first, *others = [run(k) for k in sizes]
    for k, batch in zip(sizes[1:], others):
        assert all(torch.equal(a, b[:sizes[0]]) for a, b in zip(first, batch)), k
    if not cin2:
        y, m, r = first
        v = y.double().view(sizes[0], h * w, groups, cout // groups)
        mu, sd = v.mean((1, 3)), v.var((1, 3), unbiased=False).sqrt()
        # fp32 sums shifted by a value of the block: a few 2^-24 of the values, which are up to some 5 standard deviations
        assert float(((m.double() - mu) / sd).abs().max()) <= 4e-6 and float((r.double() * (sd ** 2 + 1e-6).sqrt() - 1).abs().max()) <= 4e-6


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("cin2", [0, 96])
@pytest.mark.parametrize("sizes,c,h,w", [((1, 2, 3), 128, 131, 145), ((1, 2, 5, 7), 256, 101, 99)])
def test_a_sample_keeps_its_bits_where_the_batch_chooses_the_height(dtype, sizes, c, cin2, h, w):
    _same_bits_in_batches(dtype, sizes, c, cin2, c, h, w, 32)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("cin2", [0, 96])
def test_a_sample_keeps_its_bits_where_the_batch_chooses_the_height_and_the_ring_is_whole(dtype, cin2):
    _same_bits_in_batches(dtype, (1, 3, 4), 256, cin2, 128, 131, 145, 32)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("n,cin,cout,h,w", PAIR)
def test_a_workspace_for_the_triples_of_eight_rows(dtype, n, cin, cout, h, w):
    """What such a layer asked for before it could take six rows still gets its moments from the convolution, one triple per group and 8 x 16 tile, and the same y."""
    g, groups = torch.Generator(device="cuda"), 32
    g.manual_seed(synth.SEED_BASE + 64)

    def draw(*shape):
        return torch.randn(shape, generator=g, device="cuda")
    x, res, bias = draw(n, h, w, cin).to(G.TORCH[dtype]), draw(n, h, w, cout).to(G.TORCH[dtype]), draw(cout)
    mean, rstd, gamma, beta = draw(n * 32), draw(n * 32).abs() + 0.5, draw(cin), draw(cin)
    packed = G.pack((draw(cout, cin, 3, 3) / (9 * cin) ** 0.5).bfloat16().float().cpu().numpy(), dtype)
    tiles_y, tiles_x = -(-h // 8), -(-w // 16)
    full, few = wmdec.conv_stats_workspace_bytes(G.ENUM[dtype], G.ENUM[dtype], n, h, w, cin, cout, groups), 12 * groups * n * tiles_y * tiles_x
    assert few < full

    def run(size):
        y, ws = torch.empty((n, h, w, cout), dtype=G.TORCH[dtype], device="cuda"), torch.full((size + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        m, r = torch.empty(n * groups, device="cuda"), torch.empty(n * groups, device="cuda")
        wmdec.gn_silu_conv3x3_stats(x, mean, rstd, gamma, beta, 32, True, packed, bias, res, y, groups, 1e-6, m, r, ws[:size])
        assert bool((ws[size:] == 0xA5).all())
        return y, m, r, ws[:size]
    y, m, r, _ = run(full)
    for size in (few, full - 12):
        y2, m2, r2, ws = run(size)
        v = y2.double().view(n, h * w, groups, cout // groups)
        mu, sd = v.mean((1, 3)).flatten(), v.var((1, 3), unbiased=False).sqrt().flatten()
        # fp32 sums shifted by a value of the block: a few 2^-24 of the values, which are up to some 5 standard deviations
        assert torch.equal(y, y2) and float(((m2.double() - mu) / sd).abs().max()) <= 4e-6 and float((r2.double() * (sd ** 2 + 1e-6).sqrt() - 1).abs().max()) <= 4e-6
        count = ws[:few].view(torch.float32).view(n, groups, tiles_y, tiles_x, 3)[..., 0]
        rows, cols = ([min(t, e - t * i) for i in range(k)] for t, e, k in ((8, h, tiles_y), (16, w, tiles_x)))
        assert torch.equal(count, torch.outer(torch.tensor(rows), torch.tensor(cols)).mul(cout // groups).float().cuda().expand_as(count))
    with pytest.raises(wmdec.WmdecError) as e:
        run(few - 12)
    assert e.value.status == wmdec.ERR_WORKSPACE


# every way in which the last runs of rows end, and groups of every size
@pytest.mark.parametrize("groups", [4, 8, 16, 32, 64, 128])
def test_moments_where_the_batch_chooses_the_height(groups):
    for h in range(128 + groups.bit_length() % 3, 152, 3):
        _same_bits_in_batches("f16", (1, 3), 128, 0, 128, h, 129, groups)


# rows of more than 4096 triples, which a lane of the merge takes in several rounds (a tile of 8 x 16 pixels and 64 channels leaves four, here of few
# pixels each): one full round, 4100, remainders, and a row 100 rounds long.  The first triples lie 100 standard deviations of the others from them.
@pytest.mark.parametrize("h,w", [(8192, 3), (8193, 3), (10800, 2), (21600, 1), (819200, 1)])
@pytest.mark.parametrize("band", [0, 2, 4096])
def test_moments_of_long_rows_of_triples(h, w, band):
    g = torch.Generator(device="cuda")
    g.manual_seed(synth.SEED_BASE + 65)
    c, groups = 64, 32
    x = torch.randn((1, h, w, c), generator=g, device="cuda")
    x[:, :band] += 100
    x = x.half()
    wt = torch.zeros((c, c, 3, 3))
    wt[torch.arange(c), torch.arange(c), 1, 1] = 1
    packed, y = G.pack(wt.numpy(), "f16"), torch.empty_like(x)
    mean, rstd = torch.empty(groups, device="cuda"), torch.empty(groups, device="cuda")
    size = wmdec.conv_stats_workspace_bytes(wmdec.F16, wmdec.F16, 1, h, w, c, c, groups)
    assert size == 12 * groups * 4 * -(-h // 8)
    ws = torch.full((size + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    wmdec.gn_silu_conv3x3_stats(x, None, None, None, None, 1, False, packed, None, None, y, groups, 1e-6, mean, rstd, ws[:size])
    assert torch.equal(x, y) and bool((ws[size:] == 0xA5).all())
    v = y.double().view(h * w, groups, c // groups)
    m, sd = v.mean((0, 2)), v.var((0, 2), unbiased=False).sqrt()
    # fp32 sums shifted by a value of the block, merged about their mean: a few 2^-24 of the values
    err = float(((mean.double() - m) / sd).abs().max()), float((rstd.double() * (sd ** 2 + 1e-6).sqrt() - 1).abs().max())
    assert err[0] <= 4e-6 and err[1] <= 4e-6, err
