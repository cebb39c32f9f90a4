"""The 3x3 convolution that splits its contraction over wavefronts (small 16-bit images, fp32): every tile shape at ragged
edges against the fp64 oracle, the folded shortcut, the moments it emits, and a sample's bits at any batch."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2602_00608_amd import synth, wmdec
from tests import gpu_util as G

pytestmark = pytest.mark.gpu
EPS = 1e-6


def case(seed, dtype, n, cin, cout, h, w, cin2=0):
    r = np.random.default_rng(synth.SEED_BASE + seed)
    sixteen = dtype != "f32"
    c = {"x": G.stored(r.standard_normal((n, cin, h, w)) * 1.3 + 0.2, dtype), "res": G.stored(r.standard_normal((n, cout, h, w)), dtype),
         "gamma": (1 + 0.2 * r.standard_normal(cin)).astype(np.float32), "beta": (0.2 * r.standard_normal(cin)).astype(np.float32)}
    c["w"], c["b"] = synth.conv_params(r, cout, cin, 3, sixteen)
    if cin2:
        c["x2"] = G.stored(r.standard_normal((n, cin2, h, w)), dtype)
        c["w2"], c["b2"] = synth.conv_params(r, cout, cin2, 1, sixteen)
    return c


# tile edges: one pixel, one row, one past a 4x8 / 4x16 block; the tiles 32x32, 32x64, 64x64, 64x128; the largest
# image of the split path (2^20 outputs) and the first past it
@pytest.mark.parametrize("dtype,n,cin,cout,h,w,norm", [
    ("f16", 1, 64, 64, 1, 1, True), ("bf16", 1, 512, 512, 5, 9, True), ("f16", 1, 512, 512, 17, 23, True),
    ("bf16", 2, 128, 512, 17, 23, True), ("f16", 1, 512, 512, 34, 46, True), ("f16", 3, 256, 256, 33, 47, True),
    ("bf16", 2, 64, 64, 61, 129, True), ("f16", 1, 192, 128, 64, 128, False), ("f16", 1, 64, 128, 64, 129, True),
    ("f32", 1, 32, 32, 1, 1, True), ("f32", 2, 64, 64, 9, 17, True), ("f32", 1, 128, 64, 33, 31, True),
    ("f32", 1, 96, 32, 4, 8, False), ("f32", 1, 320, 96, 13, 11, True)])
def test_split_convolution(dtype, n, cin, cout, h, w, norm):
    c = case(40, dtype, n, cin, cout, h, w)
    xd = G.dev_nhwc(c["x"], dtype)
    mean, rstd = G.gn_stats(xd, 32, EPS) if norm else (None, None)
    y, check = G.canaried((n, h, w, cout), torch.float32)
    wmdec.gn_silu_conv3x3(xd, mean, rstd, G.dev_f32(c["gamma"]), G.dev_f32(c["beta"]), 32, True, G.pack(c["w"], dtype),
                          G.dev_f32(c["b"]), G.dev_nhwc(c["res"], dtype), y)
    torch.cuda.synchronize()
    check()
    a = ref.group_norm(c["x"], 32, EPS, c["gamma"], c["beta"], apply_silu=True) if norm else c["x"]
    err = ref.rel_err(G.host_nchw(y), ref.conv2d(a, c["w"], c["b"]) + c["res"])
    # fp32: 9 * cin products of fp32 rounding error 2^-24 each, plus the activation's few ulp; 16 bits: the operand
    # rounding alone (2^-9 / 2^-12 of a product) at the workload's bar, halved for the unrounded output
    assert err <= (1e-5 if dtype == "f32" else G.TOL[dtype] / 2), err


# any group count: the table of per-channel means behind the scale/shift table is read as 16-byte vectors
@pytest.mark.parametrize("dtype,cin,cout,groups,h,w", [("f32", 64, 32, 1, 5, 9), ("f32", 96, 64, 3, 9, 7), ("f32", 32, 32, 1, 1, 1), ("f16", 64, 64, 1, 5, 9),
                                                       ("bf16", 192, 64, 3, 9, 7)])
def test_split_convolution_with_an_odd_number_of_groups(dtype, cin, cout, groups, h, w):
    c = case(43, dtype, 2, cin, cout, h, w)
    xd = G.dev_nhwc(c["x"], dtype)
    mean, rstd = G.gn_stats(xd, groups, EPS)
    y, check = G.canaried((2, h, w, cout), torch.float32)
    wmdec.gn_silu_conv3x3(xd, mean, rstd, G.dev_f32(c["gamma"]), G.dev_f32(c["beta"]), groups, True, G.pack(c["w"], dtype), G.dev_f32(c["b"]), None, y)
    torch.cuda.synchronize()
    check()
    err = ref.rel_err(G.host_nchw(y), ref.conv2d(ref.group_norm(c["x"], groups, EPS, c["gamma"], c["beta"], apply_silu=True), c["w"], c["b"]))
    assert err <= (1e-5 if dtype == "f32" else G.TOL[dtype] / 2), err


@pytest.mark.parametrize("dtype,n,cin,cin2,cout,h,w", [("f16", 1, 128, 256, 128, 17, 23), ("bf16", 2, 256, 512, 256, 30, 44), ("f32", 1, 64, 128, 64, 9, 11),
                                                       ("f32", 1, 96, 32, 32, 7, 9)])
def test_split_convolution_with_folded_shortcut(dtype, n, cin, cin2, cout, h, w):
    c = case(41, dtype, n, cin, cout, h, w, cin2)
    xd = G.dev_nhwc(c["x"], dtype)
    mean, rstd = G.gn_stats(xd, 32, EPS)
    y, check = G.canaried((n, h, w, cout), torch.float32)
    wmdec.gn_silu_conv3x3_shortcut(xd, mean, rstd, G.dev_f32(c["gamma"]), G.dev_f32(c["beta"]), 32, True, G.pack(c["w"], dtype), G.dev_f32(c["b"]),
                                   G.dev_nhwc(c["x2"], dtype), G.pack(c["w2"], dtype), G.dev_f32(c["b2"]), y)
    torch.cuda.synchronize()
    check()
    want = ref.conv2d(ref.group_norm(c["x"], 32, EPS, c["gamma"], c["beta"], apply_silu=True), c["w"], c["b"]) + ref.conv2d(c["x2"], c["w2"], c["b2"])
    err = ref.rel_err(G.host_nchw(y), want)
    assert err <= (1e-5 if dtype == "f32" else G.TOL[dtype] / 2), err


# the last three: images past the split path whose 64 x 128 and 128 x 128 tiles the batch decides between (one sample of
# them fills at most one round); heights that end in either half of the larger tile
@pytest.mark.parametrize("cin,cout,groups,h,w", [(512, 512, 32, 17, 23), (128, 256, 32, 33, 40), (64, 128, 32, 61, 47), (64, 64, 32, 9, 31), (64, 64, 64, 5, 3),
                                                 (64, 256, 8, 13, 17), (128, 512, 32, 57, 45), (96, 256, 32, 68, 92), (64, 384, 48, 36, 90)])
def test_moments_and_bits_do_not_depend_on_the_batch(cin, cout, groups, h, w):
    """Batches of 1, 2 and 7 take different tiles (of either 16-bit kernel): the sample they share, and its statistics, must agree bit for bit, and
    the statistics with the oracle's of the stored tensor.  A workspace that only holds the widest tiles' fewer triples gives
    the same bits of y, and statistics by a pass over it."""
    c = case(42, "f16", 7, cin, cout, h, w)
    xd, wt, b = G.dev_nhwc(c["x"], "f16"), G.pack(c["w"], "f16"), G.dev_f32(c["b"])
    gamma, beta = G.dev_f32(c["gamma"]), G.dev_f32(c["beta"])
    mean, rstd = G.gn_stats(xd, 32, EPS)
    got = []
    for n in (1, 2, 7):
        y = torch.empty((n, h, w, cout), dtype=torch.float16, device="cuda")
        ws = torch.full((wmdec.conv_stats_workspace_bytes(wmdec.F16, wmdec.F16, n, h, w, cin, cout, groups),), 0xA5, dtype=torch.uint8, device="cuda")
        mo, ro = torch.empty(n * groups, device="cuda"), torch.empty(n * groups, device="cuda")
        x, m, r = xd[7 - n:].contiguous(), mean[(7 - n) * 32:].contiguous(), rstd[(7 - n) * 32:].contiguous()
        wmdec.gn_silu_conv3x3_stats(x, m, r, gamma, beta, 32, True, wt, b, None, y, groups, EPS, mo, ro, ws)
        torch.cuda.synchronize()
        wm, wr = ref.gn_stats(G.host_nchw(y), groups, EPS)
        assert np.max(np.abs(mo.cpu().numpy() - wm.ravel()) * wr.ravel()) < 2e-5 and np.max(np.abs(ro.cpu().numpy() / wr.ravel() - 1.0)) < 2e-5
        got.append((y[-1].clone(), mo[-groups:].clone(), ro[-groups:].clone()))
        wide = 12 * groups * n * (-(-h // 8)) * (-(-w // 16)) * (1 if cout % 128 == 0 else 4)
        if wide < ws.numel():
            y2 = torch.empty_like(y)
            small = torch.full((wide + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
            wmdec.gn_silu_conv3x3_stats(x, m, r, gamma, beta, 32, True, wt, b, None, y2, groups, EPS, mo, ro, small[:wide])
            torch.cuda.synchronize()
            assert torch.equal(y2, y) and bool((small[wide:] == 0x5A).all())
            assert np.max(np.abs(mo.cpu().numpy() - wm.ravel()) * wr.ravel()) < 2e-5 and np.max(np.abs(ro.cpu().numpy() / wr.ravel() - 1.0)) < 2e-5
            with pytest.raises(wmdec.WmdecError):
                wmdec.gn_silu_conv3x3_stats(x, m, r, gamma, beta, 32, True, wt, b, None, y2, groups, EPS, mo, ro, small[:wide - 12])
    for g in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got[0], g))


# batches past one round take 128 x 128 tiles: one 16-channel group per partial sum (cin 64), an odd number of them (a partial sum
# ends inside a chunk), even ones; a single column, ragged blocks in both directions; outputs as stored and in fp32.  The
# last: images of one row, which stay with the small tiles
@pytest.mark.parametrize("dtype,n,cin,cout,h,w,norm,res,y32", [
    ("f16", 48, 64, 512, 7, 1, True, False, False), ("bf16", 24, 64, 128, 35, 21, True, True, False), ("f16", 16, 192, 512, 13, 30, True, False, True),
    ("f16", 8, 512, 512, 17, 23, True, True, False), ("bf16", 4, 512, 512, 34, 46, True, False, False), ("f16", 15, 320, 256, 36, 7, True, True, True),
    ("bf16", 70, 128, 256, 5, 9, False, False, False), ("f16", 100, 128, 256, 1, 9, False, False, False)])
def test_large_batches_keep_the_bits_of_a_sample(dtype, n, cin, cout, h, w, norm, res, y32):
    c = case(44, dtype, n, cin, cout, h, w)
    xd, wt, b, rd = G.dev_nhwc(c["x"], dtype), G.pack(c["w"], dtype), G.dev_f32(c["b"]), G.dev_nhwc(c["res"], dtype) if res else None
    gamma, beta, yt = G.dev_f32(c["gamma"]), G.dev_f32(c["beta"]), torch.float32 if y32 else G.TORCH[dtype]
    mean, rstd = G.gn_stats(xd, 32, EPS) if norm else (None, None)

    def run(lo, k):
        y, check = G.canaried((k, h, w, cout), yt)
        mo, ro = torch.empty(k * 32, device="cuda"), torch.empty(k * 32, device="cuda")
        ws = torch.empty(wmdec.conv_stats_workspace_bytes(G.ENUM[dtype], wmdec.F32 if y32 else G.ENUM[dtype], k, h, w, cin, cout, 32), dtype=torch.uint8, device="cuda")
        part = lambda t, m=1: None if t is None else t[lo * m:(lo + k) * m].contiguous()
        wmdec.gn_silu_conv3x3_stats(part(xd), part(mean, 32), part(rstd, 32), gamma, beta, 32, True, wt, b, part(rd), y, 32, EPS, mo, ro, ws)
        torch.cuda.synchronize()
        check()
        return y, mo, ro

    y, mo, ro = run(0, n)
    for i in (0, n // 2, n - 1):
        y1, m1, r1 = run(i, 1)
        assert torch.equal(y[i:i + 1], y1) and torch.equal(mo[32 * i:32 * i + 32], m1) and torch.equal(ro[32 * i:32 * i + 32], r1), i
    a = ref.group_norm(c["x"][-1:], 32, EPS, c["gamma"], c["beta"], apply_silu=True) if norm else c["x"][-1:]
    want = ref.conv2d(a, c["w"], c["b"]) + (c["res"][-1:] if res else 0)
    assert ref.rel_err(G.host_nchw(y[-1:]), want) <= G.TOL[dtype]
