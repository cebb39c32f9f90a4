"""GPU parity: every per-op entry point of the C ABI against the fp64 oracle on
the same seeded inputs, element by element.  Sizes span several tiles and a
ragged tail; degenerate shapes included."""
import math

import numpy as np
import pytest
import torch

from oracle import ref
from paper_2602_00608_amd import synth, wmdec
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def rng(seed):
    return np.random.default_rng(synth.SEED_BASE + seed)


# ------------------------------------------------------------------ a1: GroupNorm statistics
@pytest.mark.parametrize("dtype,n,c,h,w,groups", [
    ("f32", 1, 64, 32, 32, 32),      # workload 1 shape
    ("f32", 2, 12, 5, 7, 4),         # general path, tiny
    ("bf16", 1, 128, 37, 53, 32),    # 4 channels per group: one 16-byte vector spans two groups
    ("bf16", 2, 256, 24, 36, 32),
    ("f16", 1, 512, 15, 23, 32),     # 16 channels per group: a group spans two vectors
    ("f16", 3, 24, 9, 11, 3),        # general path, 16 bit
    ("f32", 1, 32, 1, 1, 32),        # one element per group: variance 0
    ("bf16", 1, 128, 480, 720, 32),  # workload 3 size
    ("f16", 70, 64, 3, 5, 32),       # more samples than one 256-byte block of the workspace's head stands for
    ("f16", 2, 1024, 4, 6, 32),      # widest tensor of the vector layout (one pixel per sweep)
    ("bf16", 1, 2048, 3, 3, 32),     # wider than that: general path
])
def test_gn_stats(dtype, n, c, h, w, groups):
    x = G.stored(rng(1).standard_normal((n, c, h, w)) * 1.7 + 0.6, dtype)
    eps = 1e-6
    mean, rstd = G.gn_stats(G.dev_nhwc(x, dtype), groups, eps)
    wm, wr = ref.gn_stats(x, groups, eps)
    gm, gr = mean.cpu().numpy().reshape(n, groups), rstd.cpu().numpy().reshape(n, groups)
    sd = 1.0 / wr
    assert np.max(np.abs(gm - wm) / sd) < 2e-5, np.max(np.abs(gm - wm) / sd)
    assert np.max(np.abs(gr / wr - 1.0)) < 2e-5, np.max(np.abs(gr / wr - 1.0))


# images of up to 4096 pixels with whole groups in 64 bytes of a pixel: one pixel, fewer than the 16 wavefronts' 256 rows, a remainder behind four sweeps of
# them, both sides of the line, group sizes from one channel to 64 bytes; and a group of 128 bytes and groups of one 16-bit channel in one slab, which the other kernel takes
@pytest.mark.parametrize("dtype,n,c,h,w,groups", [("f32", 1, 16, 1, 1, 16), ("bf16", 3, 32, 15, 17, 1), ("f16", 2, 64, 16, 16, 32), ("f16", 1, 64, 1, 257, 64), ("f32", 2, 32, 41, 25, 8),
                                                  ("bf16", 1, 256, 25, 41, 64), ("f32", 1, 1024, 3, 7, 64), ("f16", 2, 128, 64, 64, 32), ("f16", 2, 128, 1, 4097, 32), ("bf16", 1, 512, 23, 17, 8),
                                                  ("f16", 2, 64, 32, 64, 64), ("bf16", 2, 64, 1, 2049, 64), ("f16", 1, 256, 27, 31, 256)])
def test_gn_stats_of_small_images(dtype, n, c, h, w, groups):
    """A sample's result is its own bit for bit; errors: a thread sums at most 16 pixels, then some ten levels of merges, each rounded once: 26 * 2^-24 = 1.6e-6."""
    x = G.stored(rng(8).standard_normal((n, c, h, w)) * 1.7 + 0.6, dtype)
    xd = G.dev_nhwc(x, dtype)
    mean, rstd = G.gn_stats(xd, groups, 1e-6)
    wm, wr = ref.gn_stats(x, groups, 1e-6)
    assert np.max(np.abs(mean.cpu().numpy() - wm.ravel()) * wr.ravel()) < 1.6e-6 * max(1.0, np.max(np.abs(wm) * wr))
    assert np.max(np.abs(rstd.cpu().numpy() / wr.ravel() - 1.0)) < 1.6e-6
    m1, r1 = G.gn_stats(xd[n - 1:].contiguous(), groups, 1e-6)
    assert torch.equal(mean[(n - 1) * groups:], m1) and torch.equal(rstd[(n - 1) * groups:], r1)


def test_gn_stats_large_offset_no_cancellation():
    # mean >> std: a naive E[x^2]-E[x]^2 in fp32 would lose the variance
    x = (rng(2).standard_normal((1, 64, 40, 40)) * 0.01 + 100.0).astype(np.float32)
    mean, rstd = G.gn_stats(G.dev_nhwc(x, "f32"), 32, 1e-6)
    wm, wr = ref.gn_stats(x, 32, 1e-6)
    assert np.max(np.abs(rstd.cpu().numpy() / wr.ravel() - 1.0)) < 1e-3
    assert np.max(np.abs(mean.cpu().numpy() - wm.ravel())) < 1e-4


@pytest.mark.parametrize("c,h,w", [(256, 120, 180), (64, 32, 32), (512, 7, 9)])
@pytest.mark.parametrize("rows,offset", [(1, 10.0), (1, 100.0), (4, 100.0)])
def test_gn_stats_with_a_first_band_off_the_rest(rows, offset, c, h, w):
    """A letterboxed image: the first slab's mean lies `offset` standard deviations from the others'.  Two passes over the
    triples round each of some 13 sequential additions (8 per lane, 5 levels across lanes) once: 13 * 2^-24 = 8e-7 at worst
    for the variance, as the sums inside a slab do; one pass about the first triple's mean was off by 1e-5."""
    x = rng(5).standard_normal((1, c, h, w)).astype(np.float32)
    x[:, :, :rows] += offset
    mean, rstd = G.gn_stats(G.dev_nhwc(x, "f32"), 32, 1e-6)
    wm, wr = ref.gn_stats(x, 32, 1e-6)
    assert np.max(np.abs(rstd.cpu().numpy() / wr.ravel() - 1.0)) < 1e-6
    assert np.max(np.abs(mean.cpu().numpy() - wm.ravel()) * wr.ravel()) < 5e-7


@pytest.mark.parametrize("c,h,w", [(64, 32, 32), (512, 10, 12), (8, 3, 5)])
def test_gn_stats_with_an_outlier_first_pixel(c, h, w):
    """The first pixel of the tensor 1000 standard deviations off.  Only one thread's sums are shifted by it, a share 1/ppi
    of the slab (ppi = 1024 * 4 / c pixels a sweep): its own cancellation is 1000^2 * 2^-24 = 6e-2 of a variance of 1, that
    of the group gains 1000^2 / pixels, so 6e-8 * pixels / ppi relative, and the sums' own 8e-7."""
    x = rng(7).standard_normal((1, c, h, w)).astype(np.float32)
    x[:, :, 0, 0] += 1000.0
    groups = min(32, c)
    mean, rstd = G.gn_stats(G.dev_nhwc(x, "f32"), groups, 1e-6)
    wm, wr = ref.gn_stats(x, groups, 1e-6)
    assert np.max(np.abs(rstd.cpu().numpy() / wr.ravel() - 1.0)) < 8e-7 + 6e-8 * max(h * w * c / 4096, 1)
    assert np.max(np.abs(mean.cpu().numpy() - wm.ravel()) * wr.ravel()) < 5e-7


@pytest.mark.parametrize("dtype,c,h,w,mean,std", [("f16", 512, 54, 24, 37.0, 0.01), ("f16", 256, 61, 47, 100.0, 0.01), ("f16", 64, 33, 9, 1000.0, 1.0), ("bf16", 512, 54, 24, 1000.0, 1.0),
                                                  ("bf16", 128, 47, 24, 100.0, 0.1), ("f32", 512, 17, 23, 100.0, 0.01), ("f32", 64, 32, 32, -1000.0, 0.3)])
def test_gn_stats_of_few_pixels_a_lane_far_from_zero(dtype, c, h, w, mean, std):
    """Means of five or six pixels, rounded at the values' exponent, would stand in the squares about the group's mean (the quantised values of 16 bits make the same error again and
    again): what counts are differences, as exact as where the mean is zero (1.6e-6 there, see test_gn_stats_of_small_images), and the mean is rounded once."""
    x = G.stored(rng(9).standard_normal((1, c, h, w)) * std + mean, dtype)
    m, r = G.gn_stats(G.dev_nhwc(x, dtype), 32, 0.0)
    v = x.astype(np.float64).reshape(32, -1)
    wm, wr = v.mean(1), 1.0 / v.std(1)
    assert np.max(np.abs(r.cpu().numpy() / wr - 1.0)) < 1.6e-6
    assert np.max(np.abs(m.cpu().numpy() - wm) - np.abs(wm) * 2.0 ** -23) * np.max(wr) < 1.6e-6


# Small images (one workgroup's columns), one workgroup, and several with a merge; groups of one to 64 bytes of a pixel.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("c,groups,h,w", [(64, 32, 32, 32), (64, 64, 64, 64), (128, 8, 1, 1), (64, 4, 5, 7), (8, 4, 3, 5), (64, 8, 120, 180)])
def test_gn_stats_of_values_near_the_end_of_the_range(dtype, c, groups, h, w):
    """Constant 3e38 in every second group: a sum of a few such values is infinite, their mean is not, and nothing deviates from it."""
    x = np.full((2, c, h, w), 3e38, np.float32)
    x[:, (np.arange(c) * groups // c) % 2 == 1] = -2.0
    x = G.stored(x, dtype)
    mean, rstd = G.gn_stats(G.dev_nhwc(x, dtype), groups, 1e-6)
    want = x[:, ::c // groups, 0, 0].ravel()
    assert np.max(np.abs(mean.cpu().numpy() / want - 1.0)) < 1e-6 and np.max(np.abs(rstd.cpu().numpy() - 1e3)) < 1e-2


@pytest.mark.parametrize("h,w", [(120, 180), (16, 16)])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("last", [False, True])
def test_gn_stats_of_a_group_that_is_not_finite(h, w, bad, last):
    """One infinity or NaN: the group's rstd must not look like one of finite data; the other groups keep their bits."""
    x = rng(6).standard_normal((1, 64, h, w)).astype(np.float32)
    good = G.gn_stats(G.dev_nhwc(x, "f32"), 32, 1e-6)
    x[0, 6, -1 if last else 0, 0] = bad      # group 3
    mean, rstd = G.gn_stats(G.dev_nhwc(x, "f32"), 32, 1e-6)
    assert not torch.isfinite(mean[3]) and not bool(rstd[3] > 0)
    keep = [g for g in range(32) if g != 3]
    assert torch.equal(mean[keep], good[0][keep]) and torch.equal(rstd[keep], good[1][keep])


def test_gn_stats_deterministic():
    x = G.dev_nhwc(G.stored(rng(3).standard_normal((2, 128, 61, 47)), "bf16"), "bf16")
    a = G.gn_stats(x, 32, 1e-6)
    b = G.gn_stats(x, 32, 1e-6)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


def test_gn_stats_workspace_reuse_across_tensors():
    """One workspace, never cleared, serves many calls on different tensors and shapes of the same batch size, back to back on one
    stream: every call must see only its own partial moments and leave the head of the workspace alone."""
    n, groups, eps = 2, 32, 1e-6
    shapes = [(128, 61, 47), (256, 30, 44), (512, 9, 13), (128, 120, 90), (64, 5, 7)]
    ws = torch.full((max(wmdec.gn_stats_workspace_bytes(n, h, w, c, groups) for c, h, w in shapes),), 0xA5, dtype=torch.uint8, device="cuda")
    xs, outs = [], []
    for rep in range(4):
        for i, (c, h, w) in enumerate(shapes):
            x = G.stored(rng(100 + 10 * rep + i).standard_normal((n, c, h, w)) * (1.0 + i) - rep, "f16")
            xd = G.dev_nhwc(x, "f16")
            mean = torch.empty(n * groups, dtype=torch.float32, device="cuda")
            rstd = torch.empty(n * groups, dtype=torch.float32, device="cuda")
            wmdec.gn_stats(xd, groups, eps, mean, rstd, ws)
            xs.append(x); outs.append((mean, rstd, xd))
    torch.cuda.synchronize()
    for x, (mean, rstd, _) in zip(xs, outs):
        wm, wr = ref.gn_stats(x, groups, eps)
        assert np.max(np.abs(mean.cpu().numpy() - wm.ravel()) * wr.ravel()) < 2e-5
        assert np.max(np.abs(rstd.cpu().numpy() / wr.ravel() - 1.0)) < 2e-5
    assert bool((ws[:256] == 0xA5).all())


def test_gn_stats_gives_the_same_bits_in_every_round():
    """Passes in one launch and in two, whose merge reads what the first one's workgroups left: many shapes and batches
    are run round-robin on one workspace, 40 rounds, and every result must equal the first round's bit for bit (and the
    oracle's to fp32 accuracy)."""
    groups, eps = 32, 1e-6
    shapes = [(1, 128, 480, 720), (2, 256, 120, 180), (4, 512, 60, 90), (3, 128, 61, 47), (1, 1024, 9, 13), (4, 64, 33, 5)]
    xs = [G.dev_nhwc(G.stored(rng(300 + i).standard_normal((n, c, h, w)) * (0.5 + i) + 0.1 * i, "f16"), "f16")
          for i, (n, c, h, w) in enumerate(shapes)]
    ws = torch.full((max(wmdec.gn_stats_workspace_bytes(n, h, w, c, groups) for n, c, h, w in shapes),), 0xA5, dtype=torch.uint8, device="cuda")
    first = None
    for rnd in range(40):
        outs = []
        for x in xs:
            n = x.shape[0]
            mean = torch.empty(n * groups, dtype=torch.float32, device="cuda")
            rstd = torch.empty(n * groups, dtype=torch.float32, device="cuda")
            wmdec.gn_stats(x, groups, eps, mean, rstd, ws)
            outs.append((mean, rstd))
        torch.cuda.synchronize()
        if first is None:
            first = outs
            for x, (mean, rstd) in zip(xs[1:], outs[1:]):     # the first shape is checked against the oracle elsewhere
                wm, wr = ref.gn_stats(G.host_nchw(x), groups, eps)
                assert np.max(np.abs(mean.cpu().numpy() - wm.ravel()) * wr.ravel()) < 2e-5
                assert np.max(np.abs(rstd.cpu().numpy() / wr.ravel() - 1.0)) < 2e-5
        else:
            for i, ((m0, r0), (m1, r1)) in enumerate(zip(first, outs)):
                assert torch.equal(m0, m1) and torch.equal(r0, r1), (rnd, shapes[i])


# ------------------------------------------------------------------ a3': nearest-2x upsample (bit exact)
@pytest.mark.parametrize("dtype,n,c,h,w", [("bf16", 1, 256, 120, 180), ("f32", 2, 3, 5, 7), ("f16", 1, 8, 1, 1),
                                           ("bf16", 2, 20, 6, 3), ("bf16", 1, 5, 4, 9)])
def test_upsample2x_nearest_bit_exact(dtype, n, c, h, w):
    x = G.stored(rng(4).standard_normal((n, c, h, w)), dtype)
    xd = G.dev_nhwc(x, dtype)
    y, check = G.canaried((n, 2 * h, 2 * w, c), G.TORCH[dtype])
    wmdec.upsample2x_nearest(xd, y)
    check()
    want = ref.upsample2x(x)      # exact in fp64
    got = G.host_nchw(y)
    assert np.array_equal(got, want)


# ------------------------------------------------------------------ layout conversion
@pytest.mark.parametrize("sd,dd", [("f32", "f32"), ("f32", "bf16"), ("bf16", "f32"), ("f16", "f16")])
def test_layout_roundtrip(sd, dd):
    x = G.stored(G.stored(rng(5).standard_normal((2, 7, 33, 45)), sd), dd)   # representable in both
    src = torch.from_numpy(x).to(G.TORCH[sd]).cuda()
    nhwc = torch.empty((2, 33, 45, 7), dtype=G.TORCH[dd], device="cuda")
    wmdec.nchw_to_nhwc(src, nhwc)
    assert np.array_equal(G.host_nchw(nhwc), x.astype(np.float64))
    back = torch.empty((2, 7, 33, 45), dtype=G.TORCH[sd], device="cuda")
    wmdec.nhwc_to_nchw(nhwc, back)
    assert torch.equal(back, src)


# ------------------------------------------------------------------ a2/a4: fused norm -> SiLU -> conv3x3 (+bias, +residual)
def run_conv(x, dtype, w, b, res, norm, silu, groups, ydtype, k=3, eps=1e-6, gamma=None, beta=None):
    """x, res: float32 NCHW arrays of storable values; returns (gpu NCHW float64, oracle NCHW float64)."""
    n, cin, h, wd = x.shape
    cout = w.shape[0]
    xd = G.dev_nhwc(x, dtype)
    wp = G.pack(w, dtype)
    wq = G.stored(w, dtype) if dtype != "f32" else w
    y, check = G.canaried((n, h, wd, cout), G.TORCH[ydtype])
    mean = rstd = gd = bd = None
    if norm:
        mean, rstd = G.gn_stats(xd, groups, eps)
        gd, bd = G.dev_f32(gamma), G.dev_f32(beta)
    fn = wmdec.gn_silu_conv3x3 if k == 3 else wmdec.gn_conv1x1
    fn(xd, mean, rstd, gd, bd, groups, silu, wp, None if b is None else G.dev_f32(b),
       None if res is None else G.dev_nhwc(res, dtype), y)
    torch.cuda.synchronize()
    check()
    u = x.astype(np.float64)
    if norm:
        u = ref.group_norm(u, groups, eps, gamma, beta, apply_silu=silu)
    want = ref.conv2d(u, wq, b)
    if res is not None:
        want = want + res
    return G.host_nchw(y), want


CONV_CASES = [
    # dtype, ydtype, n, cin, cout, h, w, norm, silu, bias, residual
    ("f32", "f32", 1, 64, 64, 32, 32, True, True, True, True),       # workload 1 conv
    ("f32", "f32", 2, 4, 3, 5, 7, False, False, True, False),        # tiny, odd channels
    ("f32", "f32", 1, 12, 20, 9, 10, True, True, False, True),
    ("f32", "f32", 1, 8, 8, 1, 1, True, False, True, False),         # one pixel
    ("bf16", "f32", 1, 128, 128, 40, 56, True, True, True, True),
    ("bf16", "bf16", 2, 64, 96, 19, 21, True, True, True, True),
    ("f16", "f16", 1, 256, 128, 17, 33, True, True, True, False),
    ("f16", "f32", 1, 128, 3, 24, 31, True, True, True, False),      # conv_out shape class
    ("bf16", "f32", 1, 4, 64, 12, 18, False, False, True, False),    # conv_in shape class
    ("f16", "f16", 2, 4, 512, 9, 70, False, False, True, False),     # conv_in: two channel blocks, three row segments
    ("f16", "f16", 1, 7, 100, 5, 33, False, False, False, False),    # few input channels, ragged channel block
    ("bf16", "f32", 1, 512, 512, 15, 23, True, True, True, True),
    ("f16", "f32", 1, 32, 32, 64, 3, True, True, True, True),        # narrow image
]


@pytest.mark.parametrize("dtype,ydtype,n,cin,cout,h,w,norm,silu,bias,residual", CONV_CASES)
def test_gn_silu_conv3x3(dtype, ydtype, n, cin, cout, h, w, norm, silu, bias, residual):
    r = rng(10)
    x = G.stored(r.standard_normal((n, cin, h, w)) * 1.3 + 0.2, dtype)
    wt, b = synth.conv_params(r, cout, cin, 3, dtype != "f32")
    res = G.stored(r.standard_normal((n, cout, h, w)), dtype) if residual else None
    groups = 32 if cin % 32 == 0 else 4
    gamma = (1 + 0.2 * r.standard_normal(cin)).astype(np.float32)
    beta = (0.2 * r.standard_normal(cin)).astype(np.float32)
    got, want = run_conv(x, dtype, wt, b if bias else None, res, norm, silu, groups, ydtype, gamma=gamma, beta=beta)
    err = ref.rel_err(got, want)
    tol = G.TOL[dtype]
    assert err <= tol, err
    if dtype != "f32" and ydtype == "f32":
        assert err <= tol / 2, err   # fp32 output of 16-bit operands: well inside the bar


# every output channel one tap of one input channel: an exact copy of the input, displaced by the tap, whatever order the
# products are summed in.  Ragged sizes of the tiles whose lanes hold rows apart: 8 rows of a wavefront, four of them, two
# blocks of four in a larger batch, 64 channels a wavefront; one, two and three chunks of input channels.
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("n,cin,cout,h,w", [(1, 64, 128, 101, 115), (1, 32, 128, 97, 129), (1, 96, 128, 27, 45), (13, 96, 128, 27, 45),
                                            (1, 32, 128, 1, 1), (1, 32, 128, 253, 262), (1, 96, 256, 253, 262), (1, 96, 256, 100, 203)])
def test_conv_of_single_taps_is_an_exact_displacement(dtype, n, cin, cout, h, w):
    x = torch.from_numpy(rng(21).standard_normal((n, h, w, cin)).astype(np.float32)).to(G.TORCH[dtype])
    wt = np.zeros((cout, cin, 3, 3), np.float32)
    want = torch.zeros((n, h, w, cout), dtype=x.dtype)
    padded = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    for co in range(cout):
        ci, ky, kx = 7 * co % cin, co % 9 // 3, co % 3
        wt[co, ci, ky, kx] = 1.0
        want[..., co] = padded[:, ky:ky + h, kx:kx + w, ci]
    y = torch.empty(want.shape, dtype=x.dtype, device="cuda")
    wmdec.gn_silu_conv3x3(x.cuda(), None, None, None, None, 32, False, G.pack(wt, dtype), None, None, y)
    assert torch.equal(y.cpu(), want)


# A bias forty times the sums, fp32 output: the bias meets finished sums.  Bound on the rms error over half a million outputs or
# more: that one addition rounds by ulp / sqrt(12) of the result in the mean, and the steps of the sums (16 products each) by at
# most 2^-23, truncation included, of partial sums of rms 1, independently of each other.  Sums that start from the bias round
# every step by ulp / sqrt(12) of the result: over five times as much at the least count of steps here with a tile of that kind (16).
@pytest.mark.parametrize("k,n,cin,cout,h,w", [(3, 1, 64, 64, 130, 131), (3, 1, 64, 128, 97, 99), (3, 1, 32, 256, 256, 257), (3, 1, 64, 512, 64, 61),
                                              (3, 2, 64, 512, 64, 61), (3, 1, 256, 512, 17, 23), (3, 16, 64, 128, 40, 41), (3, 1, 32, 256, 100, 203),
                                              (1, 1, 512, 64, 90, 91), (1, 1, 512, 128, 64, 65), (1, 1, 256, 128, 363, 363), (1, 1, 288, 192, 64, 65)])
def test_conv_adds_a_large_bias_to_finished_sums(k, n, cin, cout, h, w):
    r = rng(22)
    x = torch.from_numpy(r.standard_normal((n, h, w, cin)).astype(np.float32)).to(torch.float16)
    wt = G.stored(r.standard_normal((cout, cin, k, k)) / np.sqrt(k * k * cin), "f16")
    b = (r.choice([-1.0, 1.0], cout) * r.uniform(40, 60, cout)).astype(np.float32)
    y = torch.empty((n, h, w, cout), dtype=torch.float32, device="cuda")
    fn = wmdec.gn_silu_conv3x3 if k == 3 else wmdec.gn_conv1x1
    fn(x.cuda(), None, None, None, None, 32, False, G.pack(wt, "f16"), G.dev_f32(b), None, y)
    padded, taps = x.double(), torch.from_numpy(wt).double().permute(2, 3, 1, 0)
    if k == 3:
        padded = torch.nn.functional.pad(padded, (0, 0, 1, 1, 1, 1))
    want = torch.zeros((n, h, w, cout), dtype=torch.float64) + torch.from_numpy(b).double()
    for ky in range(k):
        for kx in range(k):
            want += padded[:, ky:ky + h, kx:kx + w].reshape(-1, cin).matmul(taps[ky, kx]).view(n, h, w, cout)
    ulp = np.spacing(np.abs(want.numpy()).astype(np.float32)).astype(np.float64)
    bound = float(np.sqrt(np.mean(ulp ** 2) / 12 + k * k * cin / 16 * 2.0 ** -46))
    err = float((y.cpu().double() - want).square().mean().sqrt())
    assert err <= bound, (err, bound)


# moments of a convolution's own output from its epilogue: one case per tile shape of the matrix-core kernel
@pytest.mark.parametrize("dtype,ydtype,n,cin,cout,h,w,residual", [
    ("f16", "f16", 1, 128, 128, 40, 56, True),      # 128 x 128 tile, wavefronts 2x2
    ("bf16", "bf16", 2, 256, 128, 24, 36, True),    # two samples
    ("f16", "f16", 1, 64, 64, 17, 33, False),       # 128 x 64 tile, ragged
    ("f16", "f32", 1, 128, 256, 19, 21, False),     # fp32 output: nothing is rounded
    ("bf16", "bf16", 1, 64, 512, 9, 13, True),      # 16 channels per group: a group spans two channel octets
    ("f16", "f16", 1, 256, 256, 240, 360, True),    # 128 x 128 tile with one weight fragment per four MFMAs
    ("f16", "f16", 1, 128, 128, 480, 720, True),    # 256 x 128 tile (full-resolution layer)
    ("bf16", "bf16", 1, 128, 128, 480, 720, False),
    ("f16", "f16", 1, 4, 512, 60, 90, False),       # conv_in: the kernel for few input channels, no normalisation of x
    ("bf16", "bf16", 2, 4, 64, 13, 37, False),      # two channels per group, ragged segment, two samples
    ("f16", "f16", 1, 8, 2048, 5, 50, False),       # 64 channels per group: a group is a whole wavefront
])
def test_conv_epilogue_statistics(dtype, ydtype, n, cin, cout, h, w, residual):
    """wmdec_gn_silu_conv3x3_stats: mean / rstd of the tensor the kernel stored, per (sample, output group), must
    equal the oracle's statistics of exactly that stored tensor, and the streaming pass over it, to fp32 accuracy."""
    r = rng(14)
    groups, eps = 32, 1e-6
    x = G.stored(r.standard_normal((n, cin, h, w)) * 1.3 + 0.2, dtype)
    wt, b = synth.conv_params(r, cout, cin, 3, True)
    b = (b + 0.5).astype(np.float32)                 # a mean well away from zero
    xd = G.dev_nhwc(x, dtype)
    res = G.dev_nhwc(G.stored(r.standard_normal((n, cout, h, w)), dtype), dtype) if residual else None
    norm = cin % groups == 0
    mean, rstd = G.gn_stats(xd, groups, eps) if norm else (None, None)
    gamma = G.dev_f32((1 + 0.2 * r.standard_normal(cin)).astype(np.float32)) if norm else None
    beta = G.dev_f32((0.2 * r.standard_normal(cin)).astype(np.float32)) if norm else None
    y = torch.empty((n, h, w, cout), dtype=G.TORCH[ydtype], device="cuda")
    nbytes = wmdec.conv_stats_workspace_bytes(G.ENUM[dtype], G.ENUM[ydtype], n, h, w, cin, cout, groups)
    assert nbytes > 0
    ws = torch.full((nbytes,), 0xA5, dtype=torch.uint8, device="cuda")     # needs no initialisation
    mo = torch.empty(n * groups, dtype=torch.float32, device="cuda")
    ro = torch.empty(n * groups, dtype=torch.float32, device="cuda")
    wmdec.gn_silu_conv3x3_stats(xd, mean, rstd, gamma, beta, groups, norm, G.pack(wt, dtype), G.dev_f32(b), res, y,
                                groups, eps, mo, ro, ws)
    torch.cuda.synchronize()
    wm, wr = ref.gn_stats(G.host_nchw(y), groups, eps)
    em = float(np.max(np.abs(mo.cpu().numpy() - wm.ravel()) * wr.ravel()))
    er = float(np.max(np.abs(ro.cpu().numpy() / wr.ravel() - 1.0)))
    assert em < 2e-5 and er < 2e-5, (em, er)
    m2, r2 = G.gn_stats(y, groups, eps)
    assert float(torch.max(torch.abs(mo - m2) * r2)) < 2e-5 and float(torch.max(torch.abs(ro / r2 - 1.0))) < 2e-5
    # the tensor itself is the one the plain entry point writes
    y2 = torch.empty_like(y)
    wmdec.gn_silu_conv3x3(xd, mean, rstd, gamma, beta, groups, norm, G.pack(wt, dtype), G.dev_f32(b), res, y2)
    assert torch.equal(y, y2)


# ... and one per width of a group (1 to 32 channels) on every form of the moments: one triple per 8x16 tile and wavefront
# row (128x64, 128x128 and 128x256 tiles), one per four rows (the small and the large tile of the pair), ragged in both directions
@pytest.mark.parametrize("dtype,ydtype,cout,h,w", [("f16", "f16", 64, 13, 37), ("bf16", "f32", 64, 9, 17), ("f16", "f16", 128, 101, 115),
                                                   ("bf16", "bf16", 128, 27, 45), ("f16", "f32", 128, 5, 19), ("bf16", "bf16", 256, 253, 262)])
@pytest.mark.parametrize("cpg", [1, 2, 4, 8, 16, 32])
def test_conv_epilogue_statistics_group_widths(dtype, ydtype, cout, h, w, cpg):
    """Means of 40 standard deviations, and outliers of 300 on single pixels: sums about the lane's first value and
    merges about the mean lose at most (300 / 8)^2 half ulps of a variance to a shift that is an outlier, 1e-4."""
    r = rng(16 + cpg)
    n, cin, groups, eps = 2, 32, cout // cpg, 1e-6
    xd = G.dev_nhwc(G.stored(r.standard_normal((n, cin, h, w)), dtype), dtype)
    wt, b = synth.conv_params(r, cout, cin, 3, True)
    b = (b + 40.0 * np.where(np.arange(cout) // cpg % 2 == 0, 1, -1)).astype(np.float32)
    rf = r.standard_normal((n, cout, h, w))
    rf[:, :, 0, 0] += 300.0
    rf[:, :, h - 1, w - 1] -= 300.0
    res = G.dev_nhwc(G.stored(rf, dtype), dtype)
    y = torch.empty((n, h, w, cout), dtype=G.TORCH[ydtype], device="cuda")
    ws = torch.full((wmdec.conv_stats_workspace_bytes(G.ENUM[dtype], G.ENUM[ydtype], n, h, w, cin, cout, groups),), 0xFF, dtype=torch.uint8, device="cuda")
    mo, ro = torch.empty(n * groups, device="cuda"), torch.empty(n * groups, device="cuda")
    wmdec.gn_silu_conv3x3_stats(xd, None, None, None, None, 32, False, G.pack(wt, dtype), G.dev_f32(b), res, y, groups, eps, mo, ro, ws)
    v = y.double().view(n, h * w, groups, cpg).permute(0, 2, 1, 3).reshape(n * groups, -1)
    wm, wr = v.mean(1), 1 / torch.sqrt(v.var(1, unbiased=False) + eps)
    em, er = float(((mo - wm).abs() * wr).max()), float((ro / wr - 1).abs().max())
    assert em < 2e-5 and er < 1e-4, (em, er)


def test_conv_epilogue_statistics_unsupported_shapes_are_refused():
    x = torch.zeros((1, 8, 8, 32), dtype=torch.float32, device="cuda")
    assert wmdec.conv_stats_workspace_bytes(wmdec.F32, wmdec.F32, 1, 8, 8, 32, 64, 32) == 0
    assert wmdec.conv_stats_workspace_bytes(wmdec.F16, wmdec.F16, 1, 8, 8, 32, 96, 32) == 0     # 3 channels per group
    y = torch.zeros((1, 8, 8, 64), dtype=torch.float32, device="cuda")
    ws = torch.zeros(1 << 16, dtype=torch.uint8, device="cuda")
    mo = torch.zeros(32, dtype=torch.float32, device="cuda")
    with pytest.raises(wmdec.WmdecError) as e:
        wmdec.gn_silu_conv3x3_stats(x, None, None, None, None, 32, False, ws, None, None, y, 32, 1e-6, mo, mo.clone(), ws)
    assert e.value.status == wmdec.ERR_UNSUPPORTED


# second convolution of a channel-changing ResBlock with the 1x1 shortcut folded into its contraction
@pytest.mark.parametrize("dtype,ydtype,n,cin,cin2,cout,h,w", [
    ("f16", "f32", 1, 256, 512, 256, 24, 36),       # 128 x 128 tile, wavefronts 2x2
    ("bf16", "bf16", 2, 128, 256, 128, 40, 56),
    ("f16", "f16", 1, 64, 96, 64, 17, 33),          # 128 x 64 tile, ragged, cin2 not a multiple of 64
    ("f16", "f16", 1, 32, 64, 32, 20, 28),          # cout % 64 != 0: two launches of the general kernel
    ("f32", "f32", 1, 24, 12, 40, 7, 9),            # fp32 path
    ("f16", "f16", 1, 256, 512, 256, 240, 360),     # full size: tile with one weight fragment per four MFMAs
    ("f16", "f32", 1, 128, 256, 128, 480, 720),     # full size: 256 x 128 tile
    ("bf16", "f32", 1, 128, 256, 128, 480, 720),
])
def test_gn_silu_conv3x3_shortcut(dtype, ydtype, n, cin, cin2, cout, h, w):
    r = rng(15)
    sixteen = dtype != "f32"
    x = G.stored(r.standard_normal((n, cin, h, w)) * 1.3 + 0.2, dtype)
    x2 = G.stored(r.standard_normal((n, cin2, h, w)), dtype)
    wt, b = synth.conv_params(r, cout, cin, 3, sixteen)
    w2, b2 = synth.conv_params(r, cout, cin2, 1, sixteen)
    groups = 32 if cin % 32 == 0 else 4
    gamma = (1 + 0.2 * r.standard_normal(cin)).astype(np.float32)
    beta = (0.2 * r.standard_normal(cin)).astype(np.float32)
    xd, x2d = G.dev_nhwc(x, dtype), G.dev_nhwc(x2, dtype)
    mean, rstd = G.gn_stats(xd, groups, 1e-6)
    y, check = G.canaried((n, h, w, cout), G.TORCH[ydtype])
    wmdec.gn_silu_conv3x3_shortcut(xd, mean, rstd, G.dev_f32(gamma), G.dev_f32(beta), groups, True, G.pack(wt, dtype),
                                   G.dev_f32(b), x2d, G.pack(w2, dtype), G.dev_f32(b2), y)
    torch.cuda.synchronize()
    check()
    want = ref.conv2d(ref.group_norm(x, groups, 1e-6, gamma, beta, apply_silu=True), wt, b) + ref.conv2d(x2, w2, b2)
    err = ref.rel_err(G.host_nchw(y), want)
    assert err <= G.TOL[dtype] / (2 if sixteen and ydtype == "f32" else 1), err


def test_conv_padding_is_applied_after_activation():
    # constant input, beta chosen so that SiLU(GN(x)) != 0: border outputs must see zeros, not SiLU(beta)
    x = np.full((1, 32, 6, 6), 3.0, np.float32)
    w = np.zeros((32, 32, 3, 3), np.float32)
    w[:, :, :, :] = 1.0 / 32
    gamma, beta = np.ones(32, np.float32), np.full(32, 2.0, np.float32)
    got, want = run_conv(x, "f32", w, None, None, True, True, 32, "f32", gamma=gamma, beta=beta)
    s = 2.0 / (1 + math.exp(-2.0))
    assert abs(want[0, 0, 0, 0] - 4 * s) < 1e-12 and abs(want[0, 0, 2, 2] - 9 * s) < 1e-12
    assert ref.rel_err(got, want) < 1e-5


@pytest.mark.parametrize("dtype,ydtype,n,cin,cout,h,w,norm,residual", [
    ("f32", "f32", 1, 24, 40, 7, 9, True, True),
    ("bf16", "f32", 1, 512, 256, 24, 36, False, False),      # ResBlock shortcut shape class
    ("f16", "f16", 2, 512, 1536, 5, 7, True, False),         # fused q,k,v projection shape class
    ("bf16", "bf16", 1, 256, 128, 31, 17, False, True),
])
def test_gn_conv1x1(dtype, ydtype, n, cin, cout, h, w, norm, residual):
    r = rng(11)
    x = G.stored(r.standard_normal((n, cin, h, w)), dtype)
    wt, b = synth.conv_params(r, cout, cin, 1, dtype != "f32")
    res = G.stored(r.standard_normal((n, cout, h, w)), dtype) if residual else None
    groups = 32 if cin % 32 == 0 else 4
    gamma = (1 + 0.2 * r.standard_normal(cin)).astype(np.float32)
    beta = (0.2 * r.standard_normal(cin)).astype(np.float32)
    got, want = run_conv(x, dtype, wt, b, res, norm, False, groups, ydtype, k=1, gamma=gamma, beta=beta)
    assert ref.rel_err(got, want) <= G.TOL[dtype]


# ------------------------------------------------------------------ a3: upsample-conv
@pytest.mark.parametrize("dtype,ydtype,n,cin,cout,h,w", [
    ("f32", "f32", 1, 6, 10, 5, 7),
    ("bf16", "f32", 1, 256, 256, 20, 28),
    ("f16", "f16", 2, 128, 64, 9, 13),
    ("bf16", "bf16", 1, 64, 64, 1, 1),
])
def test_upsample2x_conv3x3(dtype, ydtype, n, cin, cout, h, w):
    r = rng(12)
    x = G.stored(r.standard_normal((n, cin, h, w)), dtype)
    wt, b = synth.conv_params(r, cout, cin, 3, dtype != "f32")
    y, check = G.canaried((n, 2 * h, 2 * w, cout), G.TORCH[ydtype])
    wmdec.upsample2x_conv3x3(G.dev_nhwc(x, dtype), G.pack_upconv(wt, dtype), G.dev_f32(b), y)
    torch.cuda.synchronize()
    check()
    want = ref.upconv(x, G.stored(wt, dtype) if dtype != "f32" else wt, b)
    assert ref.rel_err(G.host_nchw(y), want) <= G.TOL[dtype] / (2 if ydtype == "f32" else 1)


# 32 channels: general kernel; 64: the upsampling kernel on the matrix cores
@pytest.mark.parametrize("ch,dtype", [(32, "bf16"), (64, "bf16"), (64, "f16")])
def test_upconv_gather_index_map_bit_exact(ch, dtype):
    """One-hot kernels turn the fused upsample-conv into a pure gather: the output must equal the
    shifted, zero-padded upsampled input bit for bit, for all nine taps."""
    r = rng(13)
    x = G.stored(r.standard_normal((1, ch, 7, 10)), dtype)
    up = np.pad(ref.upsample2x(x), ((0, 0), (0, 0), (1, 1), (1, 1)))
    xd = G.dev_nhwc(x, dtype)
    for ky in range(3):
        for kx in range(3):
            w = np.zeros((ch, ch, 3, 3), np.float32)
            for c in range(ch):
                w[c, c, ky, kx] = 1.0
            y = torch.empty((1, 14, 20, ch), dtype=G.TORCH[dtype], device="cuda")
            wmdec.upsample2x_conv3x3(xd, G.pack_upconv(w, dtype), None, y)
            assert np.array_equal(G.host_nchw(y), up[:, :, ky:ky + 14, kx:kx + 20]), (ky, kx)


# ------------------------------------------------------------------ a5: attention block
def run_attention(dtype, n, h, w, seed, sharpen=None):
    c, groups, eps = 512, 32, 1e-6
    r = rng(seed)
    x = G.stored(r.standard_normal((n, c, h, w)), dtype)
    p = {"norm.gamma": (1 + 0.2 * r.standard_normal(c)).astype(np.float32),
         "norm.beta": (0.2 * r.standard_normal(c)).astype(np.float32)}
    for nm in ("q", "k", "v", "proj"):
        p[nm + ".w"], p[nm + ".b"] = synth.conv_params(r, c, c, 1, True)
    # f16: sharpen the softmax (logit std 4 instead of 1) so that it is far from uniform.  bf16 keeps
    # logit std 1: q and k stored with 8 significant bits put an error of ~0.2% x logit std on every
    # logit, which a peaked softmax amplifies beyond the 2e-2 bar (a property of the format, not the kernel).
    if sharpen is None:
        sharpen = 2.0 if dtype == "f16" else 1.0
    p["q.w"] = synth.bf16_round(p["q.w"] * sharpen)
    p["k.w"] = synth.bf16_round(p["k.w"] * sharpen)
    xd = G.dev_nhwc(x, dtype)
    mean, rstd = G.gn_stats(xd, groups, eps)
    wqkv = np.concatenate([p["q.w"], p["k.w"], p["v.w"]], axis=0)
    bqkv = np.concatenate([p["q.b"], p["k.b"], p["v.b"]])
    ws = torch.empty(wmdec.attention_workspace_bytes(n, h, w, c), dtype=torch.uint8, device="cuda")
    y, check = G.canaried((n, h, w, c), G.TORCH[dtype])
    wmdec.attention(xd, mean, rstd, G.dev_f32(p["norm.gamma"]), G.dev_f32(p["norm.beta"]), groups,
                    G.pack(wqkv, dtype), G.dev_f32(bqkv), G.pack(p["proj.w"], dtype), G.dev_f32(p["proj.b"]), y, ws)
    torch.cuda.synchronize()
    check()
    want = ref.attention_block(x, p, groups, eps)
    run_attention.last_params = p
    return G.host_nchw(y), want, x


def branch_tolerance(dtype, want, x):
    """Bound for the attention branch y - x.  The kernel's own error is held to 3x the bar; on top of it the output
    y is stored in `dtype`, whose rounding error (half an ulp: 2^-9 |y| in bf16, 2^-12 |y| in f16) lands entirely
    in the branch, which is small against y when many tokens are averaged."""
    ulp_half = 2.0 ** -9 if dtype == "bf16" else 2.0 ** -12
    rms_branch = math.sqrt(float(np.mean((want - x) ** 2)))
    return 3 * G.TOL[dtype] + ulp_half * float(np.max(np.abs(want))) / rms_branch


# 5x7, 1x1: one ragged query block; 9x8, 16x20: several query blocks with a ragged last one and two key splits;
# 13x37 = 481 tokens: 8 query blocks (the last holds one query), 16 key blocks over 8 splits
@pytest.mark.parametrize("dtype,n,h,w", [("f16", 1, 5, 7), ("bf16", 2, 9, 8), ("f16", 1, 1, 1), ("bf16", 1, 16, 20),
                                         ("f16", 2, 13, 37)])
def test_attention_small(dtype, n, h, w):
    got, want, x = run_attention(dtype, n, h, w, 20)
    assert ref.rel_err(got, want) <= G.TOL[dtype]
    # the attention branch itself (output minus residual input) must agree too, not just x + small
    assert ref.rel_err(got - x, want - x) <= branch_tolerance(dtype, want, x)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_attention_full_size_5400_tokens(dtype):
    got, want, x = run_attention(dtype, 1, 60, 90, 21)
    assert ref.rel_err(got, want) <= G.TOL[dtype]
    assert ref.rel_err(got - x, want - x) <= branch_tolerance(dtype, want, x)


def test_attention_bf16_sharp_softmax_with_the_same_storage_points():
    """bf16 with a 4x sharper softmax (logit std 4).  q and k stored with 8 significant bits shift every logit by
    ~0.16 % of its size, and a peaked softmax turns that into percents of the output: a property of the format,
    which the plain oracle (exact q, k) does not share.  So here the oracle is given the same storage points: its
    q, k, v are rounded to bf16 where the kernel stores them, everything else stays fp64.  Against that reference
    the kernel itself must meet the bar, branch included."""
    dtype, n, h, w = "bf16", 1, 16, 20
    got, _, x = run_attention(dtype, n, h, w, 22, sharpen=2.0)
    p = run_attention.last_params
    c, groups, eps = 512, 32, 1e-6
    hn = ref.group_norm(x, groups, eps, p["norm.gamma"], p["norm.beta"], apply_silu=False)
    hn = G.stored(hn, dtype)                       # MFMA operand of the projection
    q, k, v = (G.stored(ref.conv2d(hn, p[m + ".w"], p[m + ".b"]), dtype).astype(np.float64) for m in ("q", "k", "v"))
    tok = lambda a: np.ascontiguousarray(a[0].reshape(c, h * w).T)
    o = ref.attention_core(tok(q), tok(k), tok(v), 1.0 / math.sqrt(c)).T.reshape(1, c, h, w)
    want = x + ref.conv2d(o, p["proj.w"], p["proj.b"])
    assert ref.rel_err(got, want) <= G.TOL[dtype]
    assert ref.rel_err(got - x, want - x) <= branch_tolerance(dtype, want, x)


# 32-token tiles, 64-token projection workgroups and 128-query blocks: one token short of, at and past their edges
@pytest.mark.parametrize("dtype,n,h,w", [("bf16", 1, 1, 31), ("f16", 2, 4, 8), ("f16", 1, 3, 11), ("bf16", 1, 8, 8), ("f16", 2, 5, 13),
                                         ("bf16", 1, 1, 127), ("f16", 1, 8, 16), ("bf16", 2, 3, 43), ("f16", 1, 7, 37)])
def test_attention_tile_edges(dtype, n, h, w):
    got, want, x = run_attention(dtype, n, h, w, 23)
    assert ref.rel_err(got, want) <= G.TOL[dtype]
    assert ref.rel_err(got - x, want - x) <= branch_tolerance(dtype, want, x)


@pytest.mark.parametrize("dtype,n,h,w", [("f16", 1, 113, 146), ("bf16", 2, 1, 16411)])
def test_attention_long_sequence_in_one_range_of_keys(dtype, n, h, w):
    """Sequences whose blocks of queries fill the chip by themselves: one range holds all keys and the core writes o itself.  64
    tokens of the last sample, its first and last among them, against 64 bits."""
    c, t, r = 512, h * w, rng(25)
    x = torch.from_numpy(r.standard_normal((n, h, w, c)).astype(np.float32)).to(G.TORCH[dtype])
    wts = {m: G.stored(r.standard_normal((c, c)) / np.sqrt(c), dtype) for m in "qkvo"}
    b = {m: (0.05 * r.standard_normal(c)).astype(np.float32) for m in "qkvo"}
    gamma, beta = (1 + 0.2 * r.standard_normal(c)).astype(np.float32), (0.2 * r.standard_normal(c)).astype(np.float32)
    mean, rstd = (0.1 * r.standard_normal(n * 32)).astype(np.float32), (1 + 0.1 * r.standard_normal(n * 32)).astype(np.float32)
    ws = torch.empty(wmdec.attention_workspace_bytes(n, h, w, c), dtype=torch.uint8, device="cuda")
    y, check = G.canaried((n, h, w, c), G.TORCH[dtype])
    four = lambda a: np.ascontiguousarray(a[:, :, None, None])
    wmdec.attention(x.cuda(), G.dev_f32(mean), G.dev_f32(rstd), G.dev_f32(gamma), G.dev_f32(beta), 32,
                    G.pack(four(np.concatenate([wts["q"], wts["k"], wts["v"]])), dtype), G.dev_f32(np.concatenate([b["q"], b["k"], b["v"]])),
                    G.pack(four(wts["o"]), dtype), G.dev_f32(b["o"]), y, ws)
    torch.cuda.synchronize()
    check()
    d = lambda a: torch.from_numpy(np.asarray(a)).double()
    xs = x[-1].reshape(t, c).double()
    hn = (xs - d(mean[-32:]).repeat_interleave(16)) * d(rstd[-32:]).repeat_interleave(16) * d(gamma) + d(beta)
    at = torch.from_numpy(np.concatenate([[0, 31, 32, t - 2, t - 1], r.integers(0, t, 59)]))
    proj = lambda m, v: v @ d(wts[m]).T + d(b[m])
    o = torch.softmax(proj("q", hn[at]) @ proj("k", hn).T / math.sqrt(c), 1) @ proj("v", hn)
    want, got = (xs[at] + proj("o", o)).numpy(), y[-1].reshape(t, c).cpu()[at].double().numpy()
    assert ref.rel_err(got, want) <= G.TOL[dtype]
    assert ref.rel_err(got - xs[at].numpy(), want - xs[at].numpy()) <= branch_tolerance(dtype, want, xs[at].numpy())


def test_attention_reference_moves_inside_a_key_range():
    """Logits of standard deviation 9 (13 in powers of two) over eight ranges of 256 keys: the maximum of a range lies about
    0.8 standard deviations above that of its first 32 keys, so that most queries cross the slack of 2^8 behind the
    first block and the output accumulators are rescaled."""
    got, want, x = run_attention("f16", 1, 32, 64, 24, sharpen=3.0)
    assert ref.rel_err(got, want) <= G.TOL["f16"]
    assert ref.rel_err(got - x, want - x) <= branch_tolerance("f16", want, x)


# ------------------------------------------------------------------ horizontally fused AdaLN projections (DiT)
# d_model = d_cond = 1920 stands for the paper's 30-head transformer (64 per head; the paper gives no widths)
@pytest.mark.parametrize("cdtype,wdtype,batch,d_cond,d_model,silu", [
    ("f32", "bf16", 1, 1920, 1920, True),      # one frame's conditioning vector
    ("f32", "bf16", 4, 1920, 1920, True),      # a batch of four frames
    ("bf16", "bf16", 8, 1920, 1920, True),
    ("f16", "f16", 3, 520, 77, False),         # ragged: d_cond not a multiple of a wavefront's 512, rows of 8 and 32
    ("f32", "f32", 2, 12, 5, True),
    ("f32", "bf16", 16, 1024, 40, True),       # the largest batch one launch takes
])
def test_adaln_fused_projection(cdtype, wdtype, batch, d_cond, d_model, silu):
    """One launch on the row-concatenated [W_shift; W_scale; W_gate] against the oracle's three separate products."""
    sixteen = wdtype != "f32"
    p = synth.adaln_params(synth.weight_seed(20), d_model, d_cond, sixteen_bit=sixteen)
    if wdtype == "f16":
        p = {k: (G.stored(v, "f16") if k.endswith(".w") else v) for k, v in p.items()}
    c = G.stored(rng(30).standard_normal((batch, d_cond)) * 1.5, cdtype)
    w_fused = np.vstack([p["shift.w"], p["scale.w"], p["gate.w"]])
    b_fused = np.concatenate([p["shift.b"], p["scale.b"], p["gate.b"]])
    cd = torch.from_numpy(c).to(G.TORCH[cdtype]).cuda()
    wd = torch.from_numpy(w_fused).to(G.TORCH[wdtype]).cuda()
    out, check = G.canaried((batch, 3 * d_model), torch.float32)
    wmdec.adaln_fused_projection(cd, wd, G.dev_f32(b_fused), out, apply_silu=silu)
    torch.cuda.synchronize()
    check()
    shift, scale, gate = ref.adaln_modulation(c, p, apply_silu=silu)
    got = out.cpu().numpy().astype(np.float64)
    for k, want in enumerate((shift, scale, gate)):
        err = ref.rel_err(got[:, k * d_model:(k + 1) * d_model], want)
        assert err <= 1e-4, (k, err)          # fp32 products and sums of exactly stored operands


def test_adaln_fused_projection_limits():
    assert wmdec.adaln_max_batch(1920) == 8 and wmdec.adaln_max_batch(512) == 16
    c = torch.zeros((9, 1920), dtype=torch.float32, device="cuda")
    w = torch.zeros((24, 1920), dtype=torch.bfloat16, device="cuda")
    out = torch.zeros((9, 24), dtype=torch.float32, device="cuda")
    with pytest.raises(wmdec.WmdecError) as e:
        wmdec.adaln_fused_projection(c, w, None, out)
    assert e.value.status == wmdec.ERR_UNSUPPORTED


# ------------------------------------------------------------------ measurement helper: the plain copy of known traffic
@pytest.mark.parametrize("nbytes", [16, 16 * 255, (1 << 20) + 16 * 7, 256 << 20])
def test_measure_copy_bit_exact(nbytes):
    """wmdec_measure_copy moves exactly the bytes it is given (counter passes are scaled by its traffic) and nothing
    next to them; sizes and pointers that are not multiples of 16, and overlapping ranges, are refused."""
    g = torch.Generator(device="cuda").manual_seed(nbytes % 9973)
    src = torch.randint(0, 256, (nbytes,), dtype=torch.uint8, device="cuda", generator=g)
    big = torch.full((nbytes + 512,), 0x5A, dtype=torch.uint8, device="cuda")
    dst = big[256:256 + nbytes]
    wmdec.measure_copy(src, dst)
    torch.cuda.synchronize()
    assert torch.equal(dst, src)
    assert bool((big[:256] == 0x5A).all()) and bool((big[256 + nbytes:] == 0x5A).all())
    if nbytes >= 64:
        for bad_src, bad_dst in ((src[:24], dst[:24]), (src[8:40], dst[:32]), (big[:64], big[32:96])):
            with pytest.raises(wmdec.WmdecError) as e:
                wmdec.measure_copy(bad_src, bad_dst)
            assert e.value.status == wmdec.ERR_INVALID_ARG


# ------------------------------------------------------------------ binding: the stream a call is enqueued on
def test_calls_are_enqueued_on_the_current_stream():
    """The raw handle the binding asks for is that of torch's current stream, inside and outside a stream context."""
    side = torch.cuda.Stream()
    outer = torch.cuda.current_stream().cuda_stream
    assert wmdec._stream() == outer
    with torch.cuda.stream(side):
        assert wmdec._stream() == side.cuda_stream != outer
    assert wmdec._stream() == outer
