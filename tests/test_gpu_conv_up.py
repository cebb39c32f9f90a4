"""Nearest-2x upsample + 3x3 convolution from nine products per input pixel: tile edges of the 7 x 15 pixel tiles against
the fp64 oracle, at one type's rounding of the result (the products and sums carry no rounding of their own)."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2602_00608_amd import synth, wmdec
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("n,cin,cout,h,w", [(1, 32, 64, 1, 1), (2, 64, 64, 7, 15), (1, 96, 128, 8, 16), (1, 64, 192, 6, 14), (3, 128, 64, 15, 31),
                                            (1, 512, 512, 17, 23)])
def test_upsampling_convolution_tile_edges(dtype, n, cin, cout, h, w):
    r = np.random.default_rng(synth.SEED_BASE + 50)
    x = G.stored(r.standard_normal((n, cin, h, w)), dtype)
    wt, b = synth.conv_params(r, cout, cin, 3, True)
    want = ref.upconv(x, wt, b)
    for ydtype in ("f32", dtype):
        y, check = G.canaried((n, 2 * h, 2 * w, cout), G.TORCH[ydtype])
        wmdec.upsample2x_conv3x3(G.dev_nhwc(x, dtype), G.pack_upconv(wt, dtype), G.dev_f32(b), y)
        torch.cuda.synchronize()
        check()
        got = G.host_nchw(y)
        # operands are exact: fp32 sums of 9 * cin products (worst case 9 * 512 * 2^-24 of the magnitudes, typically 1e-6);
        # a stored output adds half an ulp of its own size
        tol = np.full_like(want, 2e-5 * float(np.sqrt(np.mean(want ** 2))))
        if ydtype != "f32":
            tol += np.abs(want) * (2.0 ** -8 if dtype == "bf16" else 2.0 ** -11)
        assert np.all(np.abs(got - want) <= tol), float(np.max(np.abs(got - want) - tol))


# either side of the rule that splits the contraction of small images: 48 and 160 workgroups of 64 channels (the label of a
# decoder's upsampling step, of the same shape, says which kernel a shape takes), and channels that cannot be split in two
@pytest.mark.parametrize("cin,cout,h,w,split", [(64, 64, 20, 33, True), (96, 64, 20, 33, False), (512, 512, 17, 23, True), (512, 512, 28, 61, False)])
def test_upsampling_convolution_sample_bits_do_not_depend_on_the_batch(cin, cout, h, w, split):
    if cin == 512:
        cfg = wmdec.decoder_default_config()
        cfg.latent_h, cfg.latent_w = h, w
        dec = wmdec.Decoder(cfg)
        assert [k for k, _, _ in dec.step_info() if k.startswith("conv_up")][0] == "conv_up_kernel<wmdec::f16_t, 2, %d, false>" % (1 if split else 2)
        dec.close()
    r = np.random.default_rng(synth.SEED_BASE + 51)
    x = G.dev_nhwc(G.stored(r.standard_normal((3, cin, h, w)), "f16"), "f16")
    wt, b = synth.conv_params(r, cout, cin, 3, True)
    wp, bd = G.pack_upconv(wt, "f16"), G.dev_f32(b)
    y3, y1 = (torch.empty((n, 2 * h, 2 * w, cout), dtype=torch.float16, device="cuda") for n in (3, 1))
    wmdec.upsample2x_conv3x3(x, wp, bd, y3)
    wmdec.upsample2x_conv3x3(x[1:2].contiguous(), wp, bd, y1)
    assert torch.equal(y3[1:2], y1)


# 128 workgroups of 64 channels, the last count whose contraction is split in two, and the next size up; one chunk of 32 channels a half
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("w", [60, 61])
def test_upsampling_convolution_either_side_of_the_split(dtype, w):
    test_upsampling_convolution_tile_edges(dtype, 1, 64, 512, 28, w)
