"""The shapes that the GPU tests give for a tile are launched on it: a rule that sends one elsewhere fails here (no GPU needed)."""
import os
import shutil
import subprocess

import pytest

from paper_2602_00608_amd import wmdec
from tests import test_gpu_conv_rows, test_gpu_ops

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# tiles of the 3x3 kernel on 16x16x32 MFMAs: rows, 128-channel blocks, mode (1: moments per four rows), ring
NARROW4, ROWS4_RING, ROWS4, RING, NARROW, WIDE = "4, 1, 1, 18", "8, 1, 1, 18", "8, 1, 1, 0", "8, 1, 0, 18", "8, 1, 0, 0", "8, 2, 0, 0"


@pytest.fixture(scope="module")
def tiles(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not on PATH")
    wmdec.lib()   # (built)
    exe = str(tmp_path_factory.mktemp("tiles") / "tile_names")
    pkg = os.path.join(ROOT, "paper_2602_00608_amd")
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-std=c++17", "-I" + os.path.join(pkg, "csrc"), "-I" + os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "tile_names.cpp"),
                    "-L" + pkg, "-lwmdec", "-Wl,-rpath," + pkg, "-o", exe], check=True)

    def ask(shapes, residual=False):   # (ksize, n, cin, cout, h, w, fp32 output) -> tile, or the kernel's name where it is another one
        out = subprocess.run([exe] + [",".join(str(int(v)) for v in s + (residual,)) for s in shapes], check=True, capture_output=True, text=True).stdout.split("\n")[:-1]
        names = []
        for label in out:
            p = label[label.find("<") + 1:-1].split(", ")
            names.append(", ".join([p[2], p[6], p[10], p[11]]) if label.startswith("conv_mfma_kernel<") and p[3:6] == ["16", "1", "4"] and p[10] != "2" else label)
        return names
    return ask


def _cases(test, names):
    mark = [m for m in test.pytestmark if m.name == "parametrize" and m.args[0] == names]
    assert len(mark) == 1
    return mark[0].args[1]


def test_edges_of_every_tile(tiles):
    cases = _cases(test_gpu_conv_rows.test_tile_edges, "n,cin,cout,h,w")
    want = [NARROW4, ROWS4_RING, ROWS4, RING, NARROW, NARROW, NARROW, WIDE, WIDE, WIDE]
    for f32 in (False, True):
        assert tiles([(3,) + c + (f32,) for c in cases]) == want
        assert tiles([(3,) + c + (f32,) for c in cases], residual=True) == want[:7] + [RING, RING, WIDE]   # (few channels: 128 beside a residual)


def test_widths_that_the_batch_chooses(tiles):
    assert tiles([(3, n, 64, 256, 100, 100, False) for n in (1, 2, 3, 5)]) == [RING, WIDE, NARROW, WIDE]
    assert tiles([(3, n, 128, 256, 100, 100, False) for n in (1, 2, 3, 5)], residual=True) == [RING, WIDE, NARROW, WIDE]


def test_exact_displacements(tiles):
    got = tiles([(3,) + c + (False,) for c in _cases(test_gpu_ops.test_conv_of_single_taps_is_an_exact_displacement, "n,cin,cout,h,w")])
    assert {NARROW4, RING, NARROW, WIDE} <= set(got), got


def test_large_biases(tiles):
    got = tiles([c + (True,) for c in _cases(test_gpu_ops.test_conv_adds_a_large_bias_to_finished_sums, "k,n,cin,cout,h,w")])
    assert {NARROW4, RING, NARROW, WIDE} <= set(got), got


def test_heights_that_the_batch_chooses(tiles):
    six, six_wide, eight, eight_ring, eight_wide = "6, 1, 3, 18", "6, 2, 3, 0", "8, 1, 3, 0", "8, 1, 3, 18", "8, 2, 3, 0"
    got = tiles([(3,) + c + (False,) for c in test_gpu_conv_rows.PAIR])
    assert got == [six, eight, eight_ring, six, six_wide, eight_wide, eight], got
    # a whole ring up to 512 workgroups, from 256 input channels on
    assert tiles([(3, n, cin, 128, 131, 145, False) for n in (3, 4) for cin in (224, 256, 512)]) == [eight, eight_ring, eight_ring] + [eight] * 3
    assert tiles([(3, n, 128, 128, h, 129, False) for n in (1, 3) for h in (128, 151)]) == [six, six, eight, eight]
    assert tiles([(3, 1, 256, 256, 101, 99, True), (3, 1, 128, 256, 101, 99, False)]) == [RING, RING]   # (fp32 output, a layer that widens)
