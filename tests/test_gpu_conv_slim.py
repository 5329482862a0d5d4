"""Convolutions with at most 64 channels on one side: 256 pixels x 64 channels forward and for input gradients (by parity of the
pixel at stride 2, whose four products differ in size on odd images), 64 x 256 for weight gradients with their reductions
divided.  Channels below, at and above a tile, pixels that are no whole tiles, one pixel wide filters, images of one pixel.
Against the unfolded product in fp32: a bf16 result carries one rounding (2^-9 per element); fp32 sums add less than that."""
import pytest

pytestmark = pytest.mark.gpu

from test_gpu_conv_broad import g, test_forward_and_gradients as check      # noqa: F401


@pytest.mark.parametrize("n,h,ci,co,k,stride", [(1, 1, 8, 8, 1, 1), (5, 9, 8, 64, 3, 1), (16, 33, 64, 48, 3, 1), (9, 40, 56, 64, 3, 2), (40, 47, 64, 24, 3, 2),
                                                (3, 64, 72, 64, 3, 1), (17, 31, 64, 72, 5, 1), (33, 57, 8, 64, 7, 2), (30, 41, 64, 192, 1, 2), (70, 29, 40, 96, 3, 1)])
def test_few_channels(g, n, h, ci, co, k, stride):      # noqa: F811
    check(g, n, h, ci, co, k, stride)
