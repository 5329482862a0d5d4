"""Convolutions with at most 64 channels on one side: 256 pixels x 64 channels forward and for input gradients (by parity of the
pixel at stride 2, whose four products differ in size on odd images), 64 x 256 for weight gradients with their reductions
divided, the last range shorter than the others.  Channels below, at and above a tile, pixels that are no whole tiles, one pixel
wide filters; and sizes next to these that other tiles take, down to images of one pixel.  The plan says which tile each of the
three products is on.
Against the unfolded product in fp32: a bf16 result carries one rounding (2^-9 per element); fp32 sums add less than that."""
import pytest

pytestmark = pytest.mark.gpu

import paper_2008_11421_amd as K
from test_gpu_conv_broad import check, g, tiles      # noqa: F401

SLICES, SQUARE, SLIM, FLAT = K.PRODUCT_SLICES, K.PRODUCT_SMALL, K.PRODUCT_NARROW, K.PRODUCT_FLAT
CASES = [((1, 1, 8, 8, 1, 1), [SLICES, SLICES, SLICES]), ((5, 9, 8, 64, 3, 1), [SQUARE, SQUARE, SQUARE]), ((16, 33, 64, 48, 3, 1), [SQUARE, SQUARE, SQUARE]),
         ((9, 40, 56, 64, 3, 2), [SQUARE, SQUARE, SQUARE]), ((40, 47, 64, 24, 3, 2), [SQUARE, SLIM, SQUARE]), ((3, 64, 72, 64, 3, 1), [SQUARE, SQUARE, SQUARE]),
         ((17, 31, 64, 72, 5, 1), [SQUARE, SQUARE, SQUARE]), ((33, 57, 8, 64, 7, 2), [SQUARE, SLIM, SQUARE]), ((30, 41, 64, 192, 1, 2), [SQUARE, SQUARE, SQUARE]),
         ((70, 29, 40, 96, 3, 1), [SQUARE, SLIM, SQUARE]),
         # forward
         ((43, 31, 8, 24, 3, 1), [SLIM, SLIM, SQUARE]), ((37, 37, 16, 64, 3, 1), [SLIM, SLIM, SQUARE]), ((30, 67, 16, 40, 1, 2), [SLIM, SLIM, SQUARE]),
         ((11, 113, 8, 64, 7, 2), [SLIM, SLIM, SQUARE]), ((10, 71, 136, 64, 3, 1), [SLIM, K.PRODUCT_BROAD, FLAT]),
         # weight gradients; 9 ranges of 5 k-tiles, of which the last has 2
         ((22, 22, 160, 16, 7, 2), [SQUARE, SQUARE, FLAT]), ((13, 54, 48, 24, 7, 2), [SQUARE, SQUARE, FLAT]), ((1, 87, 120, 16, 5, 1), [SQUARE, SQUARE, FLAT]),
         ((43, 30, 160, 144, 3, 1), [K.PRODUCT_BROAD, K.PRODUCT_BROAD, FLAT])]


@pytest.mark.parametrize("n,h,ci,co,k,stride,on", [(*size, on) for size, on in CASES])
def test_few_channels(g, n, h, ci, co, k, stride, on):      # noqa: F811
    assert tiles(n, h, ci, co, k, stride) == on
    check(g, n, h, ci, co, k, stride)
