"""The size rule of the fp32 implicit GEMM (a host function of the library,
called by its C++ name) against measured times of the kernels it chooses
from."""

import ctypes

import pytest

from paper_2110_06037_amd import native as N

# (layout, C, K, R, stride, output pixels, then ns on one MI355X: LDS tile and
# the wave-split tiles of 16 x 16, 32 x 16 and 32 x 32 pixels x channels).  The
# first ten are pointwise layers in NCHW on which an earlier rule took a
# wave-split tile 1.3 to 1.8 times as slow as the LDS tile; the others a spread
# over the range of sizes.
MEASURED = [
    ("NCHW", 88, 16, 1, 1, 121000, 26723, 67230, 48748, 62135),
    ("NCHW", 128, 42, 1, 2, 8405, 9218, 20607, 15768, 16049),
    ("NCHW", 56, 14, 1, 1, 31212, 7866, 15949, 11136, 13650),
    ("NCHW", 120, 27, 1, 2, 18491, 11927, 28211, 19374, 16523),
    ("NCHW", 72, 16, 1, 1, 26645, 9620, 16985, 13301, 16884),
    ("NCHW", 59, 7, 1, 2, 33275, 9481, 17617, 13103, 16854),
    ("NCHW", 88, 21, 1, 1, 11520, 7890, 16310, 11229, 10847),
    ("NCHW", 88, 81, 1, 1, 4356, 8084, 18195, 14397, 11020),
    ("NCHW", 88, 90, 1, 1, 3840, 8180, 16412, 11424, 11076),
    ("NCHW", 88, 125, 1, 1, 3136, 8181, 18628, 14512, 11051),
    ("NCHW", 392, 228, 3, 1, 216, 145774, 13470, 25392, 31778),
    ("NHWC", 32, 253, 1, 2, 90, 5262, 3971, 4476, 4964),
    ("NCHW", 56, 37, 3, 1, 1350, 24479, 5443, 6865, 8173),
    ("NHWC", 32, 344, 3, 1, 87808, 184377, 815003, 566762, 384312),
    ("NHWC", 8, 10, 1, 2, 5202, 5348, 4777, 4446, 5083),
    ("NHWC", 8, 115, 7, 2, 18, 16004, 5087, 5114, 6079),
    ("NCHW", 8, 55, 1, 2, 735, 5562, 4305, 5001, 5839),
    ("NHWC", 200, 51, 3, 1, 864, 50582, 8084, 10072, 14259),
    ("NCHW", 8, 8, 1, 1, 91854, 11375, 34626, 22481, 27803),
    ("NCHW", 112, 77, 3, 1, 9375, 63776, 50386, 34628, 34268),
    ("NC8HW8", 136, 30, 5, 1, 49, 87115, 10368, 13904, 20687),
    ("NHWC", 56, 10, 7, 1, 180, 74637, 8900, 12579, 18657),
    ("NHWC", 32, 323, 5, 1, 1089, 23546, 23146, 20389, 15696),
    ("NHWC", 8, 24, 1, 1, 23328, 5190, 12743, 8453, 8301),
    ("NCHW", 96, 11, 1, 1, 64, 6970, 4817, 5519, 6575),
    ("NC8HW8", 176, 38, 1, 1, 80143, 25733, 84534, 48578, 59833),
    ("NCHW", 184, 13, 3, 1, 26908, 101604, 40930, 38464, 54139),
    ("NHWC", 72, 19, 3, 1, 3528, 21525, 7119, 6614, 8708),
]
TILES = (0, 1 * 8 + 1, 2 * 8 + 1, 2 * 8 + 2)


@pytest.mark.parametrize("row", MEASURED)
def test_fp32_implicit_gemm_takes_a_fast_kernel(row):
    layout, c, k, r, stride, m, *ns = row
    f = ctypes.CDLL(N.LIB_PATH)._ZN2sn1k15ksplit_tile_f32Eiiiiiiiiiii
    # one image of one row: m output pixels
    pick = f(N.LAYOUT[layout], 1, c, 1, (m - 1) * stride + 1, r, r, stride, r // 2, k, 0)
    t = ns[TILES.index(pick)]
    # the times repeat within a few percent; the model's error is 7 to 12 % rms
    assert t <= 1.05 * ns[0] and t <= 1.3 * min(ns), (pick, ns)
