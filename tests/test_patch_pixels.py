"""The product that takes the place of a division by a patch's width (csrc/saliency_body.h, PatchPixels), on the CPU: exact wherever it
is used."""
import numpy as np


def test_row_of_a_pixel_by_a_product_is_the_quotient():
    p = np.arange(1 << 16, dtype=np.uint64)
    for pw in range(2, 684):                                # images of up to 16384 pixels a side, 24 patches
        inverse = np.uint64(0xFFFFFFFF // pw + 1)
        assert np.array_equal((p * inverse) >> np.uint64(32), p // np.uint64(pw)), pw
