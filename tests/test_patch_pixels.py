"""The product that takes the place of a division by a patch's width (csrc/arith.h, PatchRow), on the CPU: exact wherever it
is used."""
from _util import run_host_program


def test_row_of_a_pixel_by_a_product_is_the_quotient(tmp_path):
    """The header's own code: every width of a patch (images of up to 16384 pixels a side, 24 patches: 1 to 683), every pixel of patches of one
    row, of the largest a product is used for, of the smallest it is not used for and of the largest there are."""
    run_host_program(tmp_path, """
int main() {
    for (uint32_t width = 1; width <= 683; ++width)
        for (uint32_t area : {width, 65536u / width * width, (65536u / width + 1u) * width, 683u * width}) {
            const PatchRow row(width, area);
            for (uint32_t p = 0; p < area; ++p)
                if (row(p) != p / width) { printf("width %u, area %u, pixel %u: row %u\\n", width, area, p, row(p)); return 1; }
        }
    return 0;
}
""")
