"""Which kernel a product takes where the simple and the tile kernel both could, against what both took on MI355X (us, weights from
HBM): the faster one at every shape, where they are more than 10 % apart.  No GPU: the choice is made on the host."""
import pytest

from paper_2504_11816_amd import binding

# rows, features, inputs, workspace for eight cuts or none, simple kernel, tile kernel
MEASURED = [
    (9, 4096, 10240, False, 16.6, 37.3), (9, 512, 12288, False, 11.8, 36.0), (9, 2048, 16384, False, 20.4, 55.3), (10, 4096, 12288, False, 19.6, 44.0),
    (10, 8192, 10240, False, 31.0, 40.3), (12, 4096, 5120, False, 10.0, 19.8), (16, 4224, 4096, False, 14.1, 16.1), (17, 4096, 6144, False, 13.7, 23.4),
    (17, 192, 20480, False, 29.1, 58.1), (17, 1056, 20480, False, 34.4, 68.3), (19, 3072, 2304, False, 6.1, 8.7), (36, 256, 2304, False, 7.3, 9.1),
    (40, 512, 4192, False, 10.2, 14.2), (50, 6144, 13824, False, 106.0, 50.8), (52, 5120, 4224, False, 35.6, 17.4), (77, 5120, 12288, False, 132.6, 45.5),
    (94, 4256, 20480, False, 251.4, 72.5), (108, 3072, 1056, False, 7.4, 5.4), (110, 5120, 2400, False, 32.9, 14.4),
    (10, 2304, 2240, True, 4.6, 6.4), (23, 256, 1568, True, 4.0, 5.3), (91, 320, 13824, True, 72.8, 9.6), (113, 768, 16384, True, 116.9, 15.5)]


@pytest.mark.parametrize("m,n_out,n_in,workspace,simple_us,tile_us", MEASURED)
def test_the_faster_kernel(m, n_out, n_in, workspace, simple_us, tile_us):
    assert max(simple_us, tile_us) > 1.1 * min(simple_us, tile_us)
    kernel = binding.okv_linear_plan(m, n_out, n_in, 8 * m * n_out * 4 if workspace else 0)[0]
    assert kernel == (0 if simple_us < tile_us else 2)


# rows, features, inputs, the form and cuts that measured faster than the next choice by 5 % and more, with the launch that adds the shares
@pytest.mark.parametrize("m,n_out,n_in,form,cuts", [(192, 4096, 16384, (192, 128), 8), (180, 5120, 11008, (192, 128), 6),
                                                    (1100, 16384, 4096, (192, 128), 1), (1281, 4096, 5120, (192, 128), 1),
                                                    # three, two and four cuts of 256 x 256 would leave 258, 181 and 187 MB of shares
                                                    (3507, 6144, 8192, (256, 192), 1), (1842, 12288, 10240, (256, 192), 1), (952, 12288, 20480, (256, 192), 1)])
def test_the_faster_tiles(m, n_out, n_in, form, cuts):
    assert binding.okv_linear_plan(m, n_out, n_in) == (2, *form, cuts)
