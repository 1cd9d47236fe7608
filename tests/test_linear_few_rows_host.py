"""Which kernel a product of up to 16 rows (and, at the end, of 65 to 192) takes, against what the simple and the staged kernel took on MI355X (us, weights from HBM):
the faster one wherever they are more than 12 % apart (from 9 rows on also 2 us, which a layer norm behind the simple one takes more).  No GPU: the choice is made on the host."""
import pytest

from paper_2504_11816_amd import binding

# rows, features, inputs, simple kernel, staged kernel with the launch that adds its shares
MEASURED = [
    (4, 4096, 4096, 6.8, 10.4), (8, 4096, 4096, 7.1, 10.4), (8, 16384, 4096, 21.9, 25.1), (8, 4096, 16384, 21.6, 25.3), (1, 2560, 10240, 10.5, 13.0),
    (8, 768, 3072, 4.9, 7.5), (8, 2048, 2048, 4.7, 7.5), (8, 2560, 2560, 5.0, 7.6), (1, 768, 3072, 4.5, 7.4), (1, 304, 3072, 4.6, 7.4),
    (8, 5120, 20480, 48.5, 34.9), (8, 1024, 18432, 19.4, 11.4), (2, 512, 20480, 17.3, 10.4), (7, 416, 12800, 13.6, 8.9), (8, 1632, 17920, 19.9, 14.0),
    (12, 4096, 4096, 7.3, 10.5), (16, 4096, 4096, 8.3, 10.6), (12, 2048, 2048, 4.6, 7.5), (16, 2048, 2048, 5.0, 7.4), (11, 4096, 2048, 4.9, 8.2),
    (12, 5120, 5120, 15.4, 12.9), (16, 12288, 4096, 21.3, 17.9), (12, 5120, 20480, 54.8, 36.8), (16, 20480, 5120, 45.0, 34.9), (16, 15360, 5120, 36.1, 25.7),
    # inputs that are no multiple of 1024
    (9, 2560, 2560, 5.2, 7.4), (9, 3840, 2560, 5.3, 8.3), (16, 3840, 2560, 6.3, 8.5), (12, 2400, 13568, 18.9, 32.2), (16, 1472, 9472, 15.7, 23.0),
    (12, 912, 12032, 15.3, 25.0), (10, 272, 13568, 18.5, 31.9), (16, 10240, 2560, 15.2, 10.8), (16, 2560, 10240, 17.4, 13.5),
    (12, 576, 11520, 17.7, 9.2), (13, 8672, 6656, 30.0, 21.2), (16, 2224, 16896, 26.9, 16.8)]


@pytest.mark.parametrize("m,n_out,n_in,simple_us,staged_us", MEASURED)
def test_the_faster_kernel(m, n_out, n_in, simple_us, staged_us):
    assert max(simple_us, staged_us) > 1.12 * min(simple_us, staged_us) and (m <= 8 or abs(simple_us - staged_us) > 2.0)
    assert binding.okv_linear_plan(m, n_out, n_in)[0] == (0 if simple_us < staged_us else 1)


def test_without_a_workspace_few_rows_run_uncut():
    for m in (1, 8):
        assert binding.okv_linear_plan(m, 1024, 18432, 0) == (0, 16, 16, 1)
    assert binding.okv_linear_plan(8, 1024, 18432)[3] > 1
    assert binding.okv_linear_plan(16, 4096, 4096, 0) == binding.okv_linear_plan(16, 4096, 4096, 1 << 30) == (0, 16, 16, 1)


# 65 to 192 rows: rows, features, inputs, staged kernel, tiles (with the launch that adds the shares), more than 8 % apart
@pytest.mark.parametrize("m,n_out,n_in,staged_us,tile_us", [
    (129, 496, 6400, 13.1, 8.9), (136, 608, 12032, 20.2, 12.8), (177, 480, 6144, 14.0, 9.7), (184, 400, 4096, 10.9, 7.6), (192, 768, 3072, 11.7, 8.9),
    (145, 2048, 13824, 29.0, 22.0), (192, 20480, 5120, 85.2, 72.0), (144, 4160, 13824, 50.0, 34.5),
    (128, 5120, 20480, 65.5, 49.0), (128, 20480, 5120, 66.3, 52.4), (128, 2304, 768, 6.2, 4.9), (96, 5120, 20480, 56.8, 44.7),
    (128, 12288, 4096, 28.0, 31.0), (128, 16384, 4096, 35.0, 38.0), (160, 4608, 3072, 15.0, 16.7), (136, 16384, 3072, 27.2, 30.1), (136, 12288, 4096, 30.1, 34.6), (160, 6144, 4096, 21.8, 24.6), (136, 15360, 5120, 43.2, 47.2),
    # more than 20480 features
    (128, 24576, 4096, 56.0, 46.4), (128, 28672, 4096, 62.3, 48.8), (65, 28672, 8192, 94.1, 83.4), (67, 32288, 2816, 38.2, 34.8),
    (112, 51200, 2048, 57.1, 41.2), (128, 27648, 5120, 76.9, 64.1), (65, 20736, 1024, 13.2, 14.3),
    # fewer than 288
    (97, 272, 8192, 11.4, 8.2), (128, 128, 16384, 14.9, 11.2), (65, 128, 16384, 9.5, 10.9), (76, 96, 4352, 17.1, 8.2), (129, 128, 4096, 8.1, 7.0),
    (160, 272, 8192, 13.0, 8.5), (192, 256, 4096, 10.3, 7.1), (192, 48, 512, 6.2, 4.2)])
def test_many_rows_staged_or_tiles(m, n_out, n_in, staged_us, tile_us):
    assert binding.okv_linear_plan(m, n_out, n_in)[0] == (1 if staged_us < tile_us else 2)
