"""The product kernel whose weights go through LDS as well (256 x 256 and 192 x 128 tiles): fewer half stages than there are
buffers and more than two rounds of them, an odd number of blocks of 32 inputs (the last stage half full) uncut and in the
last cut, rows and features that do not fill the last tile, one row more or less than a tile.  Tolerance as for the tiles."""
import pytest

from paper_2504_11816_amd import binding

from test_gpu_linear_tiles import product

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,cuts,m,n_out,n_in", [
    ((192, 128), 1, 370, 12304, 32), ((192, 128), 1, 384, 12304, 96), ((192, 128), 1, 370, 12304, 160), ((192, 128), 1, 384, 12304, 544),
    ((192, 128), 1, 760, 6160, 4128), ((192, 128), 3, 129, 8208, 4128), ((192, 128), 5, 190, 6160, 8224), ((192, 128), 7, 129, 4112, 8224),
    ((256, 256), 1, 570, 16400, 32), ((256, 256), 1, 570, 16400, 96), ((256, 256), 1, 570, 16400, 160), ((256, 256), 1, 1025, 12304, 544),
    ((256, 256), 3, 193, 16400, 3104), ((256, 256), 7, 1024, 2064, 8224)])
def test_wide_tiles(form, cuts, m, n_out, n_in):
    uncut = cuts == 1
    assert binding.okv_linear_plan(m, n_out, n_in, 0 if uncut else None) == (2, *form, cuts)
    product(m, n_out, n_in, 770 + m, relu=True, residual=True, workspace=not uncut)
    if uncut and n_in <= 160:
        product(m, n_out, n_in, 771 + m, bias=False, workspace=False)


# more rows than 1024: in one round of workgroups and in several, rows one more than a tile's, inputs an odd number of blocks of 32 or not
@pytest.mark.parametrize("m,n_out,n_in", [(1153, 4112, 96), (1153, 4112, 576), (4096, 1040, 544), (2111, 8208, 192)])
def test_192_by_128_tiles_beyond_1024_rows(m, n_out, n_in):
    assert binding.okv_linear_plan(m, n_out, n_in, 0) == (2, 192, 128, 1)
    product(m, n_out, n_in, 780 + m, relu=True, residual=True, workspace=False)
