"""The product kernel for few rows where its walk over the inputs can go wrong: wavefronts without a block of 32 inputs, with one, with
one less and one more than the blocks it keeps in flight (8, or 4 and 2 with more fragments of rows) and than twice as many, wavefronts
that get different numbers of blocks; one row, a full and a begun fragment.  Tolerance as for the tiles."""
import pytest

from paper_2504_11816_amd import binding

from test_gpu_linear_tiles import product

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,blocks", [(m, n) for m in (1, 8, 17) for n in (1, 2, 5, 7, 9, 17, 31, 33, 35, 37, 63, 65, 67, 71)] +
                         [(50, 5), (50, 9), (50, 17), (100, 1), (100, 5)])
def test_blocks_of_a_wavefront(m, blocks):
    n_in = 32 * blocks
    assert binding.okv_linear_plan(m, 80, n_in, 0)[0] == 0
    product(m, 80, n_in, 700 + m, relu=True, residual=True, workspace=False)
    product(m, 80, n_in, 701 + m, bias=False, workspace=False)


# the staged kernel with less than a fragment of rows: many cuts, two and one, one tile of features a workgroup to four, a last one that is not full
@pytest.mark.parametrize("m,n_out,n_in,cuts", [(1, 16, 12800, 25), (3, 512, 20480, 20), (8, 16, 8192, 16), (7, 240, 8192, 16), (5, 1040, 12800, 10),
                                               (8, 4112, 8192, 2), (8, 8208, 8192, 1)])
def test_staged_kernel(m, n_out, n_in, cuts):
    assert binding.okv_linear_plan(m, n_out, n_in)[::3] == (1, cuts)
    product(m, n_out, n_in, 720 + m, relu=True, residual=True)
    product(m, n_out, n_in, 721 + m, bias=False, residual=True, alias=True)


# 9 to 16 rows in the simple kernel, inputs that are no multiple of 1024
@pytest.mark.parametrize("m,n_out,n_in", [(9, 2560, 2560), (16, 1472, 9472), (12, 912, 7424), (10, 272, 13568)])
def test_a_begun_fragment(m, n_out, n_in):
    assert binding.okv_linear_plan(m, n_out, n_in)[0] == 0
    product(m, n_out, n_in, 740 + m, relu=True, residual=True)
    product(m, n_out, n_in, 741 + m, bias=False)
