"""The matrix-core product at the edges of its tiles: last term blocks of one to four groups of sixteen terms, one to four
blocks (four are reduced in between), one to three column tiles, row tiles that fill no workgroup, and rings that are no
multiple of 64 coefficients.  Every form of its workgroups: one or two tiles of columns by two or four of rows, with sums of more
than three blocks, and results in blocks of eight coefficients.  Ciphertexts against the oracle."""
import pytest

from tests.helpers import small_params
from tests.test_gpu_parity import conv_case

pytestmark = pytest.mark.gpu


def _all_last(par, shape, batch, **kw):
    c_n = par.n // (1 << (shape[4] * shape[5] - 1).bit_length())
    last = -(-shape[0] // c_n) - 1
    return conv_case(par, shape, batch, sorted({(0, 0), (batch // 2, 0), (batch - 1, last)}), matrix_cores=True, **kw)


def _tiles(plan, batch):
    """row tiles, column tiles, term blocks and groups of sixteen terms in the last of them"""
    terms = -(-plan.nterm // 16)
    return -(-plan.nout * plan.cn // 16), -(-2 * batch // 16), -(-terms // 4), (terms - 1) % 4 + 1


# 9 terms for each input ciphertext (4 channels at n = 64, 4x4 images)
@pytest.mark.parametrize("inputs", [1, 2, 4, 7, 8, 16, 20, 23, 28])
def test_term_blocks(inputs):
    _all_last(small_params(64), (6, 4 * inputs - 1, 3, 3, 4, 4), 3, seed=inputs)


@pytest.mark.parametrize("n", [32, 64, 1024])
@pytest.mark.parametrize("batch", [2, 8, 9, 17])
def test_column_tiles(n, batch):
    _all_last(small_params(n), (n // 16 + 1, n // 16 + 2, 3, 3, 4, 4), batch, seed=batch)


# c_n = 4 rows an output ciphertext at n = 64
@pytest.mark.parametrize("outputs", [1, 5, 17, 21])
@pytest.mark.parametrize("batch", [3, 10])
def test_row_tiles(outputs, batch):
    _all_last(small_params(64), (4 * outputs, 10, 1, 3, 4, 4), batch, seed=outputs)


@pytest.mark.parametrize("outputs", [2, 9])          # four row tiles and twenty
@pytest.mark.parametrize("batch", [3, 10])
def test_blocks_of_eight_by_row_tiles(outputs, batch):
    _all_last(small_params(1024), (64 * outputs // 2, 70, 1, 3, 4, 4), batch, seed=outputs)


# c_n = 4 rows an output ciphertext and 3 terms an input ciphertext at n = 1024 with 16x16 images: results in blocks of eight
# coefficients, several coefficients a workgroup
@pytest.mark.parametrize("outputs,row_tiles", [(2, 1), (8, 2), (9, 3)])
@pytest.mark.parametrize("batch,col_tiles", [(3, 1), (10, 2)])
@pytest.mark.parametrize("inputs,blocks,last", [(15, 1, 3), (41, 2, 4), (68, 4, 1), (72, 4, 2)])
def test_blocks_of_eight_in_every_workgroup(outputs, row_tiles, batch, col_tiles, inputs, blocks, last):
    plan = _all_last(small_params(1024), (4 * outputs, 4 * inputs, 1, 3, 16, 16), batch, seed=outputs)[2]
    assert _tiles(plan, batch) == (row_tiles, col_tiles, blocks, last)


# Four row tiles by two column tiles, where loads run two term blocks ahead, through the ends of coefficients: c_n = 8 rows
# an output ciphertext at n = 512 with 8x8 images, two coefficients a workgroup.
@pytest.mark.parametrize("inputs,blocks,last", [
    (5, 1, 1), (10, 1, 2), (15, 1, 3), (20, 1, 4), (24, 2, 1), (30, 2, 2), (36, 2, 3), (41, 2, 4),
    (45, 3, 1), (52, 3, 2), (57, 3, 3), (63, 3, 4), (68, 4, 1), (72, 4, 2), (78, 4, 3), (84, 4, 4), (150, 8, 1),
])
def test_term_blocks_of_eight_wavefronts(inputs, blocks, last):
    plan = _all_last(small_params(512), (40, 8 * inputs, 1, 3, 8, 8), 9, seed=inputs)[2]
    assert _tiles(plan, 9) == (3, 2, blocks, last)


# Two row tiles by two column tiles, and row and column tiles that leave wavefronts without one
@pytest.mark.parametrize("outputs,row_tiles,batch,col_tiles", [(4, 2, 9, 2), (2, 1, 17, 3), (9, 5, 17, 3)])
@pytest.mark.parametrize("inputs,blocks,last", [(30, 2, 2), (78, 4, 3), (132, 7, 1)])
def test_term_blocks_by_tiles(outputs, row_tiles, batch, col_tiles, inputs, blocks, last):
    plan = _all_last(small_params(512), (8 * outputs, 8 * inputs, 1, 3, 8, 8), batch, seed=inputs)[2]
    assert _tiles(plan, batch) == (row_tiles, col_tiles, blocks, last)
