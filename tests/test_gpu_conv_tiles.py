"""The matrix-core product at the edges of its tiles: last term blocks of one to four groups of sixteen terms, one to four
blocks (four are reduced in between), one to three column tiles, row tiles that fill no workgroup, and rings that are no
multiple of 64 coefficients.  Ciphertexts against the oracle."""
import pytest

from tests.helpers import small_params
from tests.test_gpu_parity import conv_case

pytestmark = pytest.mark.gpu


def _all_last(par, shape, batch, **kw):
    c_n = par.n // (1 << (shape[4] * shape[5] - 1).bit_length())
    last = -(-shape[0] // c_n) - 1
    conv_case(par, shape, batch, sorted({(0, 0), (batch // 2, 0), (batch - 1, last)}), matrix_cores=True, **kw)


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


@pytest.mark.parametrize("outputs", [2, 9])          # two row tiles at most, and three
@pytest.mark.parametrize("batch", [3, 10])
def test_blocks_of_eight_by_row_tiles(outputs, batch):
    _all_last(small_params(1024), (64 * outputs // 2, 70, 1, 3, 4, 4), batch, seed=outputs)
