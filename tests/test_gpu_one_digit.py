"""One gadget digit with several rotations in a workgroup: the Perm kernels reuse their LDS images from rotation to
rotation, and with one digit no forward transform stands between two uses.  Ciphertexts against the oracle (the keys are too
noisy to decrypt); launches of at most two workgroups a CU and larger ones, whole ciphertexts and blocks of eight."""
import dataclasses

import pytest

from paper_2105_01827_amd import workloads as wl
from tests.helpers import small_params
from tests.test_gpu_parity import conv_case, fc_case

pytestmark = pytest.mark.gpu


def _one_digit(n):
    return dataclasses.replace(wl.DEFAULT, gadget_bits=60) if n == 2048 else small_params(n, gadget_bits=60)


@pytest.mark.parametrize("n,n_o,n_i,batch,chunks", [
    (2048, 128, 1024, 64, 32), (2048, 256, 2048, 9, 128), (2048, 32, 1024, 70, 11),
    (1024, 128, 512, 40, 32), (1024, 32, 512, 64, 12), (1024, 16, 1024, 100, 8),
    (4096, 128, 4096, 7, 32), (4096, 500, 1024, 8, 32), (8192, 64, 8192, 9, 21),
])
def test_he_fc_with_several_rotations_a_chunk(n, n_o, n_i, batch, chunks):
    par = _one_digit(n)
    plan = fc_case(par, n_o, n_i, batch, sorted({0, batch // 2, batch - 1}), seed=batch)[2]
    assert plan.workspace_bytes(batch) // (batch * 2 * n * 8) - 1 == chunks < plan.G - 1


@pytest.mark.parametrize("matrix_cores", [False, True])
@pytest.mark.parametrize("n,shape,batch", [      # kernel orders (c_n), chunks an output ciphertext
    (2048, (128, 8, 1, 1, 16, 16), 16),          # 8, 3
    (1024, (64, 4, 1, 1, 16, 16), 16),           # 4, 3
    (4096, (128, 16, 1, 1, 16, 16), 5),          # 16, 5
    (8192, (64, 32, 1, 1, 16, 16), 40),          # 32, 3
])
def test_he_conv_with_several_rotations_a_chunk(n, shape, batch, matrix_cores):
    last = -(-shape[0] // (n // 256)) - 1
    conv_case(_one_digit(n), shape, batch, [(0, 0), (batch // 2, last), (batch - 1, last)], seed=n, matrix_cores=matrix_cores)
