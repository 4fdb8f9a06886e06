"""The order in which he_fc hands (input, chunk) pairs to workgroups: every input of a batch decrypts to W x and the first and
last equal the oracle, for chunk counts that divide among eight XCDs and counts that do not, with remainders."""
import numpy as np
import pytest

from paper_2105_01827_amd import workloads as wl
from tests.test_gpu_parity import fc_case, plain_matvec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_o,n_i,batch,chunks", [
    (128, 1024, 7, 64), (128, 1024, 20, 63), (64, 1024, 41, 31), (1000, 512, 3, 255), (250, 1024, 8, 127), (250, 1024, 17, 64),
])
def test_every_input_is_summed_once(n_o, n_i, batch, chunks):
    par = wl.DEFAULT
    ctx, o, plan, sk, W, x, r, got = fc_case(par, n_o, n_i, batch, [0, batch - 1], seed=batch)
    assert plan.workspace_bytes(batch) // (batch * 2 * par.n * 8) - 1 == chunks
    for b in range(batch):
        share = plan.unpack_share(ctx.decrypt(sk, got[b]))
        assert np.array_equal((share + r[b]) % np.uint64(par.p), plain_matvec(W, x[b], par.p)), b


@pytest.mark.parametrize("n_o,n_i,batch,chunks", [
    (17, 1251, 30, 17), (100, 784, 9, 56), (64, 1024, 57, 8), (32, 2048, 256, 2), (32, 2048, 257, 2), (200, 500, 7, 63),
])
def test_special_prime_sums_fill_one_round(n_o, n_i, batch, chunks):
    """With the special prime long sums are cut into at most 512 workgroups, up to 256 inputs."""
    par = wl.DEFAULT_SPECIAL
    ctx, o, plan, sk, W, x, r, got = fc_case(par, n_o, n_i, batch, [0, batch - 1], seed=batch)
    assert plan.workspace_bytes(batch) // (batch * 2 * par.n * 8) - 1 == chunks
    assert batch > 256 or batch * chunks <= 512
    for b in sorted({0, batch // 3, batch // 2, batch - 2, batch - 1}):
        share = plan.unpack_share(ctx.decrypt(sk, got[b]))
        assert np.array_equal((share + r[b]) % np.uint64(par.p), plain_matvec(W, x[b], par.p)), b
