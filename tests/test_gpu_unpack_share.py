"""The plaintext sum of every output's slots on the device for slot words over the whole 64-bit range, on rings below, at and
above one batch of slots a thread, with small and large plaintext primes."""
import numpy as np
import pytest

from paper_2105_01827_amd import workloads as wl
from tests.helpers import small_params
from tests.test_gpu_parity import both, harness

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p_bits", [20, 31])
@pytest.mark.parametrize("n,n_o,n_i", [(8, 2, 4), (64, 5, 12), (512, 3, 500), (1024, 1, 1024), (2048, 100, 784), (4096, 1000, 4),
                                       (8192, 1, 8192)])
def test_words_of_any_size(n, n_o, n_i, p_bits):
    H = harness()
    par = small_params(n, p=wl.find_prime_below(1 << p_bits, 2 * n))
    ctx, _ = both(par)
    rng = np.random.default_rng(n + p_bits)
    plan = ctx.fc_plan(rng.integers(0, par.p, size=(n_o, n_i), dtype=np.uint64))
    count = 3
    slots = rng.integers(0, 1 << 64, size=(count, n), dtype=np.uint64)
    edges = [0, par.p - 1, par.p, 2 * par.p - 1, (1 << 64) - 1, ((1 << 64) // par.p) * par.p, ((1 << 64) // par.p) * par.p - 1]
    slots[0, :len(edges)] = np.array(edges, dtype=np.uint64)
    slots[1] = np.uint64((1 << 64) - 1)
    d_out = H.dev_empty(count * n_o)
    plan.unpack_share_batch(H.to_dev(slots), count, d_out)
    got = H.to_host(d_out).reshape(count, n_o)
    for i in range(count):
        assert np.array_equal(got[i], plan.unpack_share(slots[i] % np.uint64(par.p))), i
