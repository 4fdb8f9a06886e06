"""The client's batch steps on the rings with kernels of their own, with plaintext primes of the 32-bit and of the 64-bit slot
transforms: Gaussian draws in the tails of the distribution, and decryption at the edges of its rounding, against the oracle."""
import numpy as np
import pytest

from paper_2105_01827_amd import workloads as wl
from tests.helpers import small_params
from tests.test_gpu_parity import both, harness

pytestmark = pytest.mark.gpu


def _params(n, wide_p):
    return small_params(n, p=wl.find_prime_below(1 << (27 if wide_p else 20), 2 * n))


@pytest.mark.parametrize("wide_p", [False, True])
@pytest.mark.parametrize("n", [1024, 2048, 4096, 8192])
def test_encryption(n, wide_p):
    """Of a polynomial's n draws one in 128 has a top byte with several thresholds inside."""
    H = harness()
    par, count = _params(n, wide_p), 5
    ctx, o = both(par)
    sk, osk = ctx.keygen(3), o.keygen(3)
    slots = np.random.default_rng(n).integers(0, par.p, size=(count, n), dtype=np.uint64)
    seeds = np.arange(count, dtype=np.uint64) + np.uint64(77)
    d_ct, d_slots = H.dev_empty(count * 2 * n), H.dev_empty(count * n)
    ctx.encrypt_batch(sk, H.to_dev(slots), H.to_dev(seeds), count, d_ct)
    got = H.export_cts(ctx, d_ct, count)
    for i in range(count):
        assert np.array_equal(got[i], o.encrypt(osk, slots[i], int(seeds[i]))), i
    ctx.decrypt_batch(sk, H.import_cts(ctx, got), count, d_slots)
    assert np.array_equal(H.to_host(d_slots).reshape(count, n), slots)


@pytest.mark.parametrize("wide_p", [False, True])
@pytest.mark.parametrize("n", [1024, 2048, 4096, 8192])
def test_decryption_at_the_edges_of_its_rounding(n, wide_p):
    """c1 = 0, and the coefficients of c0 next to multiples of q / (2 p): the smallest, the largest and some between."""
    H = harness()
    par = _params(n, wide_p)
    ctx, o = both(par)
    sk, osk = ctx.keygen(3), o.keygen(3)
    rng = np.random.default_rng(n)
    halves = [0, 1, 2, 2 * par.p - 1, 2 * par.p - 2, 2 * par.p] + [int(h) for h in rng.integers(0, 2 * par.p, size=n)]
    coefs = [(h * par.q // (2 * par.p) + d) % par.q for h in halves for d in (-1, 0, 1)][:n]
    ct = np.zeros((1, 2 * n), np.uint64)
    ct[0, :n] = np.array(coefs, dtype=np.uint64)
    d_slots = H.dev_empty(n)
    ctx.decrypt_batch(sk, H.import_cts(ctx, ct), 1, d_slots)
    assert np.array_equal(H.to_host(d_slots), o.decrypt(osk, ct[0]))
