"""Moduli that the ring kernels' signed products tell apart: close to 2^60 with a small low word (one multiply-add fewer) or
another one, far below 2^60, and small; on ciphertexts whose residues are the largest and the least, against the oracle."""
import numpy as np
import pytest

from oracle.oracle import Oracle
from paper_2105_01827_amd import binding, workloads as wl
from tests import gpu_harness as H

pytestmark = pytest.mark.gpu


def _modulus(kind, n):
    """A prime = 1 mod 2n of the kind, not the largest below 2^60 (which is the special prime's)."""
    top = {"low_word_small": 1 << 60, "low_word_large": (1 << 60) - (3 << 30), "middle": 3 << 58, "half": (1 << 59) + (1 << 40),
           "small": 1 << 41}[kind]
    q = wl.find_prime_below(top, 2 * n)
    if kind == "low_word_small":
        q = wl.find_prime_below(q, 2 * n)
    low = q & 0xFFFFFFFF
    if kind.startswith("low_word"):
        assert (min(low, (1 << 32) - low) <= 1 << 28) == (kind == "low_word_small")
    return q


@pytest.mark.parametrize("special", [False, True])
@pytest.mark.parametrize("kind", ["low_word_small", "low_word_large", "middle", "half", "small"])
@pytest.mark.parametrize("n", [1024, 2048, 4096, 8192])
def test_rotations_of_extreme_residues(n, kind, special):
    if special and kind == "small":
        pytest.skip("the special prime has to be below 2q for the ring kernels: any-n path, tested elsewhere")
    q, p = _modulus(kind, n), wl.find_prime_below(1 << 20, 2 * n)
    P = wl.find_prime_below(1 << 60, 2 * n) if special else 0
    ctx, o = binding.Context(n, q, p, 20, P), Oracle(n, q, p, 20, P)
    sk, osk = ctx.keygen(3), o.keygen(3)
    rng = np.random.default_rng(n)
    cts = rng.integers(0, q, (4, 2 * n), dtype=np.uint64)
    cts[1] = q - 1
    cts[2] = 0
    cts[3, ::2], cts[3, 1::2] = q - 1, 0
    # evaluation form at its largest: every residue of the internal ciphertext is q - 1
    constant = np.zeros((1, 2 * n), dtype=np.uint64)
    constant[0, 0] = constant[0, n] = q - 1
    cts = np.concatenate([cts, constant])
    d_in = H.import_cts(ctx, cts)
    assert np.array_equal(H.export_cts(ctx, d_in, len(cts)), cts)
    rots = [(0, 1), (1, 5)]
    gk = ctx.galois_keygen(sk, rots, seed=42)
    for rot in rots:
        d_out = H.dev_empty(cts.size)
        ctx.rotate(gk, d_in, len(cts), rot, d_out)
        got = H.export_cts(ctx, d_out, len(cts))
        g = o.galois_elt(*rot)
        ksk = o.galois_key(osk, g, 42)
        for i in range(len(cts)):
            assert np.array_equal(got[i], o.perm(cts[i], g, ksk)), (rot, i)
