"""Moduli that the ring kernels' signed products tell apart: close to 2^60 with a small low word (one multiply-add fewer) or
another one, far below 2^60, and small; on ciphertexts whose residues are the largest and the least, against the oracle."""
import concurrent.futures

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


def _extreme_cts(n, q, count, seed):
    """Random ciphertexts, the first five with the largest and least residues in either form."""
    cts = np.random.default_rng(seed).integers(0, q, (count, 2 * n), dtype=np.uint64)
    cts[1] = q - 1
    cts[2] = 0
    cts[3, ::2], cts[3, 1::2] = q - 1, 0
    cts[4] = 0
    cts[4, 0] = cts[4, n] = q - 1
    return cts


@pytest.mark.parametrize("n,kind,gadget_bits,special", [
    (n, kind, bits, special) for n in (1024, 2048, 4096, 8192) for kind in ("middle", "half")
    for bits, special in ((12, False), (7, False), (12, True)) if not special or n < 8192
])
def test_long_sums_far_below_2_60(n, kind, gadget_bits, special):
    """Running sums over several rotations of five and nine digits a workgroup: how far they may grow before they are brought
    near the modulus again depends on its distance from 2^60."""
    q, p = _modulus(kind, n), wl.find_prime_below(1 << 20, 2 * n)
    P = wl.find_prime_below(1 << 60, 2 * n) if special else 0
    ctx, o = binding.Context(n, q, p, gadget_bits, P), Oracle(n, q, p, gadget_bits, P)
    sk, osk = ctx.keygen(3), o.keygen(3)
    n_o, n_i, batch = 128, n // 2, 300 if n <= 2048 else 64
    W, _, r = wl.fc_inputs(wl.FcShape("t", n_o, n_i, batch), p=p, seed=n)
    plan = ctx.fc_plan(W)
    assert plan.G == 64
    plan.bind(ctx.galois_keygen(sk, plan.rotations(), seed=1))
    chunks = plan.workspace_bytes(batch) // (batch * 2 * n * 8) - 1
    assert chunks <= 16                                        # four rotations a workgroup at least
    cts = _extreme_cts(n, q, batch, seed=gadget_bits)
    got, _ = H.gpu_he_fc(ctx, plan, cts, r, mask_seed=17)
    wpoly, ksk = o.fc_encode_rowwise(W), o.fc_keys(osk, n_o, n_i, seed=1)

    def item(b):
        return o.he_fc(wpoly, cts[b], ksk, o.fc_mask_slots(n_o, n_i, r[b], 17, b))[0]

    items = [0, 1, 2, 3, 4, batch - 1]
    with concurrent.futures.ThreadPoolExecutor(len(items)) as pool:      # the C call releases the interpreter lock
        for b, want in zip(items, pool.map(item, items)):
            assert np.array_equal(got[b], want), b


@pytest.mark.parametrize("kind", ["low_word_small", "low_word_large", "middle", "half", "small"])
@pytest.mark.parametrize("n", [1024, 2048, 4096, 8192])
def test_import_of_words_below_four_moduli(n, kind):
    """Import takes words up to 4q - 1 as their residues, whatever the modulus."""
    q = _modulus(kind, n)
    ctx = binding.Context(n, q, wl.find_prime_below(1 << 20, 2 * n), 20)
    cts = _extreme_cts(n, q, 6, seed=n)
    more = np.random.default_rng(n + 1).integers(0, 4, cts.shape, dtype=np.uint64)
    more[:5] = 3
    want, got = H.import_cts(ctx, cts), H.import_cts(ctx, cts + more * np.uint64(q))
    assert np.array_equal(H.to_host(got), H.to_host(want))
    assert np.array_equal(H.export_cts(ctx, got, len(cts)), cts)
