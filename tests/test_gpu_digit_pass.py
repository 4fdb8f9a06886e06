"""The first transform pass on gadget digits, which adds up products of several digits before it reduces them: digits at both ends of
their range and mixed, digits that are too long for it beside the longest that are not, moduli whose low words are long and short, with
and without a special prime, on every ring with kernels of its own; Perm and the hoisted rotations, against the oracle."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2105_01827_amd import workloads as wl
from tests import gpu_harness as H
from tests.helpers import small_params
from tests.test_gpu_parity import both

pytestmark = pytest.mark.gpu

RINGS, BITS = [1024, 2048, 4096, 8192], [12, 20, 28, 29, 30, 31, 32]


def parameters(n, bits, special):
    if special and (n == 8192 or bits == 32):
        pytest.skip("no kernels of its own, or as without a special prime")
    par = small_params(n, gadget_bits=bits)
    if n == 2048 and bits == 20:
        par = dataclasses.replace(wl.DEFAULT, gadget_bits=bits)      # a short low word
    if special:
        par = dataclasses.replace(par, special=wl.find_prime_below(1 << 60, 2 * n))
    return par


# which of them take the sums of products: test_digit_pass_host.py
@pytest.mark.parametrize("special", [False, True])
@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("n", RINGS)
def test_rotations(n, bits, special):
    par = parameters(n, bits, special)
    ctx, o = both(par)
    sk, osk = ctx.keygen(3), o.keygen(3)
    rng = np.random.default_rng(n + bits)
    top = (1 << 59) - 1                                              # every digit but the last all ones
    one = (1 << bits) - 1
    c1 = np.stack([np.full(n, top, np.uint64), np.where(np.arange(n) % 2, one, top - one).astype(np.uint64),
                   np.where(rng.integers(0, 2, n), top, 0).astype(np.uint64), rng.integers(0, par.q, n, dtype=np.uint64),
                   np.full(n, par.q - 1, np.uint64)])
    cts = np.concatenate([rng.integers(0, par.q, c1.shape, dtype=np.uint64), c1], axis=1)
    rots = [(0, 1), (1, n // 2 - 3)]
    gk = ctx.galois_keygen(sk, rots, seed=42)
    keys = {r: (o.galois_elt(*r), o.galois_key(osk, o.galois_elt(*r), 42)) for r in rots}
    d_in, count = H.import_cts(ctx, cts), len(cts)
    d_out = H.dev_empty(count * 2 * n)
    ctx.rotate(gk, d_in, count, rots[1], d_out)
    got = H.export_cts(ctx, d_out, count)
    for i in range(count):
        assert np.array_equal(got[i], o.perm(cts[i], *keys[rots[1]])), i
    d_all, wsb = H.dev_empty(count * len(rots) * 2 * n), ctx.rotate_hoisted_workspace(count)
    ws = torch.empty(max(wsb, 8), dtype=torch.uint8, device="cuda")
    ctx.rotate_hoisted(gk, d_in, count, d_all, ws, wsb)
    got = H.export_cts(ctx, d_all, count * len(rots)).reshape(count, len(rots), 2 * n)
    for i in range(count):
        digits = o.decperm(cts[i][n:])
        for k, r in enumerate(rots):
            assert np.array_equal(got[i, k], o.hstperm(cts[i][:n], digits, *keys[r])), (i, r)
