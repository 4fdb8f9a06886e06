"""Perm with the last digit's key folded into the others, at digit counts from one to six, against the oracle:
one rotation at a time and every rotation from one shared decomposition."""
import dataclasses

import numpy as np
import pytest
import torch

from tests import gpu_harness as H
from oracle.oracle import Oracle
from paper_2105_01827_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("special", [False, True])
@pytest.mark.parametrize("gadget_bits", [62, 60, 59, 31, 30, 20, 15, 11])
def test_rotations_at_every_digit_count(gadget_bits, special):
    par = dataclasses.replace(wl.DEFAULT_SPECIAL if special else wl.DEFAULT, gadget_bits=gadget_bits)
    ctx = binding.Context(par.n, par.q, par.p, par.gadget_bits, par.special)
    o = Oracle(par.n, par.q, par.p, par.gadget_bits, par.special)
    sk, osk, n, count = ctx.keygen(3), o.keygen(3), par.n, 2
    rots = [(0, 1), (1, 5)]
    gk = ctx.galois_keygen(sk, rots, seed=42)
    rng = np.random.default_rng(gadget_bits)
    cts = rng.integers(0, par.q, (count, 2 * n), dtype=np.uint64)
    cts[1] = par.q - 1                                  # every digit of every coefficient at the modulus' own digits
    d_in = H.import_cts(ctx, cts)
    want = [[o.perm(cts[i], o.galois_elt(*rot), o.galois_key(osk, o.galois_elt(*rot), 42)) for rot in rots]
            for i in range(count)]
    for k, rot in enumerate(rots):
        d_out = H.dev_empty(count * 2 * n)
        ctx.rotate(gk, d_in, count, rot, d_out)
        got = H.export_cts(ctx, d_out, count)
        for i in range(count):
            assert np.array_equal(got[i], want[i][k])
    wsb = ctx.rotate_hoisted_workspace(count)
    ws, d_out = torch.empty(wsb, dtype=torch.uint8, device="cuda"), H.dev_empty(count * len(rots) * 2 * n)
    ctx.rotate_hoisted(gk, d_in, count, d_out, ws, wsb)
    got = H.export_cts(ctx, d_out, count * len(rots)).reshape(count, len(rots), 2 * n)
    for i in range(count):
        for k in range(len(rots)):
            assert np.array_equal(got[i, k], want[i][k])
