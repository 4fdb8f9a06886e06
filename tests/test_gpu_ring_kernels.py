"""The kernels that rings of 1024, 4096 and 8192 slots share with n = 2048, at both key types and both
multiply-accumulate paths, against the oracle (n = 1024 beside the rings of test_gpu_large_rings)."""
import dataclasses

import numpy as np
import pytest

from paper_2105_01827_amd import workloads as wl
from tests.helpers import rotate_slots, small_params
from tests.test_gpu_parity import both, conv_case, fc_case, harness, plain_matvec

pytestmark = pytest.mark.gpu


def params(n, gadget_bits, special, p_limit=None):
    par = small_params(n, p_limit=p_limit, gadget_bits=gadget_bits)
    return dataclasses.replace(par, special=wl.find_prime_below(par.q, 2 * n)) if special else par


@pytest.mark.parametrize("n,gadget_bits,special", [(1024, 20, False), (1024, 30, True), (4096, 30, True), (4096, 60, False),
                                                   (8192, 15, False)])
def test_rotations_and_client_steps(n, gadget_bits, special):
    import torch
    H = harness()
    par = params(n, gadget_bits, special)
    ctx, o = both(par)
    sk, osk = ctx.keygen(3), o.keygen(3)
    rng = np.random.default_rng(n)
    count = 3
    slots = rng.integers(0, par.p, (count, n), dtype=np.uint64)
    seeds = np.arange(count, dtype=np.uint64) + 7
    d_in = H.dev_empty(count * 2 * n)
    ctx.encrypt_batch(sk, H.to_dev(slots), H.to_dev(seeds), count, d_in)
    cts = H.export_cts(ctx, d_in, count)
    for i in range(count):
        assert np.array_equal(cts[i], o.encrypt(osk, slots[i], int(seeds[i])))
    rots = [(0, 1), (1, n // 2 - 1)]
    gk = ctx.galois_keygen(sk, rots, seed=42)
    wsb = ctx.rotate_hoisted_workspace(count)
    ws, d_hoisted = torch.empty(wsb, dtype=torch.uint8, device="cuda"), H.dev_empty(count * 2 * 2 * n)
    ctx.rotate_hoisted(gk, d_in, count, d_hoisted, ws, wsb)
    hoisted = H.export_cts(ctx, d_hoisted, count * 2).reshape(count, 2, 2 * n)
    d_slots = H.dev_empty(count * n)
    for k, (swap, step) in enumerate(rots):
        d_out = H.dev_empty(count * 2 * n)
        ctx.rotate(gk, d_in, count, (swap, step), d_out)
        got = H.export_cts(ctx, d_out, count)
        g = o.galois_elt(swap, step)
        ksk = o.galois_key(osk, g, 42)
        for i in range(count):
            want = o.perm(cts[i], g, ksk)
            assert np.array_equal(got[i], want) and np.array_equal(hoisted[i, k], want), (swap, step, i)
        if gadget_bits < 60:             # one digit of 60 bits is too noisy to decrypt
            ctx.decrypt_batch(sk, d_out, count, d_slots)
            back = H.to_host(d_slots).reshape(count, n)
            for i in range(count):
                assert np.array_equal(back[i], rotate_slots(slots[i], step, bool(swap)))


@pytest.mark.parametrize("n,n_o,n_i,batch,special", [(1024, 40, 512, 5, False), (1024, 100, 100, 3, True),
                                                     (4096, 30, 1000, 2, True), (4096, 2, 60, 3, False)])
def test_he_fc(n, n_o, n_i, batch, special):
    par = params(n, 30 if special else 20, special)
    ctx, o, plan, sk, W, x, r, got = fc_case(par, n_o, n_i, batch, list(range(batch)), seed=n_o)
    for b in range(batch):
        share = plan.unpack_share(ctx.decrypt(sk, got[b]))
        assert np.array_equal((share + r[b]) % np.uint64(par.p), plain_matvec(W, x[b], par.p))


@pytest.mark.parametrize("n,shape,batch,matrix_cores,special", [
    (1024, (9, 10, 3, 3, 11, 9), 3, True, False),
    (1024, (8, 8, 3, 3, 16, 16), 1, False, True),
    (1024, (8, 5, 3, 3, 13, 16), 2, True, True),
    (4096, (10, 12, 3, 3, 23, 20), 2, True, True),
    (4096, (6, 4, 5, 5, 20, 20), 1, False, False),
    (8192, (6, 9, 3, 3, 30, 32), 2, True, False),
])
def test_he_conv(n, shape, batch, matrix_cores, special):
    par = params(n, 30 if special else 20, special)
    _, o = both(par)
    nout = o.conv_geometry(*shape)["nout"]
    conv_case(par, shape, batch, [(b, O) for b in range(batch) for O in range(nout)], seed=n, matrix_cores=matrix_cores)
