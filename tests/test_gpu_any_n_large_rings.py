"""The any-n kernels at n = 4096 and 8192 (512 and 1024 threads a polynomial), for the parameters the rings' own kernels
do not take: q or P from 2^60 on, and n = 8192 with a special prime.  Against the oracle."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2105_01827_amd import binding, workloads as wl
from tests import gpu_harness as H
from tests.helpers import rotate_slots, small_params
from tests.test_gpu_parity import both, conv_case, fc_case, plain_matvec

pytestmark = pytest.mark.gpu


def params(kind, n):
    par = small_params(n, gadget_bits=20 if kind == "wide q" else 30)
    if kind == "wide q":
        return dataclasses.replace(par, q=wl.find_prime_below(1 << 61, 2 * n * par.p))
    return dataclasses.replace(par, special=wl.find_prime_below(1 << 61 if kind == "wide P" else par.q, 2 * n))


KINDS = [("wide q", 4096), ("wide q", 8192), ("wide P", 4096), ("special prime", 8192)]


@pytest.mark.parametrize("kind,n", KINDS)
def test_rotations_and_client_steps(kind, n):
    par = params(kind, n)
    assert (par.q >> 60 if kind == "wide q" else 1) and (par.special >> 60 if kind == "wide P" else 1)
    ctx, o = both(par)
    sk, osk = ctx.keygen(3), o.keygen(3)
    rng = np.random.default_rng(n)
    count = 3
    cts = rng.integers(0, par.q, (count, 2 * n), dtype=np.uint64)
    assert np.array_equal(H.export_cts(ctx, H.import_cts(ctx, cts), count), cts)
    slots = rng.integers(0, par.p, (count, n), dtype=np.uint64)
    d_in, d_slots = H.dev_empty(count * 2 * n), H.dev_empty(count * n)
    ctx.encrypt_batch(sk, H.to_dev(slots), H.to_dev(np.arange(count, dtype=np.uint64) + 7), count, d_in)
    cts = H.export_cts(ctx, d_in, count)
    for i in range(count):
        assert np.array_equal(cts[i], o.encrypt(osk, slots[i], 7 + i))
    rots = [(0, 1), (1, n // 2 - 1)]
    gk = ctx.galois_keygen(sk, rots, seed=42)
    wsb = ctx.rotate_hoisted_workspace(count)
    ws, d_hoisted = torch.empty(wsb, dtype=torch.uint8, device="cuda"), H.dev_empty(count * 2 * 2 * n)
    ctx.rotate_hoisted(gk, d_in, count, d_hoisted, ws, wsb)
    hoisted = H.export_cts(ctx, d_hoisted, count * 2).reshape(count, 2, 2 * n)
    for k, (swap, step) in enumerate(rots):
        d_out = H.dev_empty(count * 2 * n)
        ctx.rotate(gk, d_in, count, (swap, step), d_out)
        got = H.export_cts(ctx, d_out, count)
        g = o.galois_elt(swap, step)
        ksk = o.galois_key(osk, g, 42)
        assert np.array_equal(gk.export((swap, step)), ksk)
        ctx.decrypt_batch(sk, d_out, count, d_slots)
        back = H.to_host(d_slots).reshape(count, n)
        for i in range(count):
            want = o.perm(cts[i], g, ksk)
            assert np.array_equal(got[i], want) and np.array_equal(hoisted[i, k], want), (swap, step, i)
            assert np.array_equal(back[i], rotate_slots(slots[i], step, bool(swap)))


@pytest.mark.parametrize("kind,n", KINDS)
@pytest.mark.parametrize("n_o,n_i,batch", [(30, 1000, 2), (2, 60, 3)])
def test_he_fc(kind, n, n_o, n_i, batch):
    par = params(kind, n)
    ctx, o, plan, sk, W, x, r, got = fc_case(par, n_o, n_i, batch, list(range(batch)), seed=n_o)
    for b in range(batch):
        share = plan.unpack_share(ctx.decrypt(sk, got[b]))
        assert np.array_equal((share + r[b]) % np.uint64(par.p), plain_matvec(W, x[b], par.p))


@pytest.mark.parametrize("kind,n", KINDS)
@pytest.mark.parametrize("batch", [1, 2])
def test_he_conv(kind, n, batch):
    matrix_cores = batch == 2 and kind != "wide q"      # the matrix-core product takes q below 2^60
    conv_case(params(kind, n), (10, 12, 3, 3, 23, 20), batch, [(b, 0) for b in range(batch)], seed=n, matrix_cores=matrix_cores)
