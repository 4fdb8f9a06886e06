"""The Perm kernel at n = 1024 and 4096 in launches of more than two wavefronts per SIMD (131072 threads), where it is
another instantiation than in the smaller launches of the other tests: with weights, on the matrix-core product's blocks
of eight, and on whole ciphertexts, against the oracle."""
import numpy as np
import pytest

from oracle.oracle import Oracle
from paper_2105_01827_amd import binding
from tests import gpu_harness as H
from tests.helpers import rotate_slots, small_params
from tests.test_gpu_parity import conv_case, fc_case, plain_matvec

pytestmark = pytest.mark.gpu

FEW_THREADS = 256 * 4 * 2 * 64      # CUs, SIMDs, wavefronts per SIMD, threads


# `few`: on the other side of the limit; both ways of handing chunks to workgroups (multiples of eight, and not)
@pytest.mark.parametrize("n,n_o,n_i,batch,few,eighths", [
    (1024, 100, 500, 20, False, True), (1024, 8, 1000, 300, False, False), (1024, 100, 500, 2, True, True),
    (4096, 40, 4000, 8, False, True), (4096, 40, 4000, 12, False, False), (4096, 40, 4000, 7, True, True),
])
def test_he_fc(n, n_o, n_i, batch, few, eighths):
    par = small_params(n)
    picks = sorted({0, 1, batch // 2, batch - 1})
    ctx, o, plan, sk, W, x, r, got = fc_case(par, n_o, n_i, batch, picks, seed=n_o)
    chunks = plan.workspace_bytes(batch) // (batch * 2 * n * 8) - 1
    assert (batch * (chunks + 1) * n // 8 <= FEW_THREADS) == few and (chunks % 8 == 0) == eighths
    for b in picks:
        share = plan.unpack_share(ctx.decrypt(sk, got[b]))
        assert np.array_equal((share + r[b]) % np.uint64(par.p), plain_matvec(W, x[b], par.p))


# every output ciphertext takes at least a workgroup for its rotations and one for its mask
@pytest.mark.parametrize("matrix_cores", [False, True])
@pytest.mark.parametrize("n,shape,batch", [(1024, (60, 20, 3, 3, 8, 7), 140), (4096, (60, 20, 3, 3, 16, 14), 70)])
def test_he_conv(n, shape, batch, matrix_cores):
    par = small_params(n)
    nout = Oracle(par.n, par.q, par.p, par.gadget_bits).conv_geometry(*shape)["nout"]
    assert 2 * batch * nout * n // 8 > FEW_THREADS
    conv_case(par, shape, batch, [(b, O) for b in (0, batch // 2, batch - 1) for O in (0, nout - 1)], seed=n,
              matrix_cores=matrix_cores)


@pytest.mark.parametrize("n,count", [(1024, 1100), (4096, 300)])
def test_rotate(n, count):
    assert count * n // 8 > FEW_THREADS
    par = small_params(n)
    ctx, o = binding.Context(par.n, par.q, par.p, par.gadget_bits), Oracle(par.n, par.q, par.p, par.gadget_bits)
    sk, osk = ctx.keygen(3), o.keygen(3)
    rng = np.random.default_rng(n)
    cts = rng.integers(0, par.q, (count, 2 * n), dtype=np.uint64)
    slots = rng.integers(0, par.p, n, dtype=np.uint64)
    cts[count - 1] = ctx.encrypt(sk, slots, seed=5)
    rot = (1, n // 2 - 3)
    gk = ctx.galois_keygen(sk, [rot], seed=42)
    d_in, d_out = H.import_cts(ctx, cts), H.dev_empty(count * 2 * n)
    ctx.rotate(gk, d_in, count, rot, d_out)
    got = H.export_cts(ctx, d_out, count)
    g = o.galois_elt(*rot)
    ksk = o.galois_key(osk, g, 42)
    for i in (0, 1, count // 2, count - 1):
        assert np.array_equal(got[i], o.perm(cts[i], g, ksk)), i
    assert np.array_equal(ctx.decrypt(sk, got[count - 1]), rotate_slots(slots, rot[1], True))
