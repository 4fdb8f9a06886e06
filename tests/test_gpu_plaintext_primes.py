"""Slot transforms on both sides of the plaintext prime's 26 bits, where they change from 32-bit to 64-bit words: the
client's steps and masked layers without a rotation (outputs apart, in place and overlapping), against the oracle."""
import numpy as np
import pytest
import torch

from paper_2105_01827_amd import workloads as wl
from tests.helpers import small_params
from tests.test_gpu_parity import both, fc_case, harness

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p_limit", [1 << 17, 1 << 26, 1 << 27, 1 << 31])
@pytest.mark.parametrize("n", [1024, 2048, 4096, 8192])
def test_encrypt_and_decrypt(n, p_limit):
    H = harness()
    par = small_params(n, p=wl.find_prime_below(p_limit, 2 * n))
    ctx, o = both(par)
    sk, osk = ctx.keygen(3), o.keygen(3)
    rng = np.random.default_rng(n)
    slots = rng.integers(0, par.p, (3, n), dtype=np.uint64)
    slots[1] = par.p - 1
    d_ct, d_slots = H.dev_empty(3 * 2 * n), H.dev_empty(3 * n)
    ctx.encrypt_batch(sk, H.to_dev(slots), H.to_dev(np.arange(3, dtype=np.uint64) + 5), 3, d_ct)
    got = H.export_cts(ctx, d_ct, 3)
    for b in range(3):
        assert np.array_equal(got[b], o.encrypt(osk, slots[b], 5 + b))
    ctx.decrypt_batch(sk, d_ct, 3, d_slots)
    torch.cuda.synchronize()
    assert np.array_equal(H.to_host(d_slots).reshape(3, n), slots)


@pytest.mark.parametrize("p_limit", [1 << 26, 1 << 27])
@pytest.mark.parametrize("n,n_o,n_i,batch", [(2048, 16, 128, 3), (2048, 3, 100, 1), (1024, 64, 16, 2)])
def test_layer_without_rotations(n, n_o, n_i, batch, p_limit):
    par = small_params(n, p=wl.find_prime_below(p_limit, 2 * n))
    ctx, o, plan, sk, W, x, r, got = fc_case(par, n_o, n_i, batch, list(range(batch)), seed=n_o)
    assert plan.G == 1
    H = harness()
    cts = np.stack([ctx.encrypt(sk, plan.pack_input(x[b]), seed=b) for b in range(batch)])
    wsb = plan.workspace_bytes(batch)
    ws, words = torch.empty(wsb, dtype=torch.uint8, device="cuda"), batch * 2 * n
    for shift in (0, 2 * n, n):              # in place, one ciphertext on, half a ciphertext on
        buf = H.dev_empty(words + 2 * n)
        d_in, d_out = buf[:words], buf[shift:shift + words]
        d_in.copy_(H.import_cts(ctx, cts))
        plan.he_fc(d_in, batch, H.to_dev(r), 17, d_out, ws, wsb)
        assert np.array_equal(H.export_cts(ctx, d_out.clone(), batch), got)


@pytest.mark.parametrize("p_limit", [1 << 27, 1 << 31])
@pytest.mark.parametrize("n,n_o,n_i", [(1024, 64, 16), (1024, 20, 300), (2048, 16, 128), (2048, 30, 500)])
def test_modulus_with_a_small_low_word(n, n_o, n_i, p_limit):
    """Under such a modulus the transforms modulo p are the narrow products too, whatever p's low word: the client's steps, and
    masks of layers without and with rotations."""
    p, q = wl.find_prime_below(p_limit, 2 * n), wl.find_prime_below(1 << 60, 2 * n)
    low = q & 0xFFFFFFFF
    assert min(low, (1 << 32) - low) <= 1 << 28 and q >= (1 << 60) - (1 << 56)
    par = wl.Params(n=n, q=q, p=p, gadget_bits=20)
    H = harness()
    ctx, o, plan, sk, W, x, r, got = fc_case(par, n_o, n_i, 3, [0, 1, 2], seed=n_o)
    osk = o.keygen(0)
    slots = np.random.default_rng(n).integers(0, p, (3, n), dtype=np.uint64)
    slots[1] = p - 1
    slots[2, ::2], slots[2, 1::2] = p - 1, 0
    d_ct, d_slots = H.dev_empty(3 * 2 * n), H.dev_empty(3 * n)
    ctx.encrypt_batch(sk, H.to_dev(slots), H.to_dev(np.arange(3, dtype=np.uint64) + 5), 3, d_ct)
    cts = H.export_cts(ctx, d_ct, 3)
    for b in range(3):
        assert np.array_equal(cts[b], o.encrypt(osk, slots[b], 5 + b)), b
    ctx.decrypt_batch(sk, d_ct, 3, d_slots)
    torch.cuda.synchronize()
    assert np.array_equal(H.to_host(d_slots).reshape(3, n), np.stack([o.decrypt(osk, c) for c in cts]))
