"""Layers at n = 4096 whose masks the first chunks' workgroups build: dense layers and convolutions, keys modulo q and with the
special prime, against the oracle; and layers next to them whose masks have workgroups of their own.  Which of the two
a call takes shows in its workspace: a mask with a workgroup of its own leaves a partial ciphertext."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2105_01827_amd import workloads as wl
from tests import gpu_harness as H
from tests.helpers import small_params
from tests.test_gpu_parity import conv_case, fc_case, plain_conv

pytestmark = pytest.mark.gpu

N = 4096
UNWRITTEN = 0x5E


def params(special):
    par = small_params(N)
    return dataclasses.replace(par, special=wl.find_prime_below(1 << 60, 2 * N)) if special else par


def mask_has_no_partial(workspace, items, chunks):
    """The workspace of a call, filled with UNWRITTEN bytes before it, holds items x (chunks + 1) partial ciphertexts somewhere,
    at a multiple of 256 bytes: is the last of each item's unwritten, or zero in its second polynomial as a mask's is?"""
    rows = workspace.cpu().numpy().view(np.uint64).reshape(-1, 32)
    ct = 2 * N // 32

    def runs(flags, length):
        total = np.concatenate([[0], np.cumsum(flags)])
        return total[length:] - total[:-length]

    unwritten = runs(np.all(rows == np.uint64(int.from_bytes(bytes([UNWRITTEN]) * 8, "little")), axis=1), ct)
    zero = runs(np.all(rows == 0, axis=1), ct // 2)
    count = len(rows) - items * (chunks + 1) * ct + 1
    behind, own = np.ones(count, bool), np.ones(count, bool)
    for item in range(items):
        for slot in range(chunks + 1):
            at = (item * (chunks + 1) + slot) * ct
            left = unwritten[at:at + count]
            if slot < chunks:
                behind &= left == 0
                own &= left == 0
            else:
                behind &= left == ct
                own &= (left == 0) & (zero[at + ct // 2:at + ct // 2 + count] == ct // 2)
    assert behind.any() != own.any()
    return behind.any()


# 16x2048: eight rotations, the first of which is none; 500x4096: 512, 86 a chunk
@pytest.mark.parametrize("special", [False, True])
@pytest.mark.parametrize("n_o,n_i,batch,chunks,in_first", [
    (16, 2048, 64, 4, True), (16, 2048, 62, 4, True), (16, 2048, 60, 4, False), (16, 2048, 36, 7, False), (16, 2048, 300, 4, False),
    (60, 4000, 64, 4, True), (500, 4096, 41, 6, False),
])
def test_he_fc(n_o, n_i, batch, chunks, in_first, special):
    par = params(special)
    picks = [] if n_o > 16 else sorted({0, 1, batch // 2, batch - 1})
    ctx, o, plan, sk, W, x, r, got = fc_case(par, n_o, n_i, batch, picks, seed=batch)
    wsb = plan.workspace_bytes(batch)
    assert wsb // (batch * 2 * N * 8) - 1 == chunks
    for b in picks or range(batch):
        share = plan.unpack_share(ctx.decrypt(sk, got[b]))
        assert np.array_equal((share + r[b]) % np.uint64(par.p), (W @ x[b]) % np.uint64(par.p))
    d_in = H.import_cts(ctx, np.stack([ctx.encrypt(sk, plan.pack_input(x[b]), seed=b) for b in range(batch)]))
    d_out, ws = H.dev_empty(batch * 2 * N), torch.full((wsb,), UNWRITTEN, dtype=torch.uint8, device="cuda")
    plan.he_fc(d_in, batch, H.to_dev(r), 17, d_out, ws, wsb)
    assert np.array_equal(H.export_cts(ctx, d_out, batch), got)
    assert mask_has_no_partial(ws, batch, chunks) == in_first


# 64 channels of 16x16: sixteen kernel orders, four output ciphertexts an input; of 8x8: 64 and one
@pytest.mark.parametrize("special", [False, True])
@pytest.mark.parametrize("matrix_cores", [False, True])
@pytest.mark.parametrize("side,batch,chunks,in_first", [(16, 16, 4, True), (16, 8, 8, True), (16, 15, 4, False), (8, 8, 32, True)])
def test_he_conv(side, batch, chunks, in_first, matrix_cores, special):
    par = params(special)
    shape = (64, 16, 1, 1, side, side)
    nout = 4 if side == 16 else 1
    picks = sorted({(0, 0), (1, nout - 1), (batch // 2, nout // 2), (batch - 1, nout - 1)})
    ctx, o, plan, sk, K, x, r, got, cnt = conv_case(par, shape, batch, picks, seed=batch, matrix_cores=matrix_cores)
    assert plan.nout == nout
    for b in range(batch):
        share = np.zeros((64, side, side), np.uint64)
        for O in range(nout):
            plan.unpack_share(O, ctx.decrypt(sk, got[b, O]), share)
        if b in (0, batch // 2, batch - 1):
            assert np.array_equal((share + r[b]) % np.uint64(par.p), plain_conv(K, x[b], par.p)), b
    cts = np.stack([[ctx.encrypt(sk, slots, seed=1000 * b + I) for I, slots in enumerate(plan.pack_input(x[b]))] for b in range(batch)])
    d_in, d_out, wsb = H.import_cts(ctx, cts), H.dev_empty(batch * nout * 2 * N), plan.workspace_bytes(batch)
    ws = torch.full((wsb,), UNWRITTEN, dtype=torch.uint8, device="cuda")
    plan.he_conv(d_in, batch, H.to_dev(r), 3, d_out, ws, wsb)
    assert np.array_equal(H.export_cts(ctx, d_out, batch * nout).reshape(got.shape), got)
    assert mask_has_no_partial(ws, batch * nout, chunks) == in_first
