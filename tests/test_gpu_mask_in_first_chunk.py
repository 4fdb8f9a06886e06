"""Layers at n = 4096 whose masks the first chunks' workgroups build: keys modulo q and with the
special prime, against the oracle; and layers next to them whose masks have workgroups of their own."""
import dataclasses

import numpy as np
import pytest

from paper_2105_01827_amd import workloads as wl
from tests.helpers import small_params
from tests.test_gpu_parity import fc_case, plain_matvec

pytestmark = pytest.mark.gpu

CUS = 256


# (16x2048: eight rotations, the first of which is none)
@pytest.mark.parametrize("special", [False, True])
@pytest.mark.parametrize("batch,chunks,in_first", [(64, 4, True), (62, 4, True), (60, 4, False), (36, 7, False), (300, 4, False)])
def test_he_fc(batch, chunks, in_first, special):
    n, n_o, n_i = 4096, 16, 2048
    par = small_params(n)
    if special:
        par = dataclasses.replace(par, special=wl.find_prime_below(1 << 60, 2 * n))
    picks = sorted({0, 1, batch // 2, batch - 1})
    ctx, o, plan, sk, W, x, r, got = fc_case(par, n_o, n_i, batch, picks, seed=batch)
    assert plan.workspace_bytes(batch) // (batch * 2 * n * 8) - 1 == chunks

    idle = CUS - batch * chunks
    assert in_first == ((plan.G - 1) % chunks != 0 and 0 <= idle < batch and 4 * idle <= batch)
    for b in picks:
        share = plan.unpack_share(ctx.decrypt(sk, got[b]))
        assert np.array_equal((share + r[b]) % np.uint64(par.p), plain_matvec(W, x[b], par.p))
