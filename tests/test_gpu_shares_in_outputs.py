"""Layers without a rotation whose shares r lie in the output buffer: every share is read before an output is written,
as in layers with rotations, whose outputs are written by a launch of their own."""
import numpy as np
import pytest
import torch

from paper_2105_01827_amd import binding
from tests.gpu_harness import dev_empty, to_dev
from tests.helpers import small_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["first", "last"])
@pytest.mark.parametrize("n,batch", [(1024, 5000), (2048, 3000), (4096, 1500), (8192, 700)])
def test_he_fc_with_shares_in_the_output(n, batch, where):
    # more inputs than the chip holds workgroups: the last ones start after the first outputs are there
    par, n_o = small_params(n), 16
    ctx = binding.Context(par.n, par.q, par.p, par.gadget_bits)
    rng = np.random.default_rng(n)
    plan = ctx.fc_plan(rng.integers(0, par.p, (n_o, 64), dtype=np.uint64))
    assert plan.G == 1
    d_in = to_dev(rng.integers(0, par.q, (batch, 2 * n), dtype=np.uint64)).reshape(-1)
    d_r = to_dev(rng.integers(0, par.p, (batch, n_o), dtype=np.uint64)).reshape(-1)
    d_out, d_want = dev_empty(batch * 2 * n), dev_empty(batch * 2 * n)
    wsb = plan.workspace_bytes(batch)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    plan.he_fc(d_in, batch, d_r, 17, d_want, ws, wsb)
    at = 0 if where == "first" else batch * 2 * n - d_r.numel()
    d_out[at:at + d_r.numel()].copy_(d_r)
    plan.he_fc(d_in, batch, d_out[at:at + d_r.numel()], 17, d_out, ws, wsb)
    assert torch.equal(d_out, d_want)
