"""Workspace of he_fc on rings of 4096 and 8192 slots: the number of partial ciphertexts per call, and the calls that
fit the fixed scratch array."""
import numpy as np
import pytest

from paper_2105_01827_amd import binding
from tests.helpers import small_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_o", [(4096, 1000), (4096, 2048), (8192, 1000)])
def test_partial_ciphertexts_stay_bounded(n, n_o):
    """Partial ciphertexts are written and read back: a call keeps at most 32 of them per CU and one for each
    input's mask, or five an input where the inputs alone fill the CUs that often."""
    par = small_params(n)
    ctx = binding.Context(par.n, par.q, par.p, par.gadget_bits)
    plan = ctx.fc_plan(np.ones((n_o, n), np.uint64))
    ct = 2 * n * 8
    for batch in (1, 2, 3, 8, 33, 50, 64, 86, 100, 126, 130, 300, 1025, 2100):
        assert plan.workspace_bytes(batch) <= max(32 * 256 + batch, 5 * batch) * ct, batch
    # one round of the CUs in five chunks an input: it fits what a call without a workspace brings along
    if n == 4096:
        assert plan.workspace_bytes(50) <= ctx.lib.gala_he_fc_static_capacity()
