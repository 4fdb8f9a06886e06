"""Import and export against the definition of the two forms: word i of an imported polynomial is its value at
psi^(2 brev(i) + 1), psi the first x^((q-1)/2n), x = 2, 3, ..., with psi^n = -1; export gives the coefficients back."""
import numpy as np
import pytest
import torch

from paper_2105_01827_amd import binding, devmem as D, workloads as wl

pytestmark = pytest.mark.gpu


def _psi(q, n):
    for x in range(2, 1000):
        c = pow(x, (q - 1) // (2 * n), q)
        if pow(c, n, q) == q - 1:
            return c


def _value(poly, x, q):
    acc = 0
    for c in reversed(poly):
        acc = (acc * x + int(c)) % q
    return acc


@pytest.mark.parametrize("count", [1, 3])
@pytest.mark.parametrize("kind", ["random", "largest", "unreduced"])
@pytest.mark.parametrize("n", [256, 1024, 2048, 4096, 8192])
def test_import_is_evaluation_and_export_inverts_it(n, kind, count):
    p = wl.find_prime_below(1 << 20, 2 * n)
    q = wl.find_prime_below(1 << 60, 2 * n * p)
    ctx = binding.Context(n, q, p, 20)
    rng = np.random.default_rng(7)
    src = rng.integers(0, q, (count, 2 * n), dtype=np.uint64)
    if kind == "largest":
        src[:] = q - 1
    elif kind == "unreduced":        # words up to 4q - 1 are taken as their residues
        src += np.uint64(q) * rng.integers(0, 4, src.shape, dtype=np.uint64)
    dev, out = D.to_dev(src), D.dev_empty(src.size)
    ctx.ct_import(dev, count, out)
    ctx.ct_import(dev, count, dev)                   # in place
    torch.cuda.synchronize()
    got = D.to_host(out).reshape(count * 2, n)
    assert np.array_equal(got, D.to_host(dev).reshape(count * 2, n))
    assert int(got.max()) < q
    psi, logn = _psi(q, n), n.bit_length() - 1
    polys = src.reshape(count * 2, n)
    for i in [0, 1, n // 8 - 1, n // 2 + 3, n - 1]:
        x = pow(psi, 2 * int(format(i, f"0{logn}b")[::-1], 2) + 1, q)
        for k in {0, count * 2 - 1}:
            assert int(got[k, i]) == _value(polys[k], x, q), (i, k)
    ctx.ct_export(out, count, out)                   # in place
    assert np.array_equal(D.to_host(out).reshape(src.shape), src % np.uint64(q))
