"""The first transform pass on gadget digits, which adds up products of several digits before it reduces them (digit_pass in
gala_ring_impl.h): which contexts take it, and its arithmetic on the library's constants in big integers - the results are the transform's
first three stages, and sums and results stay where the kernels have room for them.  The library keeps constants and choice to itself;
a few lines compiled against its internal header ask for them."""
import ctypes as C
import itertools
import subprocess

import pytest

from paper_2105_01827_amd import binding, build as lib_build
from tests.test_gpu_digit_pass import BITS, RINGS, parameters

READER = """
#include "gala_internal.h"
extern "C" int read_transform(const gala_ctx *c, int special, unsigned long long *m, unsigned long long *tw, unsigned long long *words) {
    const gala::NttHost &h = special ? c->ntt_P : c->ntt_q;
    gala::u64 a[gala::kDigitPassWords];
    const bool sums = gala::digit_pass_constants(h, c->gadget_bits, a);
    *m = h.mod.q;
    for (int i = 0; i < 7; ++i) tw[i] = h.tw[1 + i];
    for (int i = 0; i < gala::kDigitPassWords; ++i) words[i] = a[i];
    return sums;
}
"""
# results of the three stages in multiples of the modulus, as stated beside the kernel; the general pass has 3.5 after the third
BOUNDS = {30: (0.63, 1.4, 2.4), 31: (0.75, 1.75, 3.25)}

# the constants whose products are added up: of x4; x2 and x6; x1, x5, x3 and x7
SUMS = [(0,), (1, 3), (2, 4)] + [(c, c + 2, c + 4, c + 6) for c in (6, 7, 14, 15)]


@pytest.fixture(scope="module")
def read_transform(tmp_path_factory):
    at = tmp_path_factory.mktemp("reader")
    (at / "reader.cpp").write_text(READER)
    binding.load()
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-I", lib_build.CSRC, str(at / "reader.cpp"), lib_build.LIB,
                           "-o", str(at / "reader.so")])
    lib = C.CDLL(str(at / "reader.so"))
    lib.read_transform.argtypes = [C.c_void_p, C.c_int] + [C.POINTER(C.c_ulonglong)] * 3

    def read(par, special):
        ctx = binding.Context(par.n, par.q, par.p, par.gadget_bits, par.special)
        m, tw, words = C.c_ulonglong(), (C.c_ulonglong * 7)(), (C.c_ulonglong * 22)()
        sums = lib.read_transform(ctx.h, special, C.byref(m), tw, words)
        return bool(sums), int(m.value), list(tw), list(words)
    return read


def three_stages(x, tw, m):
    a = list(x)
    for half, blocks in ((4, 1), (2, 2), (1, 4)):
        for b in range(blocks):
            for i in range(2 * half * b, 2 * half * b + half):
                y = tw[blocks - 1 + b] * a[i + half]
                a[i], a[i + half] = (a[i] + y) % m, (a[i] - y) % m
    return a


def signed(v, bits):
    return ((v + (1 << bits - 1)) & ((1 << bits) - 1)) - (1 << bits - 1)


def halves(v):
    """the signed words of a constant: hi 2^32 + lo with the carry of lo taken into hi already"""
    return signed(v, 32), signed(v >> 32, 32)


class Pass:
    """digit_pass, with its 64-bit sums checked"""
    def __init__(self, m, words):
        self.m, self.words = m, [halves(w) for w in words]
        self.lo, self.hi = signed(m, 32), (m - signed(m, 32)) >> 32
        self.inverse = pow(m, -1, 1 << 32)

    def reduced(self, digits, constants):
        L, H = (sum(d * self.words[c][i] for d, c in zip(digits, constants)) for i in range(2))
        k = signed(L * self.inverse, 32)
        wide = abs(self.lo) > 1 << 28
        assert abs(L) < 1 << 63 and (wide or abs(L - k * self.lo) < 1 << 63)
        # what the last word needs of L - k lo, whose low half is zero: the high words one by one where it does not fit
        value = H - k * self.hi + (L - k * self.lo >> 32)
        assert (L - k * self.lo) % (1 << 32) == 0 and abs(value) + (abs(k) * self.hi) < 1 << 63
        return value

    def run(self, x):
        e = self.reduced(x[4:5], [0])
        A, B = self.reduced((x[2], x[6]), (1, 3)), self.reduced((x[2], x[6]), (2, 4))
        first = (x[0] + e, x[0] - e)
        second = (first[0] + A, first[0] - A, first[1] + B, first[1] - B)
        out = []
        for h in range(2):
            c, odd = 6 + 8 * h, (x[1], x[5], x[3], x[7])
            for i in range(2):
                s, p = self.reduced(odd, (c + i, c + i + 2, c + i + 4, c + i + 6)), second[2 * h + i]
                out += [p + s, p - s]
        return first, second, out


@pytest.mark.parametrize("special", [False, True])
@pytest.mark.parametrize("bits", BITS)
@pytest.mark.parametrize("n", RINGS)
def test_sums_of_products(read_transform, n, bits, special):
    par, top = parameters(n, bits, special), (1 << bits) - 1
    for modulus in range(2 if special else 1):
        taken, m, tw, words = read_transform(par, modulus)
        assert m == (par.special if modulus else par.q)
        the_pass = Pass(m, words)
        if not taken:        # not for nothing: digits of zeros and ones fill the words, but for what the reduction may add
            assert bits > 30
            low = [[the_pass.words[k][0] for k in terms] for terms in SUMS]
            assert bits > 31 or max(abs(sum(w for w in s if w * sign > 0)) for s in low for sign in (1, -1)) << bits >= (1 << 63) - (1 << 59)
            continue
        assert bits <= 31
        for x in itertools.chain(itertools.product((0, top), repeat=8), [(1, top, 2, top - 1, 3, top // 2, 4, top // 3)]):
            stages = the_pass.run(x)
            assert [v % m for v in stages[2]] == three_stages(x, tw, m)
            for values, bound in zip(stages, BOUNDS[max(bits, 30)]):
                assert max(map(abs, values)) <= bound * m


@pytest.mark.parametrize("bits", BITS)
def test_routes_of_the_rings(read_transform, bits):
    """digits of up to 30 bits take the sums, of 32 none, and of 31 both kinds are among the rings"""
    taken = {read_transform(parameters(n, bits, False), 0)[0] for n in RINGS}
    assert taken == ({True} if bits <= 30 else {True, False} if bits == 31 else {False})
