"""The residue number system engine's tables on the host: the weights of a matrix's byte rows, the bounds that keep its
32- and 64-bit sums exact, and moduli that its primes divide (on the CPU build, see test_emu_kernels.py)."""
import ctypes as C
import os
import random
import subprocess

import pytest

from paper_2107_13797_amd import _cabi

from test_emu_kernels import emu, words, ws, zeros  # noqa: F401
from test_emu_rns import export_n, odd_multiple, public_ctx

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("rns") / "librns_shim.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", out, os.path.join(HERE, "rns_shim.cpp")], check=True)
    return C.CDLL(out)


def primes(shim, nr):
    k = shim.rns_primes_for(nr)
    out = []
    for residue in (3, 1):
        buf = (C.c_uint32 * k)()
        assert shim.rns_primes(k, residue, buf) == k
        assert len(set(buf)) == k and all(p % 4 == residue for p in buf)
        out.append(list(buf))
    return out


@pytest.mark.parametrize("nr", [6, 10, 18, 36])
def test_rows_stand_for_their_constant(shim, nr):
    rng = random.Random(nr)
    for p in sum(primes(shim, nr), []):
        for e in [0, 1, p - 1, p // 2, p // 2 + 1, (1 << 32) % p, p - (1 << 32) % p] + [rng.randrange(p) for _ in range(5)]:
            b = (C.c_int8 * 4)()
            shim.rns_rows(nr, rng.randrange(16), e, p, b)
            x, y = b[0] + 256 * b[1], b[2] + 256 * b[3]
            assert (x + (y << 32) - e) % p == 0
            assert abs(x) <= 30931 and abs(y) <= 13822
            assert shim.rns_times256(e, p) == 256 * e % p


@pytest.mark.parametrize("nr", [6, 10, 18, 36])
def test_sums_stay_exact(shim, nr):
    """The largest residues that reproduce themselves from one product to the next, with every byte and every matrix entry
    at its bound and of the worst sign, stay within the words that hold them."""
    both = sum(primes(shim, nr), [])
    k, p = len(both) // 2, max(both)
    rows_w = [(1 << 32) % q for q in both]
    x_max, y_max = max(rows_w) // 2 + 1, (p // 2) // min(rows_w) + 1
    half = p / 2  # a centred constant; m p / 2^32 with m in 32 bits, signed

    def upper(s):
        return k * (384 + s / 2 ** 24 + 1) * y_max + 256 * y_max

    a0 = b0 = a1 = b1 = 0.0
    for _ in range(300):
        s0, z = a0 * a0 / 2 ** 32 + half, b0 * b0 / 2 ** 32 + half
        b0 = upper(s0) + half * z / 2 ** 32 + half
        a0 = upper(b0) + half
        s1 = (2 * a0 * a1 + half * s0) / 2 ** 32 + half
        w = (2 * b0 * b1 + half * z) / 2 ** 32 + half
        b1 = upper(s1) + half * (w + b0) / 2 ** 32 + half
        a1 = upper(b1) + half
    largest = max(a0, a1, b0, b1, s0, s1, z, w)
    assert largest < 2 ** 31
    sources = max(b0, b1, s0, s1)
    assert k * (384 + sources / 2 ** 24 + 1) * x_max + 256 * x_max < 2 ** 31
    reduction = 2 ** 31 * p
    assert max(2 * b0 * b1 + half * z, 2 * a0 * a1 + half * s0) + reduction < 2 ** 63
    assert upper(s1) * 2 ** 32 + half * (w + b0) + reduction < 2 ** 63
    # alpha: its approximation is off by far less than a half, its two bytes hold it
    assert 600 / 2 ** 14 + k * (1 + max(b0, b1) / 2 ** 30 * (2 ** 30 - min(both)) / 2 ** 16) / 2 ** 14 < 0.25
    assert k * max(b0, b1) / min(both) < 128 * 127
    # the multiple of s added to every value outweighs what signed coefficients can take off
    assert k * max(s0, s1) / min(both) < 256


@pytest.mark.parametrize("base,index", [(0, 0), (0, 17), (1, 0), (1, 17)])
def test_moduli_that_a_channel_prime_divides(emu, shim, base, index):  # noqa: F811
    """They have no residues modulo that prime to work with and are served by the limb arithmetic."""
    lib, bits = emu, 512
    n = odd_multiple(primes(shim, 6)[base][index], bits, 10 * base + index)
    nsq, rng = n * n, random.Random(11)
    ctx = public_ctx(lib, n, bits)
    ms, rs = [rng.randrange(n) for _ in range(2)], [rng.randrange(1, n) for _ in range(2)]
    d_c = zeros(lib, (2, bits * 9 // 128))
    w, nb = ws(lib, ctx, _cabi.OP_ENCRYPT, 2)
    assert lib.haflo_encrypt(ctx, words(lib, ms, bits // 32).p, words(lib, rs, bits // 32).p, d_c.p, 2, w.p, nb, None) == 0
    got = export_n(lib, ctx, bits, d_c, 2)
    lib.haflo_ctx_destroy(ctx)
    assert got == [(1 + m * n) * pow(r, n, nsq) % nsq for m, r in zip(ms, rs)]
