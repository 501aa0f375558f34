"""The residue number system engine's tables on the host: the weights of a matrix's byte rows and the bounds that keep its
32- and 64-bit sums exact."""
import ctypes as C
import random

import pytest

from test_emu_rns import channel_primes, shim  # noqa: F401


def primes(shim, nr):  # noqa: F811
    k = shim.rns_primes_for(nr)
    out = [channel_primes(shim, k, residue) for residue in (3, 1)]
    for residue, base in zip((3, 1), out):
        assert len(set(base)) == k and all(p % 4 == residue for p in base)
    return out


@pytest.mark.parametrize("nr", [6, 10, 18, 36])
def test_rows_stand_for_their_constant(shim, nr):  # noqa: F811
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
def test_sums_stay_exact(shim, nr):  # noqa: F811
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
    # The way in: the sources are limbs below 2^29 + 2^8, all that are stored but the one in the bias's slot. What it leaves
    # in base B is no larger than what the products leave there.
    limbs = {6: 18, 10: 36, 18: 71, 36: 143}[nr]
    assert limbs == shim.rns_limb_sources(nr)
    fed = limbs * (384 + (2 ** 29 + 2 ** 8) / 2 ** 24 + 1) + 1
    assert fed * x_max < 2 ** 31
    assert fed * y_max * 2 ** 32 + reduction < 2 ** 63
    assert fed * y_max + half < min(b0, b1)
    # the way out: rows of radix 256 and sums from zero, base B's bytes, alpha's two and the bias
    fed = k * (384 + max(b0, b1) / 2 ** 24 + 1) + 256
    assert fed * 128 < 2 ** 31
    assert fed * 2 ** 29 < 2 ** 47  # what the pair engine reads as columns
