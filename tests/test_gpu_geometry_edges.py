"""Batch and column counts on both sides of the lines at which a kernel takes another geometry on the 256 compute units."""
import numpy as np
import pytest
import torch

from helpers import dev_to_ints, random_units_words, to_dev
from test_gpu_parity import XTD_METHODS, api, context, xtd_method  # noqa: F401 (api is a fixture)

pytestmark = pytest.mark.gpu


def plain_words(count, bits, seed):
    """Random messages below n as 32-bit words (the top bit of n is set)."""
    w = np.random.default_rng(seed).integers(0, 2 ** 32, size=(count, bits // 32), dtype=np.uint64).astype(np.uint32)
    w[:, -1] &= 0x7FFFFFFF
    return w


@pytest.mark.parametrize("bits,cols", [(1024, 42), (1024, 43), (1024, 128), (1024, 129), (2048, 42), (2048, 43), (4096, 43)])
def test_bucket_chains(api, bits, cols):
    """The folds after the bucket rounds on a wavefront per pair and on groups of lanes: X^T [[d]] equals the table method's
    and decrypts to the exact sums."""
    ctx, sk = context(api, bits)
    rows, n = 90, sk.public.n
    X = np.random.default_rng(cols).integers(-2 ** 31, 2 ** 31, size=(rows, cols), dtype=np.int64).astype(np.int32)
    m = plain_words(rows, bits, 5)
    c = api.haflo_encrypt(ctx, to_dev(m), to_dev(random_units_words(rows, bits, 6)))
    outs = {}
    for method in XTD_METHODS:
        with xtd_method(api, ctx, method):
            outs[method] = api.haflo_cipher_matvec(ctx, 0, c, to_dev(X)).clone()
    assert torch.equal(outs["tables"], outs["buckets"])
    values = dev_to_ints(to_dev(m))
    got = dev_to_ints(api.haflo_decrypt(ctx, outs["buckets"]))
    assert got == [sum(int(x) * v for x, v in zip(X[:, j], values)) % n for j in range(cols)]


# 8 and 16 elements to a block of the shared-matrix kernel, partial tiles of 32, the last full launch of that kernel, one
# and two sets of 16 to a wavefront, and the counts one above each
@pytest.mark.parametrize("bits,counts", [
    (1024, (1, 7, 8, 9, 17, 31, 33, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 16384, 16385, 32769, 49153)),
    (2048, (1, 9, 17, 33, 1024, 1025, 2048, 2049, 4096, 4097, 8193, 16385, 24577)),
    (4096, (1, 9, 17, 1024, 1025, 2048, 2049, 3001)),
])
def test_powers_by_count(api, bits, counts):
    """Encryption with the public key only, with the private key and decryption agree at every count: the two encryptions run
    r^n on different moduli, so on different geometries, and the first and last ciphertexts equal Python's."""
    ctx, sk = context(api, bits)
    n = sk.public.n
    public = api.haflo_ctx_create_public(n, bits)
    for count in counts:
        m, r = plain_words(count, bits, count), random_units_words(count, bits, count + 1)
        dm, dr = to_dev(m), to_dev(r)
        own = api.haflo_encrypt(ctx, dm, dr)
        c = api.haflo_encrypt(public, dm, dr)
        assert torch.equal(api.haflo_export_cipher(ctx, own), api.haflo_export_cipher(public, c)), count
        assert torch.equal(api.haflo_decrypt(ctx, c), dm), count
        ends = [0, count - 1]
        got = dev_to_ints(api.haflo_export_cipher(public, c)[ends].contiguous())
        for g, mi, ri in zip(got, dev_to_ints(dm[ends].contiguous()), dev_to_ints(dr[ends].contiguous())):
            assert g == (1 + mi * n) * pow(ri, n, n * n) % (n * n), count
    public.close()
