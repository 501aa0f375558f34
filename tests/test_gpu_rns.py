"""The RNS engine (residues modulo two sets of primes, reductions on the matrix cores) against the limb arithmetic that
serves calls whose workspace has no room for it, which is what the oracle pins: batches on both sides of the rule that
spreads an element over a block or gives 16 of them to a wavefront, with partial tiles and partial passes. Every
comparison is of all bits of all elements."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from conftest import oracle_key  # noqa: E402
from paper_2107_13797_amd import _cabi  # noqa: E402

from helpers import dev_to_ints, ints_to_dev, random_units_words, to_dev  # noqa: E402



def encrypt_in(lib, ctx, m, r, nbytes, out):
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    return lib.haflo_encrypt(ctx.handle, C.c_void_p(m.data_ptr()), C.c_void_p(r.data_ptr()), C.c_void_p(out.data_ptr()),
                             m.shape[0], C.c_void_p(ws.data_ptr()), nbytes,
                             C.c_void_p(torch.cuda.current_stream().cuda_stream))


def decrypt_in(lib, ctx, c, nbytes, out):
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    return lib.haflo_decrypt(ctx.handle, C.c_void_p(c.data_ptr()), C.c_void_p(out.data_ptr()), c.shape[0],
                             C.c_void_p(ws.data_ptr()), nbytes, C.c_void_p(torch.cuda.current_stream().cuda_stream))


def without_engine(call, need, out):
    """The call in ever smaller workspaces until it is refused; the smallest accepted one has no room for the engine."""
    best = None
    nbytes = need - 1
    while nbytes > 4096 and call(nbytes, out) == 0:
        best = out.clone()
        nbytes = nbytes * 3 // 4
    return best


@pytest.mark.parametrize("bits,counts", [
    (512, (1, 17, 4097, 12289)),
    (1024, (1, 15, 16, 12288, 12289, 65536 + 17)),
    (2048, (1, 33, 24576, 24577, 65536 + 1)),
    (4096, (1, 17, 12289)),
])
def test_rns_engine_matches_limb_arithmetic(bits, counts):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2107_13797_amd import api
    lib = api.lib()
    p, q = oracle_key(bits)
    n = p * q
    top = max(counts)
    # edges: the smallest and largest values, and randomness that is no unit or not reduced modulo n
    edge_m = [0, 1, n - 1, n // 2, 0, n - 1]
    edge_r = [1, n - 1, 2, 2 ** (bits - 1), 0, min(n + 2, 2 ** bits - 1)]
    m = to_dev(random_units_words(top, bits, bits + 1))
    r = to_dev(random_units_words(top, bits, bits + 2))
    m[:6], r[:6] = ints_to_dev(edge_m, bits // 32)[:top], ints_to_dev(edge_r, bits // 32)[:top]
    pub = api.haflo_ctx_create_public(n, bits)
    prv = api.haflo_ctx_create_private(p, q, bits)
    for count in counts:
        print("rns", bits, count, flush=True)
        mc, rc = m[:count].contiguous(), r[:count].contiguous()
        need = lib.haflo_workspace_bytes(pub.handle, _cabi.OP_ENCRYPT, count, 0)
        c, out = api.haflo_encrypt(pub, mc, rc), None
        out = torch.zeros_like(c)
        want = without_engine(lambda nb, o: encrypt_in(lib, pub, mc, rc, nb, o), need, out)
        if want is not None:
            assert torch.equal(c, want)
        for i in {0, count // 2, count - 1}:
            mi, ri = dev_to_ints(mc[i:i + 1])[0], dev_to_ints(rc[i:i + 1])[0]
            assert dev_to_ints(api.haflo_export_cipher(pub, c[i:i + 1].contiguous()))[0] == \
                (1 + mi * n) * pow(ri, n, n * n) % (n * n)
        assert torch.equal(api.haflo_encrypt(prv, mc, rc), c)
        plain = api.haflo_decrypt(prv, c)
        need = lib.haflo_workspace_bytes(prv.handle, _cabi.OP_DECRYPT, count, 0)
        want = without_engine(lambda nb, o: decrypt_in(lib, prv, c, nb, o), need, torch.zeros_like(plain))
        keep = torch.arange(count, device="cuda") != 4  # r = 0 gives no ciphertext: what it decrypts to is not defined
        if want is not None:
            assert torch.equal(plain[keep], want[keep])
        assert torch.equal(plain[keep], mc[keep])
        del c, plain, want, out
    pub.close()
    prv.close()


@pytest.mark.parametrize("bits,count", [(1024, 12800), (1024, 12816), (2048, 3001), (2048, 6160)])
def test_workspace_is_not_exceeded(bits, count):
    """Window tables of both moduli of a call end inside the workspace asked for, also where the wavefronts of a block
    do not divide the tiles: a guard area behind it keeps its contents."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2107_13797_amd import api
    lib = api.lib()
    p, q = oracle_key(bits)
    pub, prv = api.haflo_ctx_create_public(p * q, bits), api.haflo_ctx_create_private(p, q, bits)
    m = to_dev(random_units_words(count, bits, 3))
    r = to_dev(random_units_words(count, bits, 4))
    c, plain = api.haflo_encrypt(pub, m, r), torch.zeros_like(m)
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    guard = 64 << 20
    for ctx, op in ((pub, _cabi.OP_ENCRYPT), (prv, _cabi.OP_ENCRYPT), (prv, _cabi.OP_DECRYPT)):
        need = lib.haflo_workspace_bytes(ctx.handle, op, count, 0)
        ws = torch.full((need + guard,), 0x5A, dtype=torch.uint8, device="cuda")
        out = torch.zeros_like(c)
        if op == _cabi.OP_DECRYPT:
            rc = lib.haflo_decrypt(ctx.handle, C.c_void_p(c.data_ptr()), C.c_void_p(plain.data_ptr()), count,
                                   C.c_void_p(ws.data_ptr()), need, stream)
            assert rc == 0 and torch.equal(plain, m)
        else:
            rc = lib.haflo_encrypt(ctx.handle, C.c_void_p(m.data_ptr()), C.c_void_p(r.data_ptr()),
                                   C.c_void_p(out.data_ptr()), count, C.c_void_p(ws.data_ptr()), need, stream)
            assert rc == 0 and torch.equal(out, c)
        assert int((ws[need:] != 0x5A).sum()) == 0
        del ws
    pub.close()
    prv.close()


@pytest.mark.parametrize("bits", [512, 1024, 2048])
def test_powers_by_one_scalar_match_small_batches(bits):
    """A scalar of 17 bits and more over a large array goes through the residue form: the same bits as in slices that
    are too small for it, in place as well."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2107_13797_amd import api
    p, q = oracle_key(bits)
    n = p * q
    count = 8192 + 33
    pub = api.haflo_ctx_create_public(n, bits)
    c = api.haflo_encrypt(pub, to_dev(random_units_words(count, bits, 5)), to_dev(random_units_words(count, bits, 6)))
    for k in (2 ** 16, (1 << 21) + 1, 2 ** 63 - 1, -(1 << 40) - 77, 12345):
        print("scalar", bits, k, flush=True)
        got = api.haflo_scalar_mul_i64_bcast(pub, c, k)
        idx = [slice(0, 300), slice(count - 300, count)]
        for s in idx:
            assert torch.equal(got[s], api.haflo_scalar_mul_i64_bcast(pub, c[s].contiguous(), k))
        a, b = (dev_to_ints(api.haflo_export_cipher(pub, t[7:8].contiguous()))[0] for t in (c, got))
        assert b == pow(a, k, n * n)
    pub.close()


@pytest.mark.parametrize("bits,count", [(1024, 24576), (1024, 24577), (1024, 45000), (1024, 80000)])
def test_key_owner_is_not_slower_with_the_workspace_asked_for(bits, count):
    """Both sides of the rule that leaves the first stage on limbs: the same bits as in the least workspace, which is
    the limb arithmetic throughout, and no slower. (45000 and 80000 elements took 1.07 and 1.09 of its time with both
    stages in residues, 0.98 now; the bound leaves 6 % for what runs of one side differ.)"""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2107_13797_amd import api
    lib = api.lib()
    p, q = oracle_key(bits)
    prv = api.haflo_ctx_create_private(p, q, bits)
    m, r = to_dev(random_units_words(count, bits, 8)), to_dev(random_units_words(count, bits, 9))
    sizes = [f(prv.handle, _cabi.OP_ENCRYPT, count, 0) for f in (lib.haflo_workspace_bytes, lib.haflo_workspace_bytes_least)]
    ws = torch.empty(max(sizes), dtype=torch.uint8, device="cuda")
    out = [torch.zeros((count, prv.cipher_words), dtype=torch.int32, device="cuda") for _ in sizes]
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    best = [1e9, 1e9]
    for _ in range(9):
        for i, nbytes in enumerate(sizes):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            assert lib.haflo_encrypt(prv.handle, C.c_void_p(m.data_ptr()), C.c_void_p(r.data_ptr()),
                                     C.c_void_p(out[i].data_ptr()), count, C.c_void_p(ws.data_ptr()), nbytes, stream) == 0
            b.record()
            b.synchronize()
            best[i] = min(best[i], a.elapsed_time(b))
    print("owner", bits, count, best, flush=True)
    prv.close()
    assert torch.equal(out[0], out[1])
    assert best[0] < 1.04 * best[1]
