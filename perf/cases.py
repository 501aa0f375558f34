"""The work that users of the Paillier operator path have it do, as timed cases.

Every case is one pass through the public entry points of `paper_2107_13797_amd.api` on operands that are
resident on the GPU, the way the parties of a federated logistic regression call them: encoding and
decoding of fixed-point values, encryption with the public key and by the key owner, decryption,
aggregation of ciphertext vectors, scaling by plaintext scalars, and the two ciphertext matrix-vector
products. Key sizes are 1024, 2048 and 4096 bits; batches reach from one minibatch's handful of values to
chip-filling vectors. All results are integers (or exact conversions of integers), so every case is exact.
"""
import functools
import math

import torch

from paper_2107_13797_amd import api, synth

SCALE = 24    # fraction bits of residuals and weights
SCALE_X = 16  # fraction bits of feature matrices

_LISTED = [
    # a minibatch of residuals quantised before encryption and decoded values read back after decryption:
    # the smallest call, launches and memory traffic only
    dict(name="codec_1024_b4096", op="codec", bits=1024, count=4096),
    # the operator mix's encryption: a small batch at the paper's key size, bound by the length of one chain
    dict(name="encrypt_1024_b1024", op="encrypt", bits=1024, count=1024),
    # the residual vector of one gradient step at the headline key size, a batch that fills the chip
    dict(name="encrypt_2048_b65536", op="encrypt", bits=2048, count=65536),
    # a ragged mid-sized batch of residuals at the largest key size
    dict(name="encrypt_4096_b3001", op="encrypt", bits=4096, count=3001),
    # a party that holds the key encrypts its weight vector (homogeneous LR)
    dict(name="encrypt_owner_2048_b20001", op="encrypt_owner", bits=2048, count=20001),
    # the arbiter decrypts the operator mix's results
    dict(name="decrypt_1024_b3072", op="decrypt", bits=1024, count=3072),
    # the arbiter decrypts one forward pass
    dict(name="decrypt_2048_b16384", op="decrypt", bits=2048, count=16384),
    # the arbiter decrypts one gradient at the largest key size: a few elements, latency only
    dict(name="decrypt_4096_b64", op="decrypt", bits=4096, count=64),
    # encrypted gradient X^T [[d]]: minibatch at the paper's key size, and a whole step at the headline size
    dict(name="gradient_1024_4096x32", op="gradient", bits=1024, rows=4096, cols=32),
    dict(name="gradient_2048_65536x32", op="gradient", bits=2048, rows=65536, cols=32),
    # encrypted forward pass X [[w]] over a sparse feature matrix
    dict(name="forward_2048_16384x256", op="forward", bits=2048, rows=16384, cols=256),
    # homogeneous LR: the coordinator weights a party's ciphertext vector and adds it to another one
    dict(name="aggregate_2048_b50000", op="aggregate", bits=2048, count=50000),
]


def listed():
    return [dict(c) for c in _LISTED]


# ---------------------------------------------------------------------------------------------------
# what a pass cannot do without


def _mads(limbs):
    """32-bit multiply-adds of one modular product on `limbs` 32-bit words (product and reduction)."""
    return 2 * limbs * limbs + limbs


def _elements(case):
    return case["count"] if "count" in case else case["rows"]


def work(case):
    """Bytes: inputs read once, outputs written once. Flops: two per 32-bit multiply-add of the modular
    products of the textbook form of the operator (one product per exponent bit, or per non-zero digit)."""
    bits, n = case["bits"], _elements(case)
    lp, lc = bits // 32, bits // 16
    plain, cipher = 4 * lp, 4 * (bits * 9 // 128)  # a stored ciphertext holds 29 bits of each 32
    op = case["op"]
    if op == "codec":
        return dict(bytes=n * (4 + plain + plain + 16), flops=n * 2 * lp)
    if op == "encrypt":
        return dict(bytes=n * (2 * plain + cipher), flops=2 * n * bits * _mads(lc))
    if op == "encrypt_owner":  # half-length exponents modulo both prime squares
        return dict(bytes=n * (2 * plain + cipher), flops=2 * n * 2 * (bits // 2) * _mads(lc // 2))
    if op == "decrypt":
        return dict(bytes=n * (cipher + plain), flops=2 * n * 2 * (bits // 2) * _mads(lc // 2))
    if op == "aggregate":
        return dict(bytes=n * 3 * cipher, flops=2 * n * (SCALE - 3 + 1) * _mads(lc))
    rows, cols = case["rows"], case["cols"]
    if op == "gradient":  # two digits of an entry
        return dict(bytes=rows * cipher + 4 * rows * cols + cols * cipher, flops=2 * 2 * rows * cols * _mads(lc))
    if op == "forward":  # 30 % of the entries, two digits each
        return dict(bytes=cols * cipher + 4 * rows * cols + rows * cipher,
                    flops=int(2 * 2 * 0.3 * rows * cols) * _mads(lc))
    raise ValueError(op)


def tolerance(case):
    return "exact"


# ---------------------------------------------------------------------------------------------------
# further cases of the same ranges


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


_COUNTS = {  # smallest and largest batch of an element-wise operator
    "codec": (16, 1000000),
    "encrypt": (1, 65536),
    "encrypt_owner": (1, 100000),
    "decrypt": (1, 100000),
    "aggregate": (1, 100000),
}


def draw(rng):
    """One more case: operator, key size and shape drawn over their ranges, none above the largest listed one."""
    limit = max(work(c)["flops"] for c in _LISTED)
    while True:
        op = rng.choice(["codec", "encrypt", "encrypt_owner", "decrypt", "aggregate", "gradient", "forward"])
        case = dict(op=op, bits=rng.choice([1024, 2048, 4096]))
        if op in _COUNTS:
            case["count"] = _log_int(rng, *_COUNTS[op])
        elif op == "gradient":
            case["rows"], case["cols"] = _log_int(rng, 64, 65536), _log_int(rng, 1, 64)
        else:
            case["rows"], case["cols"] = _log_int(rng, 64, 65536), _log_int(rng, 1, 256)
        if work(case)["flops"] <= limit:
            return case


# ---------------------------------------------------------------------------------------------------
# operands and the pass itself


@functools.lru_cache(maxsize=None)
def _key(bits):
    return api.haflo_keygen(bits, synth.BASE_SEED + bits)


def _units(gen, count, bits):
    """Encryption randomness: uniform below 2^(bits-1), coprime to n except with negligible probability."""
    words = torch.randint(-2 ** 31, 2 ** 31, (count, bits // 32), dtype=torch.int32, device="cuda", generator=gen)
    words[:, -1] &= 0x7FFFFFFF
    return words


def prepare(case, seed):
    op, bits, n = case["op"], case["bits"], _elements(case)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    p, q = _key(bits)
    state = dict(op=op)
    if op in ("encrypt", "aggregate", "gradient", "forward"):  # the parties without the private key
        state["ctx"] = ctx = api.haflo_ctx_create_public(p * q, bits)
    else:
        state["ctx"] = ctx = api.haflo_ctx_create_private(p, q, bits)
    sigma = 0.1 if op == "forward" else (0.05 if op == "aggregate" else 0.25)
    values = torch.randn(case["cols"] if op == "forward" else n, device="cuda", generator=gen) * sigma
    if op == "codec":
        state["values"] = values
        return state
    state["plain"] = plain = api.haflo_encode_f32(ctx, values, SCALE)
    state["r"] = r = _units(gen, plain.shape[0], bits)
    if op in ("encrypt", "encrypt_owner"):
        return state
    # ciphertexts as a party receives them; made by the key owner, which is the quicker way to the same bits
    owner = ctx if op == "decrypt" else api.haflo_ctx_create_private(p, q, bits)
    state["c"] = api.haflo_encrypt(owner, plain, r)
    if op == "aggregate":
        other = torch.randn(n, device="cuda", generator=gen) * sigma
        state["acc"] = api.haflo_encrypt(owner, api.haflo_encode_f32(owner, other, SCALE), _units(gen, n, bits))
        state["weight"] = (1 << (SCALE - 3)) + 1  # an instance share as a fixed-point scalar
    if op in ("gradient", "forward"):
        x = torch.randn((case["rows"], case["cols"]), device="cuda", generator=gen)
        if op == "forward":  # sparse features in (-1, 1)
            x = torch.rand(x.shape, device="cuda", generator=gen) * 2 - 1
            x = torch.where(torch.rand(x.shape, device="cuda", generator=gen) < 0.7, torch.zeros_like(x), x)
        state["x"] = api.haflo_encode_exponents_f32(x.contiguous(), SCALE_X)
    if owner is not ctx:
        owner.close()
    return state


def run(state):
    op, ctx = state["op"], state["ctx"]
    if op == "codec":
        plain = api.haflo_encode_f32(ctx, state["values"], SCALE)
        quantised, values = api.haflo_decode(ctx, plain, SCALE)
        return plain, quantised, values
    if op in ("encrypt", "encrypt_owner"):
        return api.haflo_encrypt(ctx, state["plain"], state["r"])
    if op == "decrypt":
        return api.haflo_decrypt(ctx, state["c"])
    if op == "aggregate":
        weighted = api.haflo_scalar_mul_i64_bcast(ctx, state["c"], state["weight"])
        return api.haflo_add(ctx, weighted, state["acc"])
    return api.haflo_cipher_matvec(ctx, 0 if op == "gradient" else 1, state["c"], state["x"])
