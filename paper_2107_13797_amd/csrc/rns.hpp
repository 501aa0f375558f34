// Geometry and host-built tables of the residue-number-system (RNS) engine: exponentiation modulo s^2 on pairs of
// residues modulo s (x0 + s x1), where every half is held by its residues modulo two sets of 30-bit primes and
// the Montgomery reductions are constant integer matrices applied to the residues' bytes on the matrix cores
// (kernels_rns.hip has the arithmetic). Host code only builds tables here; sizes are shared with the kernels.
//
// Base A: k primes a_i, all 3 modulo 4; base B: k primes b_j, all 1 modulo 4; all between 2^30 - 15465 and 2^30 - 9700,
// so that 2^32 mod p = 4 (2^30 - p) lies between 38844 and 61860 (Matrix says why). M_A, M_B are their products; M_A is
// the Montgomery radix. Residues are signed and not reduced to one representative: below 2.02 x 10^9 in absolute value.
// Four lanes hold an element; a lane keeps `regs` residues of each base and half of the pair: channel
// slot 4 i + g in register i of lane group g (lane / 16).
#pragma once
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "hostbig.hpp"

namespace haflo {
namespace rns {

constexpr uint32_t kOmega = 0x00808080u;     // the lower bytes are fed to the signed matrix product as byte - 128
constexpr int kStart = 1 << 23;              // where the second byte row's sums start: 2^31 added to every column
constexpr int kOffset = 256;                 // multiple of s added to every reduced value, so that none is negative
constexpr uint32_t kTop = (1u << 30) - 9700; // the primes lie below

// registers per lane, base and half for a modulus of `nl` 29-bit limbs, 0: no such engine
constexpr int regs_for(int nl) { return nl == 18 ? 6 : nl == 36 ? 10 : nl == 72 ? 18 : nl == 144 ? 36 : 0; }
// primes per base: 30 k bits exceed the modulus's bits by 28, 26, 22 and 14
constexpr int primes_for(int nr) { return nr == 6 ? 18 : nr == 10 ? 35 : nr == 18 ? 69 : nr == 36 ? 137 : 0; }
constexpr int slots(int nr) { return 4 * nr; }
// tiles of 16 byte rows (4 slots) that hold the primes, and those that hold the limbs of a value
constexpr int tiles(int nr) { return (primes_for(nr) + 3) / 4; }
constexpr int limb_tiles(int nr) { return nr == 36 ? 36 : tiles(nr); }
// The slots of the matrix products' two extra source values, in lane groups of the last register: the multiple of M_B to
// subtract, and the constant 1. The first one's lane group has no prime in the last tile either: there the matrix from
// base B to base A has the row that sums what the multiple is the rounded quotient of.
constexpr int alpha_group(int nr) { return nr == 10 ? 3 : nr == 18 ? 1 : 2; }
constexpr int bias_group(int nr) { return nr == 10 ? 2 : 3; }
constexpr int alpha_slot(int nr) { return 4 * nr - 4 + alpha_group(nr); }
constexpr int bias_slot(int nr) { return 4 * nr - 4 + bias_group(nr); }
constexpr int alpha_row(int nr) { return 4 * tiles(nr) - 4 + alpha_group(nr); }
// what is added to that sum of (rho_j - kOmega) / 2^16 before the division by 2^14: half of it, kOmega's share, and less
// what the columns start from
constexpr uint32_t alpha_round(int nr) { return (1u << 13) + (uint32_t)primes_for(nr) * 257 / 2 - (uint32_t)kStart * 256; }
// A tile's fragments: nr / 4 of 64 source bytes per row and, unless nr is a multiple of 4, one of 32. Of the last tile with 18 registers only the
// first 4 rows are kept (8 of the matrix to base A; its other slots have no prime): both matrices of a 2048-bit modulus
// then fit the 160 KB of LDS.
constexpr int full_blocks(int nr) { return nr / 4; }
constexpr int last_rows(int nr, int matrix) { return nr == 18 ? 4 + 4 * matrix : 16; }
constexpr int tile_bytes(int nr, int rows) { return full_blocks(nr) * rows * 64 + (nr % 4 ? rows * 32 : 0); }
constexpr int lds_matrix_bytes(int nr, int matrix) {
  return (tiles(nr) - 1) * tile_bytes(nr, 16) + tile_bytes(nr, last_rows(nr, matrix));
}
constexpr int lds_matrices_bytes(int nr) { return lds_matrix_bytes(nr, 0) + lds_matrix_bytes(nr, 1); }
constexpr int in_matrix_bytes(int nr) { return tiles(nr) * tile_bytes(nr, 16); }
constexpr int out_matrix_bytes(int nr) { return limb_tiles(nr) * tile_bytes(nr, 16); }
// an element in memory by itself: the quads of x0's and x1's registers, of both bases, for four lanes
constexpr int item_words(int nr) { return 2 * (2 * (nr / 4) + (nr % 4 ? 1 : 0)) * 4 * 4; }
// constants of a slot: base A {p, -1/p, e, 0}, base B {p, -1/p, e, 0} for products and {p, -1/p, kappa, -e} for sums
constexpr int cst_bytes(int nr) { return 3 * slots(nr) * 16; }

// Device layout: [A -> B][B -> A][constants of A][of B][of B] as the kernel copies them to LDS, then, with all rows,
// [limbs -> B][B -> limbs]
constexpr int lds_bytes(int nr) { return lds_matrices_bytes(nr) + cst_bytes(nr); }
constexpr int table_bytes(int nr) { return lds_bytes(nr) + in_matrix_bytes(nr) + out_matrix_bytes(nr); }

inline uint32_t mulmod(uint32_t a, uint32_t b, uint32_t p) { return (uint32_t)((uint64_t)a * b % p); }
// v mod p for two channel primes, which differ by less than either
inline uint32_t prime_mod(uint32_t v, uint32_t p) { return v < p ? v : v - p; }
// 256 v mod p for the channel primes, all just below 2^30
inline uint32_t times256(uint32_t v, uint32_t p) {
  const uint64_t t = (uint64_t)v << 8;
  const uint32_t r = (uint32_t)(t - (t >> 30) * p);
  return r < p ? r : r - p;
}
inline uint32_t powmod(uint32_t a, uint64_t e, uint32_t p) {
  uint32_t r = 1 % p;
  for (a %= p; e; e >>= 1, a = mulmod(a, a, p))
    if (e & 1) r = mulmod(r, a, p);
  return r;
}
inline uint32_t invmod(uint32_t a, uint32_t p) { return powmod(a, p - 2, p); }
// Miller-Rabin with bases 2, 3, 5, 7: exact below 3.2 x 10^9
inline bool is_prime30(uint32_t n) {
  for (uint32_t d : {2u, 3u, 5u, 7u, 11u, 13u})
    if (n % d == 0) return n == d;
  uint32_t d = n - 1;
  int s = 0;
  while (!(d & 1)) d >>= 1, ++s;
  for (uint32_t b : {2u, 3u, 5u, 7u}) {
    uint32_t x = powmod(b, d, n);
    bool ok = x == 1 || x == n - 1;
    for (int i = 1; i < s && !ok; ++i) {
      x = mulmod(x, x, n);
      ok = x == n - 1;
    }
    if (!ok) return false;
  }
  return true;
}
// the signed number next to zero that v stands for modulo p, as a word
inline uint32_t centred(uint32_t v, uint32_t p) { return v > p / 2 ? v - p : v; }
// the k largest primes below kTop of a residue class, k <= 137; found once per process
inline std::vector<uint32_t> primes(int k, uint32_t residue_mod_4) {
  const auto find = [](uint32_t residue) {
    std::vector<uint32_t> r;
    for (uint32_t c = kTop / 4 * 4 - 4 + residue; (int)r.size() < primes_for(36); c -= 4)
      if (is_prime30(c)) r.push_back(c);
    return r;
  };
  static const std::vector<uint32_t> one = find(1), three = find(3);
  const std::vector<uint32_t>& all = residue_mod_4 == 1 ? one : three;
  return std::vector<uint32_t>(all.begin(), all.begin() + k);
}
// the inverses of the channel primes v modulo p (not among them), one inversion for all of them; *prod: the product of v
inline std::vector<uint32_t> inverses(const std::vector<uint32_t>& v, uint32_t p, uint32_t* prod) {
  std::vector<uint32_t> r(v.size());
  uint32_t acc = 1;
  for (size_t i = 0; i < v.size(); ++i) {
    r[i] = acc;
    acc = mulmod(acc, prime_mod(v[i], p), p);
  }
  *prod = acc;
  uint32_t inv = invmod(acc, p);
  for (size_t i = v.size(); i-- > 0;) {
    r[i] = mulmod(r[i], inv, p);
    inv = mulmod(inv, prime_mod(v[i], p), p);
  }
  return r;
}
inline Big product(const std::vector<uint32_t>& v) {
  Big r(1);
  for (uint32_t p : v) r = Big::mul(r, Big((uint64_t)p));
  return r;
}

// Matrix with byte entries: four rows for a destination slot, the four bytes of a source slot as columns. A fragment
// holds, as one wavefront reads it for v_mfma_i32_16x16x64_i8 (of the last block 8 bytes per lane), row 4 g + v of its
// tile for row v of slot 4 tile + g, and in bytes 4 c + u of lane group g byte u of slot 4 (4 block + c) + g.
//
// A constant E modulo p is written in the rows as e0 + 2^8 e1 + 2^32 (e2 + 2^8 e3) modulo p: with w = 2^32 mod p between
// 38844 and 61860, the quotient of E, centred, by w is e2 + 2^8 e3, at most 13822, and the remainder, centred, e0 + 2^8 e1,
// at most 30931. The four sums that a lane gets for a slot are then, after two shifts and additions, the lower and the
// upper word of a 64-bit number for the Montgomery reduction. What that reduction leaves is fed to the next product as it
// is; with 137 sources, whose lower bytes are at most 128 (alpha's two are below 128, the bias is 1), the largest values
// that reproduce themselves are
//   halves in base B  x0 1.52, x1 1.90, z 1.08, w 2.02 (x 10^9); base A: x0 1.45, x1 1.49, sigma 1.03 and 1.66
//   lower word        137 (384 + 1.90 x 10^9 / 2^24) 30931 + 256 x 30931 = 0.99 x 2^31: with the start at 2^31 it is not
//                     negative as a 32-bit number
//   upper word        137 (384 + 1.66 x 10^9 / 2^24) 13822 + 256 x 13822 = 0.92 x 10^9
//   products          x0 y1 + x1 y0 + e z + m p, the largest 64-bit sum, 0.94 x 2^63
class Matrix {
 public:
  Matrix(int nr, int tiles_, int last_rows_)
      : nr_(nr), tiles_n_(tiles_), last_(last_rows_),
        bytes_((size_t)((tiles_ - 1) * tile_bytes(nr, 16) + tile_bytes(nr, last_rows_)), 0) {}
  // A prime's weight of the upper rows
  struct Weight {
    int32_t p, w;
    double inverse;
    explicit Weight(uint32_t p_) : p((int32_t)p_), w((int32_t)((1ull << 32) % p_)), inverse(1.0 / w) {}
  };
  // row v of slot `dst` for byte u of slot `src`
  void set_byte(int src, int u, int dst, int v, int8_t value) {
    const Rows r = rows(src, dst);
    if (r.first) r.first[v * r.width + u] = (uint8_t)value;
  }
  // the constant for byte u of slot `src` towards slot `dst`: modulo p, and (radix 256) as the integer it is
  void set(int src, int u, int dst, uint32_t value, const Weight& k) {
    int8_t b[4];
    split(value, k, b);
    store(rows(src, dst), u, b);
  }
  void set_integer(int src, int u, int dst, int64_t value) {
    int8_t b[4];
    for (int v = 0; v < 4; ++v) {
      b[v] = (int8_t)(value & 0xFF);
      value = (value - b[v]) / 256;  // exact
    }
    store(rows(src, dst), u, b);
  }
  // the constants for all bytes of slot `src` modulo p: `value`, 256 times it and so on
  void set_word(int src, int dst, uint32_t value, const Weight& k) {
    const Rows r = rows(src, dst);
    if (!r.first) return;
    int8_t b[4];
    for (int u = 0; u < 4; ++u, value = times256(value, (uint32_t)k.p)) {
      split(value, k, b);
      store(r, u, b);
    }
  }
  const std::vector<uint8_t>& bytes() const { return bytes_; }

 private:
  // the first of the rows of slot `dst`, where the bytes of slot `src` are, and the bytes from one to the next; null for a
  // slot without a prime
  struct Rows {
    uint8_t* first;
    int width;
  };
  Rows rows(int src, int dst) {
    const int tile = dst / 4, g = dst % 4, block = src / 16, c = src / 4 % 4, gs = src % 4;
    const int n = tile == tiles_n_ - 1 ? last_ : 16;
    if (tile >= tiles_n_ || 4 * g >= n) return {nullptr, 0};
    const int width = block < full_blocks(nr_) ? 16 : 8;  // bytes per lane
    return {&bytes_[(size_t)tile * tile_bytes(nr_, 16) + (size_t)block * n * 64 + (size_t)(gs * n + 4 * g) * width + 4 * c], width};
  }
  static void split(uint32_t value, const Weight& k, int8_t (&b)[4]) {
    const int32_t e = (int32_t)centred(value, (uint32_t)k.p);
    const int32_t y = (int32_t)(e * k.inverse + (e < 0 ? -0.5 : 0.5)), x = e - y * k.w;
    b[0] = (int8_t)x, b[1] = (int8_t)((x - (int8_t)x) / 256), b[2] = (int8_t)y, b[3] = (int8_t)((y - (int8_t)y) / 256);
  }
  static void store(const Rows& r, int u, const int8_t (&b)[4]) {
    if (r.first)
      for (int v = 0; v < 4; ++v) r.first[v * r.width + u] = (uint8_t)b[v];
  }
  int nr_, tiles_n_, last_;
  std::vector<uint8_t> bytes_;
};

// Whether the engine can work modulo s on nl 29-bit limbs: there is one for this size, and no prime of either base divides
// s (1 / s is a constant of every channel). Keys have no factor of 30 bits; a public modulus may be any odd number.
inline bool usable(const Big& s, int nl) {
  const int nr = regs_for(nl);
  if (!nr) return false;
  for (uint32_t residue : {1u, 3u})
    for (uint32_t p : primes(primes_for(nr), residue))
      if (s.mod_small(p) == 0) return false;
  return true;
}

// All tables for the modulus s (odd, usable()), as one array of 32-bit words, and M_A.
inline std::vector<uint32_t> build_tables(const Big& s, int nl, Big* m_a) {
  const int nr = regs_for(nl), k = primes_for(nr);
  const std::vector<uint32_t> a = primes(k, 3), b = primes(k, 1);
  const Big ma = product(a), mb = product(b);
  *m_a = ma;
  const int alpha = alpha_slot(nr), bias = bias_slot(nr);
  std::vector<uint32_t> f(k), h(k), sgn(k), cst((size_t)cst_bytes(nr) / 4, 0);
  for (int i = 0; i < k; ++i) {
    // x is kept as f x with f^2 = +-(-1/s) / (M_A / a_i) 2^32: the reduced product of two such residues is the
    // coefficient of the quotient in base A itself (up to the sign, which the matrix takes)
    const uint32_t p = a[i], w = (uint32_t)((1ull << 32) % p), sinv = invmod(s.mod_small(p), p);
    uint32_t rest = 1;
    for (int t = 0; t < k; ++t)
      if (t != i) rest = mulmod(rest, prime_mod(a[t], p), p);
    const uint32_t c = mulmod(mulmod(p - sinv, invmod(rest, p), p), w, p);
    sgn[i] = powmod(c, (p - 1) / 2, p) == 1 ? 0 : 1;
    f[i] = powmod(sgn[i] ? p - c : c, (p + 1) / 4, p);
    uint32_t* t = &cst[(size_t)i * 4];
    t[0] = p;
    t[1] = neg_inv32(p);
    t[2] = centred(mulmod(sinv, w, p), p);
  }
  for (int j = 0; j < k; ++j) {
    // x is kept as h x, h = 1 / (M_B / b_j): the coefficient of x in base B itself
    const uint32_t p = b[j], w = (uint32_t)((1ull << 32) % p), sinv = invmod(s.mod_small(p), p);
    uint32_t rest = 1;
    for (int t = 0; t < k; ++t)
      if (t != j) rest = mulmod(rest, prime_mod(b[t], p), p);
    h[j] = invmod(rest, p);
    uint32_t* t = &cst[(size_t)(slots(nr) + j) * 4];
    t[0] = p;
    t[1] = neg_inv32(p);
    t[2] = centred(mulmod(sinv, w, p), p);
    uint32_t* t2 = &cst[(size_t)(2 * slots(nr) + j) * 4];
    t2[0] = t[0];
    t2[1] = t[1];
    t2[2] = centred(mulmod(mulmod(mulmod(rest, invmod(ma.mod_small(p), p), p), w, p), w, p), p);
    t2[3] = 0u - t[2];
  }
  Matrix ab(nr, tiles(nr), last_rows(nr, 0)), ba(nr, tiles(nr), last_rows(nr, 1)), in(nr, tiles(nr), 16), out(nr, limb_tiles(nr), 16);
  const auto channel = [&](Matrix& m, int dst, uint32_t p, const std::vector<std::pair<int, uint32_t>>& src, uint32_t extra) {
    const Matrix::Weight weight(p);
    // sources hold value - kOmega; the bias gives it back, adds `extra` and takes off what the sums start from
    uint32_t sum = 0;
    for (const auto& e : src) {
      sum = (uint32_t)(((uint64_t)sum + e.second) % p);
      m.set_word(e.first, dst, e.second, weight);
    }
    const uint64_t bv = (uint64_t)mulmod(sum, kOmega, p) + extra + (3ull * p - (uint32_t)kStart * 256u);
    m.set(bias, 0, dst, (uint32_t)(bv % p), weight);
  };
  for (int j = 0; j < k; ++j) {
    const uint32_t p = b[j], w = (uint32_t)((1ull << 32) % p);
    const uint32_t hw = mulmod(h[j], w, p), nhw = mulmod(s.mod_small(p), hw, p);
    uint32_t ma_p;
    const std::vector<uint32_t> ainv = inverses(a, p, &ma_p);
    std::vector<std::pair<int, uint32_t>> src;
    for (int i = 0; i < k; ++i) {
      uint32_t c = mulmod(ainv[i], nhw, p);
      if (sgn[i] && c) c = p - c;
      src.push_back({i, c});
    }
    channel(ab, j, p, src, mulmod((uint32_t)kOffset, nhw, p));
    src.clear();
    const uint32_t step = (uint32_t)((1u << 29) % p);
    uint32_t c = hw;
    for (int l = 0; l < nl && l < bias; ++l, c = mulmod(c, step, p)) src.push_back({l, c});
    channel(in, j, p, src, 0);
  }
  for (int i = 0; i < k; ++i) {
    const uint32_t p = a[i], w = (uint32_t)((1ull << 32) % p);
    uint32_t mb_p;
    const std::vector<uint32_t> binv = inverses(b, p, &mb_p);
    const uint32_t fw = mulmod(f[i], w, p), mbfw = mulmod(mb_p, fw, p);
    std::vector<std::pair<int, uint32_t>> src;
    for (int j = 0; j < k; ++j) src.push_back({j, mulmod(binv[j], mbfw, p)});
    const int dst = i;
    channel(ba, dst, p, src, 0);
    const uint32_t neg = mbfw ? p - mbfw : 0;
    ba.set(alpha, 0, dst, neg, Matrix::Weight(p));
    ba.set(alpha, 1, dst, mulmod(neg, 128, p), Matrix::Weight(p));
  }
  for (int j = 0; j < k; ++j) {  // the sum of the sources' upper halves
    ba.set_byte(j, 2, alpha_row(nr), 0, 1);
    ba.set_byte(j, 3, alpha_row(nr), 1, 1);
  }
  // out: the integer sum rho_j M_B / b_j - alpha M_B as columns of weight 2^(29 l)
  {
    std::vector<Big> pre(k + 1, Big(1)), suf(k + 1, Big(1));
    for (int j = 0; j < k; ++j) pre[j + 1] = Big::mul(pre[j], Big((uint64_t)b[j]));
    for (int j = k - 1; j >= 0; --j) suf[j] = Big::mul(suf[j + 1], Big((uint64_t)b[j]));
    const auto integer = [&](int src, int u, const Big& x, int sign) {
      for (int l = 0; l < 4 * limb_tiles(nr); ++l) out.set_integer(src, u, l, sign * (int64_t)x.extract((size_t)29 * l, 29));
    };
    Big total(0);
    for (int j = 0; j < k; ++j) {
      Big x = Big::mul(pre[j], suf[j + 1]);
      total = Big::add(total, x);
      for (int u = 0; u < 4; ++u, x = Big::mul(x, Big(256))) integer(j, u, x, 1);
    }
    integer(bias, 0, Big::mul(total, Big((uint64_t)kOmega)), 1);
    integer(alpha, 0, mb, -1);
    integer(alpha, 1, Big::mul(mb, Big(128)), -1);
  }
  std::vector<uint32_t> t((size_t)table_bytes(nr) / 4);
  auto to = t.begin();
  const auto put = [&](const std::vector<uint8_t>& v) {
    for (size_t o = 0; o < v.size(); o += 4)
      *to++ = (uint32_t)v[o] | (uint32_t)v[o + 1] << 8 | (uint32_t)v[o + 2] << 16 | (uint32_t)v[o + 3] << 24;
  };
  put(ab.bytes());
  put(ba.bytes());
  to = std::copy(cst.begin(), cst.end(), to);
  put(in.bytes());
  put(out.bytes());
  return t;
}

}  // namespace rns
}  // namespace haflo
