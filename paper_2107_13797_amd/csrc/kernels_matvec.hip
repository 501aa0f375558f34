// Ciphertext matrix-vector products, ciphertext summation and the modular
// inverse they need for negative exponents. Kernels and C entry points.
//
// X^T [[d]] (orientation 0): the bases c_i are shared by every output column,
//   so each base gets a table of its powers c_i^0..c_i^16; with signed 5-bit
//   digits d_s of |x_ij| output column j is
//   prod_s ( prod_i table_i[|d_s|] )^(32^s), with the terms of either sign
//   collected separately and one inversion per column. Where the workspace has
//   room for it, the bucket method of kernels_buckets.hip takes its place, which
//   ends in the same per-column pair of products.
// X [[w]] (orientation 1): the few bases c_j are shared by every output row,
//   so each base (and its inverse) gets positional tables c_j^(d 2^(w s)); an
//   output row is a plain product of table entries over its non-zero entries,
//   which are compacted per row first; rows are processed in the order of
//   their list lengths.
#include "kernels_common.hpp"

#include <stdlib.h>

#include <algorithm>

using namespace haflo;
using namespace haflo::dev;

namespace {

// Orientation 1: unsigned 8-bit digits of |x|, positional tables.
constexpr int kWin = 8;                    // window width of the exponent digits
constexpr int kWinEntries = 1 << kWin;     // table entries per base and position (entry 0 unused)
constexpr int kMaxPos = (32 + kWin - 1) / kWin;  // digit positions of a 32-bit magnitude

// Orientation 0: signed 5-bit digits. |x| + c, c = 16 (32^S - 1) / 31, is read in base 32 and
// each digit e is taken as d = e - 16 in [-16, 15], so |x| = sum d_s 32^s: the table holds only
// c^0..c^16 and a negative digit sends the term to the accumulator of the opposite sign.
constexpr int kSWin = 5;
constexpr int kSEntries = 17;
constexpr int kSMaxPos = 7;  // 32^7 - c_7 > 2^31
__host__ __device__ inline unsigned long long signed_digit_offset(int npos) {
  unsigned long long c = 0;
  for (int s = 0; s < npos; ++s) c = c * 32ull + 16ull;
  return c;
}
// positions needed so that maxmag + c_S < 32^S (0 for an all-zero matrix)
__host__ __device__ inline int signed_digit_positions(unsigned maxmag) {
  if (maxmag == 0) return 0;
  for (int s = 1; s < kSMaxPos; ++s)
    if ((unsigned long long)maxmag + signed_digit_offset(s) < (1ull << (kSWin * s))) return s;
  return kSMaxPos;
}

// ---------------------------------------------------------------------------
// modular inverse by batched division steps
// ---------------------------------------------------------------------------

// 29 division steps of the Bernstein-Yang 2-adic gcd recurrence on the low
// bits of (f, g), f odd:
//   g odd and delta > 0:  (delta, f, g) <- (1 - delta, g, (g - f) / 2)
//   g odd otherwise:      (delta, f, g) <- (1 + delta, f, (g + f) / 2)
//   g even:               (delta, f, g) <- (1 + delta, f, g / 2)
// Returns the integer matrix with 2^29 (f', g') = (u f + v g, q f + r g); every
// entry has magnitude at most 2^29 and each row sums to at most 2^29 in
// magnitude.
// The steps are taken in runs: all the halvings that g's trailing zeros allow at once (a count of
// trailing zeros), then, g being odd, the combination of one odd step without its halving, which the
// next run takes. Both of the odd step's outcomes are formed and one is selected - (f, g) <- (g, g - f) and the matrix rows
// likewise when delta > 0, else (f, g + f) - so that it is straight-line code on the scalar unit (a whole-wavefront group,
// where f0 and g0 are wave-uniform) as well as on the vector unit; a row of the matrix is one 64-bit integer, u + 2^32 v,
// on which shifts, sums and differences are those of its entries. About half as many loop rounds as steps, of 23 scalar
// instructions each. They bound the inversion, whose wavefront issues one at a time: with masks on four entries, 36 of them,
// 32 inversions took 142, 280 us at 1024 and 2048 bits, now 104 and 205. Several integers to a wavefront, on the vector unit, gain
// too: 20000 powers by -5 at 1024, 2048 and 4096 bits 466, 1297 and 4134 us, now 426, 1169 and 3766.
__device__ __forceinline__ void divsteps29(int& delta, u32 f0, u32 g0, s32& u, s32& v, s32& q, s32& r) {
  s32 eta = -delta;  // the swap condition is eta < 0
  u64 row_f = 1, row_g = 1ull << 32;
  int left = LIMB_BITS;
  const auto halve = [&]() {
    const int z = __builtin_ctz(g0 | (1u << left));  // bits [0, left) of g0 are exact, bit `left` ends the run
    g0 >>= z;
    row_f <<= z;
    eta -= z;
    left -= z;
  };
  halve();
  while (left > 0) {
    const bool swap = eta < 0;
    const u32 sum = g0 + f0, less = g0 - f0;
    const u64 row_sum = row_g + row_f, row_less = row_g - row_f;
    f0 = swap ? g0 : f0;
    g0 = swap ? less : sum;
    row_f = swap ? row_g : row_f;
    row_g = swap ? row_less : row_sum;
    eta = swap ? -eta : eta;
    halve();
  }
  delta = -eta;
  u = (s32)(u32)row_f;
  v = (s32)((s64)(row_f - (u64)(s64)u) >> 32);
  q = (s32)(u32)row_g;
  r = (s32)((s64)(row_g - (u64)(s64)q) >> 32);
}

// Shared tail of the two linear updates: absorb the carry of the lane below,
// then drop the (vanished) lowest limb; the top lane's carry becomes the new,
// signed, top limb.
template <int LPT, int T>
__device__ __forceinline__ void shift_down(s32 (&x)[LPT], s32 (&nx)[LPT], s64 carry, const Grp<T>& g) {
  if (T > 1) {
    s32 cin = (s32)g.from_lower((u32)(s32)carry);
    s64 v0 = (s64)nx[0] + (s64)cin;
    nx[0] = (s32)(v0 & (s64)LIMB_MASK);
    nx[1] += (s32)(v0 >> LIMB_BITS);
  }
  s32 down = (s32)g.from_upper((u32)nx[0]);
#pragma unroll
  for (int j = 0; j + 1 < LPT; ++j) x[j] = nx[j + 1];
  x[LPT - 1] = (g.k == T - 1) ? (s32)carry : down;
}

// out = in^-1 * R^2 ... precisely: for `a` the Montgomery form x R of a unit x
// modulo the odd modulus m, returns the Montgomery form x^-1 R (canonical).
// Works on signed numbers in radix 2^29 whose top limb carries the sign:
// (f, g) start at (m, a) and are driven to (+-1, 0) by batches of 29 division
// steps, (d, e) start at (0, 1) and follow the same matrices modulo m, so that
// d * a = f (mod m) throughout; |d| grows by at most m per batch, which the
// head-room of the radix above m absorbs. nbatch bounds the number of batches.
template <int LPT, int T>
__device__ __forceinline__ void invert_mont(u32 (&out)[LPT], const u32 (&a)[LPT], const ModRegs<LPT>& M,
                                            const u32* r3, int nbatch, const Grp<T>& g) {
  s32 f[LPT], gg[LPT], d[LPT], e[LPT];
#pragma unroll
  for (int j = 0; j < LPT; ++j) {
    f[j] = (s32)M.n[j];
    gg[j] = (s32)a[j];
    d[j] = 0;
    e[j] = 0;
  }
  if (g.k == 0) e[0] = 1;
  int delta = 1;
#pragma unroll 1
  for (int b = 0; b < nbatch; ++b) {
    s32 any = 0;
#pragma unroll
    for (int j = 0; j < LPT; ++j) any |= gg[j];
    if (!wave_any(any != 0)) break;
    u32 f0 = g.bcast0((u32)f[0]), g0 = g.bcast0((u32)gg[0]);
    s32 u, v, q, r;
    divsteps29(delta, f0, g0, u, v, q, r);
    {
      s64 cf = 0, cg = 0;
      s32 nf[LPT], ng[LPT];
#pragma unroll
      for (int j = 0; j < LPT; ++j) {
        s64 tf = (s64)u * f[j] + (s64)v * gg[j] + cf;
        s64 tg = (s64)q * f[j] + (s64)r * gg[j] + cg;
        nf[j] = (s32)(tf & (s64)LIMB_MASK);
        cf = tf >> LIMB_BITS;
        ng[j] = (s32)(tg & (s64)LIMB_MASK);
        cg = tg >> LIMB_BITS;
      }
      shift_down<LPT, T>(f, nf, cf, g);
      shift_down<LPT, T>(gg, ng, cg, g);
    }
    {
      // multiples of m that clear the lowest limb of each combination
      u32 lowd = (u32)u * (u32)d[0] + (u32)v * (u32)e[0];
      u32 lowe = (u32)q * (u32)d[0] + (u32)r * (u32)e[0];
      u32 kd = g.bcast0((lowd * M.n0inv) & LIMB_MASK);
      u32 ke = g.bcast0((lowe * M.n0inv) & LIMB_MASK);
      s64 cd = 0, ce = 0;
      s32 nd[LPT], ne[LPT];
#pragma unroll
      for (int j = 0; j < LPT; ++j) {
        s64 td = (s64)u * d[j] + (s64)v * e[j] + (s64)((u64)kd * M.n[j]) + cd;
        s64 te = (s64)q * d[j] + (s64)r * e[j] + (s64)((u64)ke * M.n[j]) + ce;
        nd[j] = (s32)(td & (s64)LIMB_MASK);
        cd = td >> LIMB_BITS;
        ne[j] = (s32)(te & (s64)LIMB_MASK);
        ce = te >> LIMB_BITS;
      }
      shift_down<LPT, T>(d, nd, cd, g);
      shift_down<LPT, T>(e, ne, ce, g);
    }
  }
  // f = +-1 now; the inverse is sign(f) * d modulo m
  u32 f0 = g.bcast0((u32)f[0]) & LIMB_MASK;
  bool fneg = (f0 != 1u);
#pragma unroll
  for (int j = 0; j < LPT; ++j) d[j] = fneg ? -d[j] : d[j];
  int top = resolve<LPT, T>(d, g);
  bool neg = top < 0;
  // from here on every group of the wave runs the same cross-lane code and
  // only selects differ
#pragma unroll
  for (int j = 0; j < LPT; ++j) d[j] = neg ? -d[j] : d[j];
  resolve<LPT, T>(d, g);
  u32 x[LPT], t[LPT];
#pragma unroll
  for (int j = 0; j < LPT; ++j) x[j] = (u32)d[j];
  load_limbs<LPT, T>(t, r3, g);
  montmul<LPT, T>(x, x, t, M.n, M.n0inv, g);  // |d| R^-1 * R^3 / R = |d| R
  canonicalise<LPT, T>(x, M.n, g);
  s32 y[LPT];
#pragma unroll
  for (int j = 0; j < LPT; ++j) y[j] = neg ? (s32)M.n[j] - (s32)x[j] : (s32)x[j];
  resolve<LPT, T>(y, g);
#pragma unroll
  for (int j = 0; j < LPT; ++j) x[j] = (u32)y[j];
  canonicalise<LPT, T>(x, M.n, g);  // m - 0 = m folds back to 0
#pragma unroll
  for (int j = 0; j < LPT; ++j) out[j] = x[j];
}

// The same inverse modulo n^2, through n: y = x^-1 mod n costs half the division steps (the modulus
// has half the bits), and one Newton step lifts it, x^-1 = y (2 - x y) mod n^2.
//   a: Montgomery form x R mod n^2 (lazy), M2/mod2: n^2, Mn: the modulus n with the same R and limb
//   count, nbatch_n: batches for the bit length of n. Returns x^-1 R mod n^2, canonical.
template <int LPT, int T>
__device__ __forceinline__ void invert_lifted(u32 (&out)[LPT], const u32 (&a)[LPT], const ModRegs<LPT>& mod2,
                                              const ModRef& M2, const ModRef& Mn, int nbatch_n, const Grp<T>& g) {
  ModRegs<LPT> mn;
  load_mod<LPT, T>(mn, Mn, g);
  u32 y[LPT], t[LPT];
  load_limbs<LPT, T>(t, Mn.r1, g);
  montmul<LPT, T>(y, a, t, mn.n, mn.n0inv, g);  // a (R mod n) / R = a mod n, which is x R mod n
  canonicalise<LPT, T>(y, mn.n, g);
  invert_mont<LPT, T>(y, y, mn, Mn.r3, nbatch_n, g);  // (x^-1 mod n) R mod n
  load_limbs<LPT, T>(t, Mn.one, g);
  montmul<LPT, T>(y, y, t, mn.n, mn.n0inv, g);  // x^-1 mod n, as a plain integer
  canonicalise<LPT, T>(y, mn.n, g);
  load_limbs<LPT, T>(t, M2.r2, g);
  montmul<LPT, T>(y, y, t, mod2.n, mod2.n0inv, g);  // Y = y R mod n^2
  montmul<LPT, T>(t, a, y, mod2.n, mod2.n0inv, g);  // x y R mod n^2
  canonicalise<LPT, T>(t, mod2.n, g);
  // u = (2 - x y) R + n^2 > 0, below 3 n^2
  u32 r1[LPT];
  load_limbs<LPT, T>(r1, M2.r1, g);
  s32 u[LPT];
#pragma unroll
  for (int j = 0; j < LPT; ++j) u[j] = (s32)(2u * r1[j] + mod2.n[j]) - (s32)t[j];
  resolve<LPT, T>(u, g);
#pragma unroll
  for (int j = 0; j < LPT; ++j) t[j] = (u32)u[j];
  montmul<LPT, T>(y, y, t, mod2.n, mod2.n0inv, g);
  canonicalise<LPT, T>(y, mod2.n, g);
#pragma unroll
  for (int j = 0; j < LPT; ++j) out[j] = y[j];
}

template <int LPT, int T>
__global__ __launch_bounds__(kBlockThreads) void k_invert(ModRef M, ModRef Mn, const u32* in, u32* out, size_t count,
                                                          int nbatch_n) {
  constexpr int NL = LPT * T;
  Grp<T> g;
  Batch<T> bt;
  ModRegs<LPT> mod;
  load_mod<LPT, T>(mod, M, g);
  for (size_t base = bt.first(); base < count; base += bt.stride()) {
    size_t item = base + bt.gib;
    bool active = item < count;
    u32 x[LPT];
    if (active) load_limbs<LPT, T>(x, in + item * (size_t)NL, g);
    else zero_limbs<LPT>(x);
    invert_lifted<LPT, T>(x, x, mod, M, Mn, nbatch_n, g);
    if (active) store_limbs<LPT, T>(out + item * (size_t)NL, x, g);
  }
}

// ---------------------------------------------------------------------------
// shared pieces
// ---------------------------------------------------------------------------

// largest |x| in the matrix (atomicMax into a zeroed word)
__global__ __launch_bounds__(kBlockThreads) void k_zero_word(u32* p, int n) {
  // the largest |x|, a work counter and, for orientation 1, the histogram of list lengths
  if (blockIdx.x == 0)
    for (int i = (int)threadIdx.x; i < n; i += (int)blockDim.x) p[i] = 0u;
}
__global__ __launch_bounds__(kBlockThreads) void k_maxmag(const int* __restrict__ X, size_t total, u32* maxmag) {
  u32 m = 0;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    int x = X[i];
    u32 mag = x < 0 ? 0u - (u32)x : (u32)x;
    m = mag > m ? mag : m;
  }
  // the word only grows: a wavefront whose maximum is already there leaves it alone, so the atomics on the one
  // address stay few
  const u32 best = wave_max(m);
  if ((threadIdx.x & (WAVE - 1)) == 0 && best > *(volatile u32*)maxmag) atomicMax(maxmag, best);
}
__device__ __forceinline__ int bit_length(u32 v) { return v ? 32 - __builtin_clz(v) : 0; }

// product of the per-group accumulators of a block, left in group 0.
// lds: (groups per block / 2) * NL limbs.
template <int LPT, int T>
__device__ __forceinline__ void block_product(u32 (&acc)[LPT], u32* lds, const ModRegs<LPT>& mod, const Batch<T>& bt,
                                              const Grp<T>& g) {
  constexpr int NL = LPT * T;
  for (int stride = bt.gpb >> 1; stride >= 1; stride >>= 1) {
    if (bt.gib >= stride && bt.gib < 2 * stride) {
      u32* dst = lds + (bt.gib - stride) * NL + g.k * LPT;
#pragma unroll
      for (int j = 0; j < LPT; ++j) dst[j] = acc[j];
    }
    __syncthreads();
    u32 t[LPT], r[LPT];
    bool take = bt.gib < stride;
    const u32* src = lds + (take ? bt.gib : 0) * NL + g.k * LPT;
#pragma unroll
    for (int j = 0; j < LPT; ++j) t[j] = src[j];
    montmul<LPT, T>(r, acc, t, mod.n, mod.n0inv, g);
    if (take) {
#pragma unroll
      for (int j = 0; j < LPT; ++j) acc[j] = r[j];
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// orientation 0: out[j] = prod_i c_i^X[i][j]
// ---------------------------------------------------------------------------

// block (j, s, rs): product over the rows of slice rs of table_i[digit s of
// |X[i][j]|], positive and negative entries apart -> partials[j][s][sign][rs]
template <int LPT, int T>
__global__ __launch_bounds__(kBlockThreads, 3) void k_xtd_main(ModRef M, const int* __restrict__ X, size_t rows,
                                                            size_t cols, const u32* __restrict__ tables, int rsplit,
                                                            u32* __restrict__ partials,
                                                            const u32* __restrict__ maxmag) {
  constexpr int NL = LPT * T;
  __shared__ u32 lds[(kBlockThreads / 2) * LPT];
  Grp<T> g;
  Batch<T> bt;
  // Blocks are handed to the 8 XCDs round-robin. The `cols` blocks of one (s, rs) slice read
  // the same table entries, so a slice is kept on one XCD (whose L2 then serves the re-reads)
  // and consecutive slices go to consecutive XCDs. The grid holds a multiple of 8 slices.
  const size_t xcd = blockIdx.x % 8u, local = blockIdx.x / 8u;
  const size_t slice = xcd + 8u * (local / cols);
  const size_t j = local % cols;
  const int rs = (int)(slice % (size_t)rsplit);
  const int s = (int)(slice / (size_t)rsplit);
  if (s >= kSMaxPos) return;  // padding slices
  const int npos = signed_digit_positions(*maxmag);
  if (s >= npos) return;  // no digit at this position anywhere
  const u64 offset = signed_digit_offset(npos);
  ModRegs<LPT> mod;
  load_mod<LPT, T>(mod, M, g);
  const size_t r0 = rows * (size_t)rs / (size_t)rsplit, r1 = rows * (size_t)(rs + 1) / (size_t)rsplit;
  u32 accp[LPT], accn[LPT];
  load_limbs<LPT, T>(accp, M.r1, g);
#pragma unroll
  for (int jj = 0; jj < LPT; ++jj) accn[jj] = accp[jj];
  for (size_t base = r0; base < r1; base += (size_t)bt.gpb) {
    size_t i = base + bt.gib;
    bool active = i < r1;
    int x = active ? X[i * cols + j] : 0;
    u32 mag = x < 0 ? 0u - (u32)x : (u32)x;
    int d = (int)((((u64)mag + offset) >> (s * kSWin)) & 31ull) - 16;
    u32 dgt = (u32)(d < 0 ? -d : d);
    const u32* entry = active ? tables + (i * (size_t)kSEntries + dgt) * NL : M.r1;
    u32 cur[LPT];
    bool neg = (x < 0) != (d < 0);
#pragma unroll
    for (int jj = 0; jj < LPT; ++jj) cur[jj] = neg ? accn[jj] : accp[jj];
    montmul_mem<LPT, T>(cur, cur, entry, mod.n, mod.n0inv, g);
#pragma unroll
    for (int jj = 0; jj < LPT; ++jj) {
      if (neg) accn[jj] = cur[jj];
      else accp[jj] = cur[jj];
    }
  }
  block_product<LPT, T>(accp, lds, mod, bt, g);
  block_product<LPT, T>(accn, lds, mod, bt, g);
  if (bt.gib == 0) {
    size_t slot = ((j * (size_t)kSMaxPos + (size_t)s) * 2) * (size_t)rsplit + (size_t)rs;
    store_limbs<LPT, T>(partials + slot * NL, accp, g);
    store_limbs<LPT, T>(partials + (slot + (size_t)rsplit) * NL, accn, g);
  }
}

// one group per (j, sign): P = prod_s (prod_rs partial[j][s][sign][rs])^(2^(w s)), top position first
template <int LPT, int T>
__global__ __launch_bounds__(kBlockThreads) void k_xtd_horner(ModRef M, size_t cols, int rsplit,
                                                              const u32* __restrict__ partials, u32* __restrict__ P,
                                                              const u32* __restrict__ maxmag) {
  constexpr int NL = LPT * T;
  Grp<T> g;
  Batch<T> bt;
  ModRegs<LPT> mod;
  load_mod<LPT, T>(mod, M, g);
  const int npos = signed_digit_positions(*maxmag);
  const size_t count = cols * 2;
  for (size_t base = bt.first(); base < count; base += bt.stride()) {
    size_t item = base + bt.gib;
    bool active = item < count;
    size_t j = active ? item >> 1 : 0;
    size_t sign = item & 1;
    u32 acc[LPT], t[LPT];
    load_limbs<LPT, T>(acc, M.r1, g);
#pragma unroll 1
    for (int s = npos - 1; s >= 0; --s) {
      if (s != npos - 1) {
#pragma unroll 1
        for (int i = 0; i < kSWin; ++i) montsqr<LPT, T>(acc, acc, mod.n, mod.n0inv, g);
      }
#pragma unroll 1
      for (int rs = 0; rs < rsplit; ++rs) {
        size_t slot = ((j * (size_t)kSMaxPos + (size_t)s) * 2 + sign) * (size_t)rsplit + (size_t)rs;
        load_limbs<LPT, T>(t, partials + slot * NL, g);
        montmul<LPT, T>(acc, acc, t, mod.n, mod.n0inv, g);
      }
    }
    if (active) store_limbs<LPT, T>(P + item * (size_t)NL, acc, g);
  }
}

// out[j] = P[j][+] * (P[j][-])^-1
template <int LPT, int T>
__global__ __launch_bounds__(kBlockThreads) void k_xtd_finish(ModRef M, ModRef Mn, size_t cols,
                                                              const u32* __restrict__ P, u32* __restrict__ out,
                                                              int nbatch_n) {
  constexpr int NL = LPT * T;
  Grp<T> g;
  Batch<T> bt;
  ModRegs<LPT> mod;
  load_mod<LPT, T>(mod, M, g);
  for (size_t base = bt.first(); base < cols; base += bt.stride()) {
    size_t j = base + bt.gib;
    bool active = j < cols;
    u32 pos[LPT], neg[LPT];
    if (active) {
      load_limbs<LPT, T>(pos, P + (2 * j) * (size_t)NL, g);
      load_limbs<LPT, T>(neg, P + (2 * j + 1) * (size_t)NL, g);
    } else {
      load_limbs<LPT, T>(pos, M.r1, g);
      load_limbs<LPT, T>(neg, M.r1, g);
    }
    invert_lifted<LPT, T>(neg, neg, mod, M, Mn, nbatch_n, g);
    montmul<LPT, T>(pos, pos, neg, mod.n, mod.n0inv, g);
    canonicalise<LPT, T>(pos, mod.n, g);
    if (active) store_limbs<LPT, T>(out + j * (size_t)NL, pos, g);
  }
}

// ---------------------------------------------------------------------------
// orientation 1: out[i] = prod_j c_j^X[i][j]
// ---------------------------------------------------------------------------

// Positional tables T[j][sign][s][d] = b^(d 256^s), b = c_j or its inverse, d = 1..255.
// k_xw_positions, one group per (j, sign, s): T[1] = b^(256^s) by 8 s squarings. Then eight launches of
// k_xw_level with B = 1, 2, 4, .., 128, one group per entry d in (B, 2 B]: T[d] = T[d - B] * T[B]. Every entry
// costs one product and the chain is 8 s + 8 products long.
// PAIR: the tables are in the pair form modulo M (see Elem); the bases, stored ciphertexts, are taken into it
// as they are loaded (k_lo, k_hi: see to_pair).
template <int LPT, int T, bool PAIR>
__global__ __launch_bounds__(kBlockThreads) void k_xw_positions(ModRef M, const u32* __restrict__ k_lo,
                                                                const u32* __restrict__ k_hi,
                                                                const u32* __restrict__ bases,
                                                                const u32* __restrict__ invbases, size_t cols,
                                                                u32* __restrict__ tables,
                                                                const u32* __restrict__ maxmag) {
  using Ops = ElemOps<LPT, T, PAIR>;
  constexpr int EL = Ops::kLimbs;
  Grp<T> g;
  Batch<T> bt;
  ModRegs<LPT> mod;
  load_mod<LPT, T>(mod, M, g);
  const int npos = (bit_length(*maxmag) + kWin - 1) / kWin;
  const size_t count = cols * 2 * (size_t)npos;
  for (size_t base = bt.first(); base < count; base += bt.stride()) {
    const size_t it = base + bt.gib;
    const bool active = it < count;
    const size_t item = active ? it / (size_t)npos : 0;  // j * 2 + sign
    const int s = active ? (int)(it - item * (size_t)npos) : 0;
    const u32* src = (item & 1) ? invbases : bases;
    typename Ops::E x, t;
    if constexpr (PAIR) to_pair<LPT, T>(x.x0, x.x1, src + (item >> 1) * (size_t)EL, k_lo, k_hi, mod, g);
    else Ops::load(x, src + (item >> 1) * (size_t)EL, g);
    // every group of a wavefront runs the same squarings; the ones that are done discard theirs
#pragma unroll 1
    for (int i = 0; wave_any(i < kWin * s); ++i) {
      Ops::copy(t, x);
      Ops::sqr(t, mod, g);
      if (i < kWin * s) Ops::copy(x, t);
    }
    u32* tb = tables + ((item * (size_t)kMaxPos + (size_t)s) * (size_t)kWinEntries) * EL;
    if (active) Ops::store(tb + EL, x, g);
  }
}

template <int LPT, int T, bool PAIR>
__global__ __launch_bounds__(kBlockThreads) void k_xw_level(ModRef M, const u32* __restrict__ one, size_t cols, int B,
                                                            u32* __restrict__ tables,
                                                            const u32* __restrict__ maxmag) {
  using Ops = ElemOps<LPT, T, PAIR>;
  constexpr int EL = Ops::kLimbs;
  Grp<T> g;
  Batch<T> bt;
  ModRegs<LPT> mod;
  load_mod<LPT, T>(mod, M, g);
  const int npos = (bit_length(*maxmag) + kWin - 1) / kWin;
  const int per = B < kWinEntries - 1 - B ? B : kWinEntries - 1 - B;  // entries B + 1 .. min(2 B, 255)
  const size_t count = cols * 2 * (size_t)npos * (size_t)per;
  for (size_t base = bt.first(); base < count; base += bt.stride()) {
    const size_t it = base + bt.gib;
    const bool active = it < count;
    const size_t tab = active ? it / (size_t)per : 0;  // (j * 2 + sign) * npos + s
    const int d = B + 1 + (active ? (int)(it - tab * (size_t)per) : 0);
    const size_t item = tab / (size_t)(npos ? npos : 1);
    const int s = (int)(tab - item * (size_t)(npos ? npos : 1));
    u32* tb = tables + ((item * (size_t)kMaxPos + (size_t)s) * (size_t)kWinEntries) * EL;
    typename Ops::E a;
    Ops::load(a, active ? tb + (size_t)(d - B) * EL : one, g);
    Ops::mul_mem(a, active ? tb + (size_t)B * EL : one, mod, g);
    if (active) Ops::store(tb + (size_t)d * EL, a, g);
  }
}

// The tables in the residue form are two programs (RnsLists) and one set of chains:
//   1. c_j or its inverse (and, behind them, one): its powers to 16^q, q = 0 to 7, as far as the exponents go
//   2. base and q: the powers to 1, .., 15 of that, T[d] (q even) or T[16 d] of position q / 2
//   3. T[16 h + l] = T[16 h] T[l], of the last position up to the largest digit
constexpr int kNibbles = 2 * kMaxPos, kMixed = 225;
struct XwTablePlan {  // words from the start of the workspace
  size_t operands, places[2], live, index, chains, control;
};
__global__ __launch_bounds__(kBlockThreads) void k_xw_places(u32 cols, u32* __restrict__ ws, XwTablePlan p,
                                                             const u32* __restrict__ one, u32 limbs, u32* __restrict__ pair,
                                                             const u32* __restrict__ maxmag) {
  const u32 npos = (u32)((bit_length(*maxmag) + kWin - 1) / kWin), bases = cols * 2;
  const u32 top = npos ? *maxmag >> (npos - 1) * kWin : 0;  // the largest digit of the last position
  const u32 top_mixed = top < 17 ? 0 : (top / 16 - 1) * 15 + top % 16, mixed = npos ? bases * ((npos - 1) * kMixed + top_mixed) : 0;
  const u32 at = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
  if (at == 0) {
    u32* live = ws + p.live;
    live[0] = bases + 1;
    live[1] = bases * 2 * npos;
    live[2] = npos ? 2 + 5 * (2 * npos - 1) : 2;  // of the first program's instructions
    ws[p.control + kChainsTotal] = mixed;
    ws[p.control + kChainsColumns] = 0;
  }
  for (u32 i = at; i < limbs; i += step) pair[i] = one[i];
  // the powers: of the bases, of the inverses, of one
  for (u32 i = at; i < (bases + 1) * kNibbles; i += step) ws[p.places[0] + i] = i % (bases + 1) * kNibbles + i / (bases + 1);
  for (u32 i = at; i < bases * kNibbles; i += step) {
    const u32 e = i % bases, q = i / bases;  // e: 2 j + sign
    ws[p.operands + i] = (e / 2 + e % 2 * cols) * kNibbles + q;
    for (u32 d = 1; d < 16; ++d)
      ws[p.places[1] + (size_t)(d - 1) * bases * kNibbles + i] = (e * kMaxPos + q / 2) * kWinEntries + (q % 2 ? 16 * d : d);
  }
  for (u32 i = at; i < mixed; i += step) {
    const u32 full = bases * (npos - 1) * kMixed;
    const u32 tab = i < full ? i / kMixed : bases * (npos - 1) + (i - full) / top_mixed;
    const u32 r = i < full ? i % kMixed : (i - full) % top_mixed, high = 16 * (r / 15 + 1), low = r % 15 + 1;
    const u32 t = (tab % bases * kMaxPos + tab / bases) * kWinEntries;
    ws[p.index + 2 * (size_t)i] = t + high;
    ws[p.index + 2 * (size_t)i + 1] = t + low;
    ((uint4*)(ws + p.chains))[i] = make_uint4(t + high + low, 2 * i, 2u, 0u);
  }
}

// Rows' products as chains: 2^seg_shift of near-equal length for a row, in the order `order`, and behind them (unless a row
// is one chain) those that combine a row's. The chains that end in a row's product are launched `portion` at a time, each time
// with kPortionWords of control words and counter of their own. Where a row is one chain its product's place is that of the row in
// the order, and the rows with empty lists, all behind the first *filled, take no part: of narrow sparse matrices they are most, and
// their way out of the residue form took longer than everything did on limbs. us of whole calls, limbs / all rows / the filled ones,
// 5 % of the entries non-zero: 4096 bits 65536 by 4 1203 / 1377 / 1003, by 16 1528 / 1520 / 1302, 262144 by 4 2364 / 3050 / 1439;
// 2048 bits 65536 by 4 509 / 540 / 466, 262144 by 4 880 / 1014 / 600. With no empty rows 65536 by 32 at 2048 bits 2006 / 2011.
enum { kPortionNext = kChainsControl, kPortionWords = 4 };
__global__ __launch_bounds__(kBlockThreads) void k_xw_chains(size_t rows, size_t list_stride, int seg_shift, size_t portion,
                                                             const u32* __restrict__ counts, const u32* __restrict__ order,
                                                             const u32* __restrict__ filled, uint4* __restrict__ chains,
                                                             u32* __restrict__ control, u32* __restrict__ portions) {
  const size_t items = rows << seg_shift, leaving = seg_shift ? rows : (size_t)*filled, at = (size_t)blockIdx.x * blockDim.x + threadIdx.x, step = (size_t)gridDim.x * blockDim.x;
  if (at == 0) {
    control[kChainsTotal] = (u32)items;
    control[kChainsColumns] = 0;
  }
  for (size_t i = at; i * portion < rows; i += step) {
    u32* c = portions + i * kPortionWords;
    c[kChainsTotal] = (u32)(leaving > i * portion ? std::min(leaving - i * portion, portion) : 0);
    c[kChainsColumns] = 1;
    c[kPortionNext] = 0;
  }
  for (size_t i = at; i < items; i += step) {
    const u32 row = order[i >> seg_shift], seg = (u32)i & ((1u << seg_shift) - 1u);
    const u64 len = counts[row];
    const u32 e0 = (u32)((len * seg) >> seg_shift), e1 = (u32)((len * (seg + 1u)) >> seg_shift);
    const u32 place = seg_shift ? (row << seg_shift) + seg : (u32)(i % portion);
    chains[i] = make_uint4(place, (u32)(row * list_stride) + e0, e1 - e0, 0u);
    if (seg == 0 && seg_shift) chains[items + row] = make_uint4(row, row << seg_shift, 1u << seg_shift, 0u);
  }
}

// Rows are handed to the wavefronts of k_xw_main in the order of their list lengths, longest
// first, so that the rows a wavefront multiplies side by side finish together. The lengths are
// sorted by counting in kLenBins classes, of which the empty lists are one.
constexpr int kLenBins = 1024;
__device__ __forceinline__ u32 length_bin(u32 len, size_t longest) {
  return len == 0u ? 0u : 1u + (u32)(((u64)len * (u64)(kLenBins - 2)) / (u64)longest);
}

// Per row: the list of table entries its product consists of, one per non-zero 8-bit digit
// of every non-zero |X[row][c]|: entry index ((c*2 + sign)*kMaxPos + s)*256 + digit, in units of
// one table entry. One wave per row; lists: rows * cols * kMaxPos words, counts: rows.
__global__ __launch_bounds__(kBlockThreads) void k_xw_lists(const int* __restrict__ X, size_t rows, size_t cols,
                                                            u32* __restrict__ lists, u32* __restrict__ counts,
                                                            const u32* __restrict__ maxmag) {
  const int lane = (int)(threadIdx.x & (WAVE - 1));
  const size_t wave = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
  const size_t nwaves = ((size_t)gridDim.x * blockDim.x) / WAVE;
  const int npos = (bit_length(*maxmag) + kWin - 1) / kWin;
  for (size_t row = wave; row < rows; row += nwaves) {
    u32* mine = lists + row * cols * (size_t)kMaxPos;
    u32 written = 0;
    for (size_t c0 = 0; c0 < cols; c0 += WAVE) {
      size_t c = c0 + (size_t)lane;
      int x = (c < cols) ? X[row * cols + c] : 0;
      u32 mag = x < 0 ? 0u - (u32)x : (u32)x;
      u32 tsel = (u32)c * 2u + (x < 0 ? 1u : 0u);
      for (int s = 0; s < npos; ++s) {
        u32 dgt = (mag >> (s * kWin)) & (u32)(kWinEntries - 1);
        u64 mask = __builtin_amdgcn_ballot_w64(dgt != 0u);
        if (dgt != 0u) {
          u32 before = (u32)__builtin_popcountll(mask & ((1ull << lane) - 1ull));
          mine[written + before] = (tsel * (u32)kMaxPos + (u32)s) * (u32)kWinEntries + dgt;
        }
        written += (u32)__builtin_popcountll(mask);
      }
    }
    if (lane == 0) counts[row] = written;
  }
}

// Counting sort of the rows by length class, in two passes around k_xw_order_scan. A block takes 256
// rows at a time and counts them in LDS first, so that global memory sees one atomic per class and
// block. SCATTER = false: bins[b] += rows of class b. SCATTER = true: bins[] are the cursors left by the
// scan; the block reserves its share of every class and writes order[cursor + rank in the block] = row.
template <bool SCATTER>
__global__ __launch_bounds__(kBlockThreads) void k_xw_order(const u32* __restrict__ counts, size_t rows, size_t cols,
                                                            u32* __restrict__ bins, u32* __restrict__ order,
                                                            const u32* __restrict__ maxmag) {
  __shared__ u32 hist[kLenBins];
  __shared__ u32 start[SCATTER ? kLenBins : 1];
  const int npos = (bit_length(*maxmag) + kWin - 1) / kWin;
  const size_t longest = cols * (size_t)npos;
  for (size_t r0 = (size_t)blockIdx.x * kBlockThreads; r0 < rows; r0 += (size_t)gridDim.x * kBlockThreads) {
    for (int l = (int)threadIdx.x; l < kLenBins; l += kBlockThreads) hist[l] = 0u;
    __syncthreads();
    const size_t row = r0 + threadIdx.x;
    const bool active = row < rows;
    const u32 bin = active ? length_bin(counts[row], longest) : 0u;
    const u32 rank = active ? atomicAdd(&hist[bin], 1u) : 0u;
    __syncthreads();
    for (int l = (int)threadIdx.x; l < kLenBins; l += kBlockThreads) {
      const u32 c = hist[l];
      if (c == 0u) continue;
      const u32 before = atomicAdd(&bins[l], c);
      if (SCATTER) start[l] = before;
    }
    if (SCATTER) {
      __syncthreads();
      if (active) order[start[bin] + rank] = (u32)row;
    }
    __syncthreads();
  }
}

// bins[b] = number of rows in longer classes than b: where class b starts in the sorted order.
// One block.
__global__ __launch_bounds__(kBlockThreads) void k_xw_order_scan(u32* __restrict__ bins) {
  constexpr int PER = kLenBins / kBlockThreads;
  __shared__ u32 part[kBlockThreads];
  const int t = (int)threadIdx.x;
  // thread t owns the classes kLenBins-1 - (t*PER + i), i = 0..PER-1, i.e. the order longest first
  u32 own[PER], sum = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    own[i] = bins[kLenBins - 1 - (t * PER + i)];
    sum += own[i];
  }
  part[t] = sum;
  __syncthreads();
  for (int d = 1; d < kBlockThreads; d <<= 1) {
    u32 add = t >= d ? part[t - d] : 0u;
    __syncthreads();
    part[t] += add;
    __syncthreads();
  }
  u32 run = part[t] - sum;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    bins[kLenBins - 1 - (t * PER + i)] = run;
    run += own[i];
  }
}

// The product of the listed table entries of every row. A row's list is cut into 2^seg_shift segments of
// near-equal length and one lane group multiplies one segment (few rows with long lists would otherwise
// leave most of the chip idle); with one segment the group writes the canonical result to out[row], else
// its lazy partial product to partial[row][segment] for k_xw_combine. Work items are taken in the order
// `order` (rows with the longest lists first): a wavefront takes the run of its own index first, then
// runs drawn from a counter (zero at launch), so that long lists do not leave the rest of the chip waiting.
// PAIR: the table entries are pairs modulo M (see Elem); a finished product leaves the pair form (`leave` = the
// pair constant R_N) and is stored as the canonical integer, the form of a stored ciphertext.
template <int LPT, int T, bool PAIR>
__device__ __forceinline__ void xw_store_result(u32* dst, Elem<LPT, PAIR>& acc, bool active, const u32* leave,
                                                const ModRegs<LPT>& mod, const Grp<T>& g) {
  if constexpr (PAIR) {
    pairmul_mem<LPT, T>(acc.x0, acc.x1, acc.x0, acc.x1, leave, mod.n, mod.n0inv, g);
    pair_canonical<LPT, T>(acc.x0, acc.x1, mod.n, g);
    u32 lo[LPT], hi[LPT];
    pair_to_integer<LPT, T>(lo, hi, acc.x0, acc.x1, mod.n, g);
    if (active) {
      store_limbs<LPT, T>(dst, lo, g);
      store_limbs<LPT, T>(dst + LPT * T, hi, g);
    }
  } else {
    canonicalise<LPT, T>(acc.x0, mod.n, g);
    if (active) store_limbs<LPT, T>(dst, acc.x0, g);
  }
}

// The same from the residue engine's columns, those of row order[at + i], if there is an order, at place i. From *filled on the rows
// of the order are empty: one (r1, as it is stored), and no columns.
template <int LPT, int T>
__global__ __launch_bounds__(kBlockThreads, 4) void k_xw_leave(ModRef M, const u32* __restrict__ leave,
                                                               const long long* __restrict__ columns, int stride,
                                                               size_t rows, const u32* __restrict__ order, size_t at,
                                                               const u32* __restrict__ filled,
                                                               const u32* __restrict__ r1, u32* __restrict__ out) {
  constexpr int EL = 2 * LPT * T;
  const size_t products = !order ? rows : *filled > at ? *filled - at : 0;
  Grp<T> g;
  Batch<T> bt;
  ModRegs<LPT> mod;
  load_mod<LPT, T>(mod, M, g);
  for (size_t base = bt.first(); base < rows; base += bt.stride()) {
    const size_t row = base + bt.gib;
    const bool active = row < rows, product = active && row < products;
    u32* to = out + (!active ? 0 : order ? order[at + row] : row) * (size_t)EL;
    if (active && !product)
      for (int i = g.k; i < EL; i += T) to[i] = r1[i];
    if (!wave_any(product)) continue;
    const long long* src = columns + (product ? row : 0) * (size_t)(2 * stride);
    Elem<LPT, true> acc;
    load_columns<LPT, T>(acc.x0, src, g);
    load_columns<LPT, T>(acc.x1, src + stride, g);
    xw_store_result<LPT, T, true>(to, acc, product, leave, mod, g);
  }
}

template <int LPT, int T, bool PAIR>
__global__ __launch_bounds__(kBlockThreads, 3) void k_xw_main(ModRef M, const u32* __restrict__ one,
                                                           const u32* __restrict__ leave, size_t rows,
                                                           size_t list_stride, const u32* __restrict__ lists,
                                                           const u32* __restrict__ counts,
                                                           const u32* __restrict__ order,
                                                           const u32* __restrict__ tables, u32* __restrict__ next_item,
                                                           int seg_shift, u32* __restrict__ partial,
                                                           u32* __restrict__ out) {
  using Ops = ElemOps<LPT, T, PAIR>;
  constexpr int EL = Ops::kLimbs;
  constexpr int GW = WAVE / T;
  Grp<T> g;
  ModRegs<LPT> mod;
  load_mod<LPT, T>(mod, M, g);
  const int lane = (int)(threadIdx.x & (WAVE - 1));
  const size_t nwaves = ((size_t)gridDim.x * blockDim.x) / WAVE;
  const size_t items = rows << seg_shift;
  const u32 nseg = 1u << seg_shift;
  size_t w0 = (((size_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE) * GW;
  while (w0 < items) {
    const size_t item = w0 + (size_t)(lane / T);
    const bool active = item < items;
    const size_t row = active ? (size_t)order[item >> seg_shift] : 0;
    const u32 seg = (u32)item & (nseg - 1u);
    const u32 cnt = active ? counts[row] : 0u;
    const u32 e0 = (u32)(((u64)cnt * seg) >> seg_shift), e1 = (u32)(((u64)cnt * (seg + 1u)) >> seg_shift);
    const u32* mine = lists + row * list_stride;
    auto entry = [&](u32 e) -> const u32* { return (e < e1) ? tables + (size_t)mine[e] * EL : one; };
    typename Ops::E acc;
    Ops::load(acc, entry(e0), g);
#pragma unroll 1
    for (u32 e = e0 + 1; wave_any(e < e1); ++e) {
      // the next entry is looked up and touched while this one is multiplied; a group that has run out
      // of entries multiplies by one and stays in step with its wave
      const u32 touch = Ops::touch(entry(e + 1), g);
      Ops::mul_mem(acc, entry(e), mod, g);
      keep_live(touch);
    }
    if (seg_shift == 0) {
      xw_store_result<LPT, T, PAIR>(out + row * (size_t)EL, acc, active, leave, mod, g);
    } else if (active) {
      Ops::store(partial + ((row << seg_shift) + seg) * (size_t)EL, acc, g);
    }
    u32 drawn = 0;
    if (lane == 0) drawn = atomicAdd(next_item, (u32)GW);
    w0 = nwaves * GW + (size_t)(u32)__builtin_amdgcn_ds_bpermute(0, (int)drawn);
  }
}

// out[row] = product of the row's 2^seg_shift partial products, canonical
template <int LPT, int T, bool PAIR>
__global__ __launch_bounds__(kBlockThreads) void k_xw_combine(ModRef M, const u32* __restrict__ leave, size_t rows,
                                                              int seg_shift, const u32* __restrict__ partial,
                                                              u32* __restrict__ out) {
  using Ops = ElemOps<LPT, T, PAIR>;
  constexpr int EL = Ops::kLimbs;
  Grp<T> g;
  Batch<T> bt;
  ModRegs<LPT> mod;
  load_mod<LPT, T>(mod, M, g);
  for (size_t base = bt.first(); base < rows; base += bt.stride()) {
    const size_t row = base + bt.gib;
    const bool active = row < rows;
    const u32* mine = partial + ((active ? row : 0) << seg_shift) * (size_t)EL;
    typename Ops::E acc;
    Ops::load(acc, mine, g);
#pragma unroll 1
    for (int sgm = 1; sgm < (1 << seg_shift); ++sgm) Ops::mul_mem(acc, mine + (size_t)sgm * EL, mod, g);
    xw_store_result<LPT, T, PAIR>(out + (active ? row : 0) * (size_t)EL, acc, active, leave, mod, g);
  }
}

// ---------------------------------------------------------------------------
// summation
// ---------------------------------------------------------------------------
template <int LPT, int T>
__global__ __launch_bounds__(kBlockThreads) void k_sum(ModRef M, const u32* __restrict__ in, size_t count,
                                                       u32* __restrict__ out, int canonical) {
  constexpr int NL = LPT * T;
  __shared__ u32 lds[(kBlockThreads / 2) * LPT];
  Grp<T> g;
  Batch<T> bt;
  ModRegs<LPT> mod;
  load_mod<LPT, T>(mod, M, g);
  u32 acc[LPT], t[LPT];
  load_limbs<LPT, T>(acc, M.r1, g);
  for (size_t base = bt.first(); base < count; base += bt.stride()) {
    size_t item = base + bt.gib;
    const u32* src = item < count ? in + item * (size_t)NL : M.r1;
    load_limbs<LPT, T>(t, src, g);
    montmul<LPT, T>(acc, acc, t, mod.n, mod.n0inv, g);
  }
  block_product<LPT, T>(acc, lds, mod, bt, g);
  if (canonical) canonicalise<LPT, T>(acc, mod.n, g);
  if (bt.gib == 0) store_limbs<LPT, T>(out + (size_t)blockIdx.x * NL, acc, g);
}

// batches of 29 division steps that always suffice for the modulus n
int inverse_batches(const haflo_ctx* ctx) {
  size_t bits = ctx->Nw.mod.bits();
  size_t steps = (49 * bits + 57) / 17;
  return (int)((steps + LIMB_BITS - 1) / LIMB_BITS);
}

struct XtdPlan {
  int rsplit;
  size_t off_tables, off_partials, off_P, total;  // in u32 words; word 0 holds the largest |x|
};
XtdPlan xtd_plan(const haflo_ctx* ctx, size_t rows, size_t cols) {
  XtdPlan p;
  const int gpb = kBlockThreads / ctx->N.t;
  // aim at ~4 blocks per compute unit assuming 4 live digit positions, keep >= 2 rows per group
  size_t want = ((size_t)ctx->num_cu * 4 + cols * 4 - 1) / (cols ? cols * 4 : 1);
  size_t maxsplit = rows / ((size_t)gpb * 2);
  if (want > maxsplit) want = maxsplit;
  if (want < 1) want = 1;
  if (want > 64) want = 64;
  p.rsplit = (int)want;
  const size_t nl = (size_t)ctx->N.nl;
  p.off_tables = 64;
  p.off_partials = p.off_tables + rows * kSEntries * nl;
  p.off_P = p.off_partials + cols * kSMaxPos * 2 * (size_t)p.rsplit * nl;
  p.total = p.off_P + cols * 2 * nl;
  return p;
}

// The bucket method forms one product per exponent digit instead of four or five, and no tables, but folds some thousand buckets per
// column and digit position, and takes more memory, which a call on few rows never asked for: below a number of rows, a setting of
// the context (haflo_ctx_set_xtd_bucket_min_rows), the tables' workspace is enough. Unless that number was set, such a call asks for
// the buckets' as well, up to kShortWords of it, and takes them when it gets it. us, tables / buckets on limbs / in residues:
//   1024 bits, two digits: 1 by 1 354 / 266, 64 by 64 450 / 437, 600 by 16 443 / 389, 1000 by 128 828 / 810, 4000 by 16 980 / 488, 1 by
//   1024 2512 / 747, 64 by 1024 2537 / 1569; one digit, 5 % of the entries: 1000 by 16 338 / 375, 1000 by 256 1476 / 552.
//   2048 bits, two digits: 1 by 1 620 / 483 / 435, 64 by 16 657 / 645 / 507, 64 by 64 805 / 914 / 641, 1000 by 16 1598 / 778 / 582, 1 by
//   1024 4139 / 1730 / 2125; one digit, 5 %: 64 by 64 653 / 600 / 514, 1000 by 16 659 / 656 / 503.
//   4096 bits, two digits: 1 by 1 1496 / 1050 / 994, 64 by 64 1954 / 1971 / 1544, 64 by 512 5373 / 5119 / 5407, 1000 by 4 4809 / 1415 /
//   1142, 4000 by 64 8873 / 4443 / 2710; one digit, 5 %: 64 by 64 1444 / 1361 / 1084, 64 by 512 5003 / 2822 / 1815.
// In residues they are the quicker everywhere, or within 2 % of it (4096 bits, some 64 by 512); on limbs where an entry has two digits, as
// those of fixed-point features have, but for what few_rows_on_limbs() leaves out. With dense entries of one digit, which is one
// position to the tables, limbs lose up to a third on up to 64 columns (1024 bits, 1000 by 16 345 / 462).
// kShortWords is a line of memory and not of speed: from it on limbs where they are below it, then tables. 4096 bits, 4000 by 80 (942 MB on
// limbs, 1987 in residues) 10.5 / 5.6 / 3.1 ms, by 96 (1129, 2385) 15.0 / 6.4 / 3.5, by 256 (2803, 5959) 45.5 / 14.0 / 7.7; tables take
// 84 MB. What few rows cost by their columns: 1 by 64 at 4096 bits 176 MB in residues and 1.1 for tables.
constexpr size_t kShortWords = (size_t)1 << 29;  // 2 GiB
// Buckets on limbs at 2048 bits, which is where contexts with the private key have them: the middle, where the folds of that many columns
// fill the chip, but not yet the tables' products. us, tables / buckets, two digits an entry: 16 by 64 775 / 769, 24 by 64 776 / 827, 64
// by 16 657 / 645, 64 by 24 663 / 724, 128 by 96 995 / 1278, 192 by 96 1437 / 1291, 192 by 128 1160 / 1386, 512 by 160 1660 / 1833, 700
// by 160 1844 / 1852, 96 by 192 1401 / 1577, 96 by 256 1687 / 1765, 96 by 512 2746 / 2496. At 1024 bits there is no such middle. At
// 4096 tables gain up to 14 % in it with all entries of two digits and lose 8 to 29 % with three in ten.
bool few_rows_on_limbs(const haflo_ctx* ctx, size_t rows, size_t cols) {
  if (ctx->Nh.nl != 72 || rows <= 16 || cols >= 224) return true;
  return rows < 160 ? cols < 24 : rows >= 640 || cols < 112;
}
bool needs_buckets(const haflo_ctx* ctx, size_t rows, size_t cols) {
  const size_t from = ctx->xtd_bucket_min_rows ? ctx->xtd_bucket_min_rows : (size_t)HAFLO_XTD_BUCKET_MIN_ROWS_DEFAULT;
  return rows >= from && rows > 0 && xtd_buckets_fit(rows, cols);
}
bool may_use_buckets(const haflo_ctx* ctx, size_t rows, size_t cols) {
  return needs_buckets(ctx, rows, cols) || (!ctx->xtd_bucket_min_rows && rows > 0 && xtd_buckets_fit(rows, cols));
}
struct XtdBucketLayout {
  size_t off_P, off_ws, total;  // in u32 words; word 0 holds the largest |x|
};
XtdBucketLayout xtd_bucket_layout(const haflo_ctx* ctx, size_t rows, size_t cols, bool residues) {
  XtdBucketLayout l;
  l.off_P = 64;
  l.off_ws = (l.off_P + cols * 2 * (size_t)ctx->N.nl + 63) & ~(size_t)63;
  l.total = l.off_ws + xtd_bucket_plan(ctx, rows, cols, residues).total;
  return l;
}

struct XwPlan {
  // in u32 words; word 0 holds the largest |x|, word 1 the row counter of k_xw_main, words
  // [kXwBinsAt, kXwBinsAt + kLenBins) the length classes
  size_t off_inv, off_tables, off_nz, off_cnt, off_order, off_partial, total;
  int seg_shift;  // every row's list is multiplied in 2^seg_shift segments
  // in the residue form word 2 is a counter too, from 8 on there is what the device finds about programs and chains
  size_t off_pairs, off_portions, off_powers, off_chains, off_items, off_columns;
  size_t portion;  // rows whose products lie in columns at a time
  XwTablePlan tables;
};
constexpr size_t kXwControlAt = 8;
constexpr size_t kXwBinsAt = 64;
// Segments per row: doubled while the chip would hold fewer than four wavefronts per SIMD, up to 8
// and while a full row still gives every segment a few entries.
int xw_seg_shift(const haflo_ctx* ctx, size_t rows, size_t cols) {
  const size_t per_wave = (size_t)(64 / ctx->N.t), want_waves = (size_t)ctx->num_cu * 32;
  int sh = 0;
  while (sh < 3 && (rows << sh) < want_waves * per_wave && cols >= ((size_t)4 << sh)) ++sh;
  return sh;
}
XwPlan xw_plan(const haflo_ctx* ctx, size_t rows, size_t cols) {
  XwPlan p = {};
  const size_t nl = (size_t)ctx->N.nl;
  p.off_inv = kXwBinsAt + kLenBins;
  p.off_tables = p.off_inv + cols * nl;
  p.off_nz = p.off_tables + cols * 2 * kMaxPos * kWinEntries * nl;
  p.off_cnt = p.off_nz + rows * cols * kMaxPos;
  p.off_order = p.off_cnt + rows;
  p.off_partial = p.off_order + rows;
  p.seg_shift = xw_seg_shift(ctx, rows, cols);
  p.total = p.off_partial + (p.seg_shift ? (rows << p.seg_shift) * nl : 0);
  return p;
}
// Tables and rows in the residue form. Whole calls on limbs / in residues, ms, 70 % zeros. 2048 bits: 65536 by 1 0.482 / 0.492, 16384
// by 2 0.408 / 0.406; 40000 by 4 0.62 / 0.50, 4096 by 8 0.46 / 0.40, 1000 by 64 0.62 / 0.46, 64 by 256 1.11 / 0.62, 65536 by 32
// 1.89 / 0.99, 16384 by 256 3.78 / 1.69. 4096 bits: 65536 by 1 1.19 / 1.30; 64 by 4 0.79 / 0.80, 4096 by 4 0.84 / 0.87, 65536 by 4 1.45
// / 1.36, 1000 by 8 0.87 / 0.87, 4096 by 16 1.16 / 0.97, 2000 by 32 1.29 / 1.02, 300 by 48 1.34 / 1.01, 16384 by 64 3.70 / 2.00. At
// 1024 bits limbs are the quicker: 16384 by 64 0.54 / 0.69. The shape does not say how many entries are zero, nor how large they are.
// At 4096 bits none zero, 64 by 4 0.93 / 0.86, 65536 by 4 3.3 / 2.1; 5 % of one digit, 64 by 4 0.68 / 0.72, 4096 by 4 0.72 / 0.74, 65536
// by 4 0.98 / 0.85, by 16 1.06 / 1.07.
// List places and table entries are 32-bit. An entry takes twice the memory of limbs: beyond 2048 columns (tables of 5 GB at 2048
// bits, 10 at 4096) limbs. Rows take no more than on limbs but for one portion's columns (xw_portion) and 16 bytes each.
bool xw_in_residues(const haflo_ctx* ctx, size_t rows, size_t cols) {
  if (!ctx->Nh.d_rns || rows >= (1u << 28) || cols > 2048 || rows > 0xFFFFFFFFull / kMaxPos / (cols ? cols : 1)) return false;
  return ctx->Nh.nl >= 72 && cols >= 4;
}
// Segments per row: doubled while the engine has no more than its fill of chains, and a list of 30 % a few factors a chain. A
// compute unit has 192 chains in flight at 2048 bits and 16 at 4096, where a further segment's product weighs more: 20000 by 64 with
// 30 % of four digits 3.55 ms at up to 256 chains to a compute unit, 3.47 at 64, 3.48 at 16; with 5 % of one digit 1.52, 1.28, 1.27;
// 5000 by 64 with 30 % 1.94, 1.91, 2.23.
int xw_residue_shift(const haflo_ctx* ctx, size_t rows, size_t cols) {
  int sh = 0;
  const size_t fill = (size_t)ctx->num_cu * (ctx->Nh.nl == 144 ? 64 : 256);
  while (sh < 5 && (rows << sh) < fill && cols >= ((size_t)16 << sh)) ++sh;
  return sh;
}
// Rows that leave the residue form at a time: at most 524288 on 256 compute units, 0.6 GB of columns at 2048 bits and 1.2 at 4096, in
// portions of one size. A further portion costs some 45 us (1000000 rows by 4 at 2048 bits 2.78 ms in one, 2.82 in two, 2.95 in
// four, 3.41 in sixteen). Far more than what is cut into segments.
size_t xw_portion(const haflo_ctx* ctx, size_t rows) {
  const size_t most = (size_t)ctx->num_cu * 2048, portions = (rows + most - 1) / most;
  return portions > 1 ? ((rows + portions - 1) / portions + 15) & ~(size_t)15 : most;
}
XwPlan xw_residue_plan(const haflo_ctx* ctx, size_t rows, size_t cols) {
  XwPlan p = {};
  const size_t nl = (size_t)ctx->N.nl, item = rns_item_words(ctx->Nh), tabs = cols * 2 * kMaxPos;
  const auto aligned = [](size_t w) { return (w + 63) & ~(size_t)63; };
  p.seg_shift = xw_residue_shift(ctx, rows, cols);
  const size_t chains = (rows << p.seg_shift) + (p.seg_shift ? rows : 0);
  p.portion = xw_portion(ctx, rows);
  p.off_inv = kXwBinsAt + kLenBins;
  p.off_pairs = p.off_inv + cols * nl;
  size_t at = p.off_pairs + (cols * 2 + 1) * nl;
  const size_t words[4] = {cols * 2 * kNibbles, (cols * 2 + 1) * kNibbles, cols * 2 * kNibbles * 15, tabs * kMixed * 2};
  size_t* const parts[4] = {&p.tables.operands, &p.tables.places[0], &p.tables.places[1], &p.tables.index};
  for (int i = 0; i < 4; ++i) {
    *parts[i] = at;
    at += words[i];
  }
  p.tables.control = kXwControlAt;
  p.tables.live = kXwControlAt + 2 * kChainsControl;
  p.off_portions = at;
  p.off_nz = at + (rows + p.portion - 1) / p.portion * kPortionWords;
  p.off_cnt = p.off_nz + rows * cols * kMaxPos;
  p.off_order = p.off_cnt + rows;
  p.off_chains = p.tables.chains = aligned(p.off_order + rows);
  p.off_powers = aligned(p.off_chains + std::max(tabs * kMixed, chains) * 4);
  p.off_items = p.off_powers + (cols * 2 + 1) * kNibbles * item;
  p.off_partial = p.off_items + tabs * kWinEntries * item;
  p.off_columns = p.off_partial + (p.seg_shift ? (rows << p.seg_shift) * item : 0);
  p.total = p.off_columns + std::min(rows, p.portion) * 4 * (size_t)rns_columns(ctx->Nh);
  return p;
}
// what a call asks for where the residue engine serves it (its start is aligned to 256 bytes), else 0
size_t ws_xw_residues(const haflo_ctx* ctx, size_t rows, size_t cols) {
  return xw_in_residues(ctx, rows, cols) ? xw_residue_plan(ctx, rows, cols).total * 4 + 256 : 0;
}

// X^T [[d]]: what a call can do with, and what it asks for where it takes the bucket method, on limbs or in residues (else 0)
size_t ws_xtd_min(const haflo_ctx* ctx, size_t rows, size_t cols) {
  if (!cols) return 0;
  return (needs_buckets(ctx, rows, cols) ? xtd_bucket_layout(ctx, rows, cols, false).total : xtd_plan(ctx, rows, cols).total) * 4;
}
size_t ws_xtd_buckets(const haflo_ctx* ctx, size_t rows, size_t cols, bool residues) {
  if (!cols || !may_use_buckets(ctx, rows, cols) || (residues && !xtd_buckets_in_residues(ctx, rows, cols))) return 0;
  const size_t words = xtd_bucket_layout(ctx, rows, cols, residues).total;
  const bool few = !needs_buckets(ctx, rows, cols);
  if (few && (words > kShortWords || !(residues || few_rows_on_limbs(ctx, rows, cols)))) return 0;
  return words * 4 + (residues || few ? 256 : 0);  // their start is aligned to 256 bytes
}

// The tables of 256 entries per base and position, and `chains` as the rows' products need it
int xw_residue_tables(const haflo_ctx* ctx, const XwPlan& p, const u32* d_c, size_t cols, u32* ws, RnsChains& chains,
                      hipStream_t st) {
  const ModHost& mh = ctx->Nh;
  const size_t tabs = cols * 2 * kMaxPos;
  const XwTablePlan& t = p.tables;
  const LaunchShape sh = launch_shape(ctx, cols * 2, 2 * mh.t, 8);
  const u32* lo = mh.d_pairs + (size_t)kConstMLo * 2 * mh.nl;
  const u32* hi = mh.d_pairs + (size_t)kConstMHi * 2 * mh.nl;
  u32* pairs = ws + p.off_pairs;
#define CALL(LPT, T) \
  HAFLO_LAUNCH((k_to_pairs<LPT, T>), sh, st, mh.ref(), lo, hi, d_c, (const u32*)(ws + p.off_inv), cols, cols * 2, pairs)
  HAFLO_DISPATCH_PAIRS(mh, CALL);
#undef CALL
  HAFLO_LAUNCH(k_xw_places, launch_shape(ctx, tabs * kMixed, 1, 8), st, (u32)cols, ws, t,
               (const u32*)(mh.d_pairs + (size_t)kConstMOne * 2 * mh.nl), (u32)(2 * mh.nl), pairs + cols * 4 * mh.nl, (const u32*)ws);
  const u32* one = ws + p.off_powers + cols * 2 * kNibbles * rns_item_words(mh);
  for (int i = 0; i < 2; ++i) {
    RnsLists j = {};
    j.places = ws + t.places[i];
    j.stride = i ? cols * 2 * kNibbles : cols * 2 + 1;
    j.live = ws + t.live + i;
    j.out = ws + (i ? p.off_items : p.off_powers);
    if (i == 0) {
      j.limit = ws + t.live + 2;
      j.limbs = pairs;
      j.add(LIST_ACC_LIMBS);
      j.add(LIST_STORE_ACC);
      for (int q = 1; q < kNibbles; ++q) {
        j.add(LIST_ACC_SQ, 4);
        j.add(LIST_STORE_ACC);
      }
    } else {
      j.items = ws + p.off_powers;
      j.one = one;
      j.operands = ws + t.operands;
      j.rows = 1;
      j.add(LIST_RUN_ITEM);
      for (int d = 1; d < 16; ++d) {
        j.add(LIST_ACC_RUN);
        j.add(LIST_STORE_ACC);
      }
    }
    if (int rc = rns_lists(ctx, mh, j, j.stride, st)) return rc;
  }
  chains.items = ws + p.off_items;
  chains.one = one;
  chains.chains = ws + t.chains;
  chains.index = ws + t.index;
  chains.control = ws + t.control;
  chains.next = ws + 2;
  chains.out = ws + p.off_items;
  return rns_chains(ctx, mh, chains, tabs * kMixed, tabs / 2 * kMixed, st);
}

int sum_blocks(const haflo_ctx* ctx, size_t count) {
  const int gpb = kBlockThreads / ctx->N.t;
  size_t need = (count + (size_t)gpb * 4 - 1) / ((size_t)gpb * 4);
  size_t cap = (size_t)ctx->num_cu * 4;
  if (need < 1) need = 1;
  return (int)(need < cap ? need : cap);
}

int launch_maxmag(const haflo_ctx* ctx, const int32_t* X, size_t total, u32* word, int zero_words, hipStream_t st) {
  LaunchShape one;
  one.blocks = 1;
  one.threads = kBlockThreads;
  one.gpb = kBlockThreads;
  HAFLO_LAUNCH(k_zero_word, one, st, word, zero_words);
  if (total) {
    LaunchShape sh = launch_shape(ctx, (total + 15) / 16, 1, 8);  // sixteen entries per lane: few wavefronts, few atomics
    HAFLO_LAUNCH(k_maxmag, sh, st, X, total, word);
  }
  return hip_status(hipGetLastError());
}

// Launch shape and geometry of a short, latency-bound kernel over `count` big integers modulo `m`: one
// wavefront per integer while every integer can have a SIMD to itself, else twice the lanes per integer
// while the chip is mostly idle, else the modulus's own geometry.
LaunchShape latency_shape(const haflo_ctx* ctx, size_t count, const ModHost& m) {
  LaunchShape sh;
  if (haflo_has_wave_geometry(m) && count <= (size_t)ctx->num_cu * 4) {
    sh.blocks = (int)(count ? count : 1);
    sh.threads = 64;
    sh.gpb = 1;
    sh.geo = kGeoWave;
    return sh;
  }
  const bool wide = haflo::few_groups(ctx, count);
  sh = launch_shape(ctx, count, wide ? haflo_wide_lanes(m) : m.t, 8);
  sh.geo = wide ? kGeoWide : kGeoPlain;
  return sh;
}
#define HAFLO_DISPATCH_SHAPE(sh, m, CALL)                                    \
  do {                                                                       \
    if ((sh).geo == kGeoWave) { HAFLO_DISPATCH_GEOMETRY_WAVE(m, CALL); }     \
    else if ((sh).geo == kGeoWide) { HAFLO_DISPATCH_GEOMETRY_WIDE(m, CALL); } \
    else { HAFLO_DISPATCH_GEOMETRY(m, CALL); }                               \
  } while (0)

}  // namespace

namespace haflo {

int invert_batch(const haflo_ctx* ctx, const uint32_t* in, uint32_t* out, size_t count, hipStream_t st) {
  const ModHost& m = ctx->N;
  const LaunchShape sh = latency_shape(ctx, count, m);
  const int nbatch = inverse_batches(ctx);
#define CALL(LPT, T) HAFLO_LAUNCH((k_invert<LPT, T>), sh, st, m.ref(), ctx->Nw.ref(), in, out, count, nbatch)
  HAFLO_DISPATCH_SHAPE(sh, m, CALL);
#undef CALL
  return hip_status(hipGetLastError());
}

}  // namespace haflo

extern "C" {

size_t haflo_workspace_bytes(const haflo_ctx* ctx, int op, size_t rows, size_t cols) {
  if (!ctx) return (size_t)-1;
  switch (op) {
    case HAFLO_OP_ENCRYPT: return ws_encrypt(ctx, rows);
    case HAFLO_OP_DECRYPT: return ctx->has_priv ? ws_decrypt(ctx, rows) : (size_t)-1;
    case HAFLO_OP_SCALAR_MUL: return ws_scalar_mul(ctx, rows);
    case HAFLO_OP_TAYLOR_LOSS: return ws_taylor_loss(ctx, rows);
    case HAFLO_OP_ENCRYPT_OBFUSCATOR: return ws_encrypt_obf(ctx, rows);
    case HAFLO_OP_FORE_GRADIENT:
      return ((rows * (size_t)ctx->lp * 4 + 255) & ~(size_t)255) + ((rows * (size_t)ctx->N.nl * 4 + 255) & ~(size_t)255) +
             ws_encrypt(ctx, rows);
    case HAFLO_OP_MATVEC_XT_D:
      return std::max({ws_xtd_min(ctx, rows, cols), ws_xtd_buckets(ctx, rows, cols, false), ws_xtd_buckets(ctx, rows, cols, true)});
    case HAFLO_OP_MATVEC_X_W: return std::max(xw_plan(ctx, rows, cols).total * 4, ws_xw_residues(ctx, rows, cols));
    case HAFLO_OP_SUM_SEGMENTS:
      if (rows >= (1ull << 32) || cols >= (1ull << 24)) return (size_t)-1;
      return cols ? seg_sum_plan(ctx, rows, cols).total * 4 : 0;
    default: return (size_t)-1;
  }
}

size_t haflo_workspace_bytes_least(const haflo_ctx* ctx, int op, size_t rows, size_t cols) {
  const size_t asked = haflo_workspace_bytes(ctx, op, rows, cols);
  if (asked == (size_t)-1) return asked;
  switch (op) {
    case HAFLO_OP_ENCRYPT: return ws_encrypt_min(ctx, rows);
    case HAFLO_OP_DECRYPT: return ws_decrypt_min(ctx, rows);
    case HAFLO_OP_SCALAR_MUL: return ws_scalar_mul_min(ctx, rows);
    case HAFLO_OP_MATVEC_XT_D: return ws_xtd_min(ctx, rows, cols);
    case HAFLO_OP_MATVEC_X_W: return xw_plan(ctx, rows, cols).total * 4;
    case HAFLO_OP_FORE_GRADIENT: return asked - ws_encrypt(ctx, rows) + ws_encrypt_min(ctx, rows);
    case HAFLO_OP_TAYLOR_LOSS: return ws_taylor_loss_min(ctx, rows);
    default: return asked;
  }
}

int haflo_cipher_matvec(const haflo_ctx* ctx, int orientation, const void* d_c, const int32_t* d_X, size_t rows,
                        size_t cols, void* d_out, void* d_workspace, size_t workspace_bytes, void* stream) {
  if (!ctx || (orientation != 0 && orientation != 1)) return HAFLO_EINVAL;
  const size_t nin = orientation == 0 ? rows : cols;
  const size_t nout = orientation == 0 ? cols : rows;
  if (nout == 0) return HAFLO_OK;
  if (!d_out || (nin && (!d_c || !d_X))) return HAFLO_EINVAL;
  const ModHost& m = ctx->N;
  hipStream_t st = (hipStream_t)stream;
  const size_t need = haflo_workspace_bytes_least(ctx, orientation == 0 ? HAFLO_OP_MATVEC_XT_D : HAFLO_OP_MATVEC_X_W, rows, cols);
  if (!d_workspace || workspace_bytes < need) return HAFLO_EINVAL;
  u32* ws = (u32*)d_workspace;
  const size_t asked = orientation == 0 ? ws_xtd_buckets(ctx, rows, cols, true) : ws_xw_residues(ctx, rows, cols);
  const bool residues = asked != 0 && workspace_bytes >= asked;
  const size_t on_limbs = orientation == 0 ? ws_xtd_buckets(ctx, rows, cols, false) : 0;
  const bool buckets = orientation == 0 && (residues || (on_limbs != 0 && workspace_bytes >= on_limbs));
  if (residues || (buckets && !needs_buckets(ctx, rows, cols))) ws = (u32*)(((uintptr_t)ws + 255) & ~(uintptr_t)255);
  int rc = buckets ? HAFLO_OK
                   : launch_maxmag(ctx, d_X, rows * cols, ws, orientation == 0 ? 2 : (int)(kXwBinsAt + kLenBins), st);
  if (rc != HAFLO_OK) return rc;
  const int nbatch = inverse_batches(ctx);
  if (buckets) {
    const XtdBucketLayout l = xtd_bucket_layout(ctx, rows, cols, residues);
    u32* P = ws + l.off_P;
    rc = xtd_buckets(ctx, (const u32*)d_c, d_X, rows, cols, residues, ws + l.off_ws, P, st);
    if (rc != HAFLO_OK) return rc;
    const LaunchShape sh = latency_shape(ctx, cols, m);
#define CALL(LPT, T) HAFLO_LAUNCH((k_xtd_finish<LPT, T>), sh, st, m.ref(), ctx->Nw.ref(), cols, (const u32*)P, (u32*)d_out, nbatch)
    HAFLO_DISPATCH_SHAPE(sh, m, CALL);
#undef CALL
  } else if (orientation == 0) {
    const XtdPlan p = xtd_plan(ctx, rows, cols);
    u32* tables = ws + p.off_tables;
    u32* partials = ws + p.off_partials;
    u32* P = ws + p.off_P;
    if (rows) {
      rc = power_tables(ctx, (const u32*)d_c, tables, kSEntries, rows, st);
      if (rc != HAFLO_OK) return rc;
      LaunchShape mainsh;
      mainsh.threads = kBlockThreads;
      mainsh.gpb = kBlockThreads / m.t;
      mainsh.blocks = (int)(cols * ((((size_t)p.rsplit * kSMaxPos) + 7) / 8 * 8));
#define CALL(LPT, T) \
  HAFLO_LAUNCH((k_xtd_main<LPT, T>), mainsh, st, m.ref(), d_X, rows, cols, (const u32*)tables, p.rsplit, partials, (const u32*)ws)
      HAFLO_DISPATCH_GEOMETRY(m, CALL);
#undef CALL
    }
    {
      const bool wide = haflo::few_groups(ctx, cols * 2);
      const LaunchShape sh = launch_shape(ctx, cols * 2, wide ? haflo_wide_lanes(m) : m.t, 8);
#define CALL(LPT, T) \
  HAFLO_LAUNCH((k_xtd_horner<LPT, T>), sh, st, m.ref(), cols, p.rsplit, (const u32*)partials, P, (const u32*)ws)
      if (wide) { HAFLO_DISPATCH_GEOMETRY_WIDE(m, CALL); } else { HAFLO_DISPATCH_GEOMETRY(m, CALL); }
#undef CALL
    }
    {
      const LaunchShape sh = latency_shape(ctx, cols, m);
#define CALL(LPT, T) HAFLO_LAUNCH((k_xtd_finish<LPT, T>), sh, st, m.ref(), ctx->Nw.ref(), cols, (const u32*)P, (u32*)d_out, nbatch)
      HAFLO_DISPATCH_SHAPE(sh, m, CALL);
#undef CALL
    }
  } else {
    const XwPlan p = residues ? xw_residue_plan(ctx, rows, cols) : xw_plan(ctx, rows, cols);
    u32* inv = ws + p.off_inv;
    u32* tables = ws + p.off_tables;
    u32* lists = ws + p.off_nz;
    u32* cnt = ws + p.off_cnt;
    // The tables and the row products are in the pair form modulo n (5/8 of the limb products of a full-length
    // product; every supported key size has that geometry); a row's result leaves it as it is stored.
    const ModHost& mh = ctx->Nh;
    if (!haflo_has_pair_geometry(mh)) return HAFLO_EINVAL;
    const ModRef M = mh.ref();
    const int lanes = 2 * mh.t;
    const u32* one = mh.d_pairs + (size_t)kConstR1 * 2 * mh.nl;
    const u32* leave = mh.d_pairs + (size_t)kConstR3 * 2 * mh.nl;
    if (cols) {
      rc = invert_batch(ctx, (const u32*)d_c, inv, cols, st);
      if (rc != HAFLO_OK) return rc;
    }
    RnsChains chains = {};
    if (residues) {
      rc = xw_residue_tables(ctx, p, (const u32*)d_c, cols, ws, chains, st);
      if (rc != HAFLO_OK) return rc;
    } else if (cols) {
      // The squarings and the first levels are as many products as there are launches and positions, on few pairs: the
      // latency of a product bounds them, so a wavefront for each pair while launch_pairs allows. 1000 rows by 32 columns
      // 0.40 -> 0.35 ms at 1024 bits and 0.74 -> 0.65 at 2048, 300 by 32 at 4096 bits 1.57 -> 1.42, 16384 by 256 at 2048
      // 3.60 -> 3.48 (256 columns are the last whose squarings fit: 64 rows by 256 | 300 at 1024 bits 0.78 -> 0.74 | 0.86).
      bool wave;
      {
        const LaunchShape sh = launch_pairs(ctx, mh, cols * 2 * kMaxPos, lanes, wave);
#define CALL(LPT, T)                                                                                                \
  HAFLO_LAUNCH((k_xw_positions<LPT, T, true>), sh, st, M, (const u32*)(mh.d_pairs + (size_t)kConstR4 * 2 * mh.nl), \
               (const u32*)(mh.d_pairs + (size_t)kConstR5 * 2 * mh.nl), (const u32*)d_c, (const u32*)inv, cols,     \
               tables, (const u32*)ws)
        HAFLO_DISPATCH_PAIRS_FEW(mh, wave, CALL);
#undef CALL
      }
      for (int B = 1; B < kWinEntries; B *= 2) {
        const size_t groups = cols * 2 * kMaxPos * (size_t)std::min(B, kWinEntries - 1 - B);
        const LaunchShape sh = launch_pairs(ctx, mh, groups, lanes, wave);
#define CALL(LPT, T) HAFLO_LAUNCH((k_xw_level<LPT, T, true>), sh, st, M, one, cols, B, tables, (const u32*)ws)
        HAFLO_DISPATCH_PAIRS_FEW(mh, wave, CALL);
#undef CALL
      }
    }
    u32* bins = ws + kXwBinsAt;
    u32* order = ws + p.off_order;
    {
      const LaunchShape sh = launch_shape(ctx, rows, 64, 8);
      HAFLO_LAUNCH(k_xw_lists, sh, st, d_X, rows, cols, lists, cnt, (const u32*)ws);
      LaunchShape per_row, single;
      per_row.threads = single.threads = kBlockThreads;
      per_row.gpb = single.gpb = kBlockThreads;
      per_row.blocks = (int)std::min((rows + kBlockThreads - 1) / kBlockThreads, (size_t)ctx->num_cu * 8);
      single.blocks = 1;
      HAFLO_LAUNCH(k_xw_order<false>, per_row, st, (const u32*)cnt, rows, cols, bins, order, (const u32*)ws);
      HAFLO_LAUNCH(k_xw_order_scan, single, st, bins);
      HAFLO_LAUNCH(k_xw_order<true>, per_row, st, (const u32*)cnt, rows, cols, bins, order, (const u32*)ws);
    }
    u32* partial = ws + p.off_partial;
    if (residues) {
      u32* control = ws + kXwControlAt + kChainsControl;
      u32* portions = ws + p.off_portions;
      const u32* filled = bins + 1;  // the end of the shortest class that is not empty
      HAFLO_LAUNCH(k_xw_chains, launch_shape(ctx, rows << p.seg_shift, 1, 8), st, rows, cols * (size_t)kMaxPos, p.seg_shift,
                   p.portion, (const u32*)cnt, (const u32*)order, filled, (uint4*)(ws + p.off_chains), control, portions);
      chains.chains = ws + p.off_chains;
      chains.index = lists;
      chains.out = partial;
      chains.columns = (long long*)(ws + p.off_columns);
      if (p.seg_shift) {
        chains.control = control;
        chains.next = ws + 1;
        rc = rns_chains(ctx, mh, chains, rows << p.seg_shift, rows << p.seg_shift, st);
        if (rc != HAFLO_OK) return rc;
        chains.items = partial;
        chains.chains += (rows << p.seg_shift) * 4;
        chains.index = nullptr;
      }
      for (size_t at = 0; at < rows; at += p.portion) {
        const size_t count = std::min(rows - at, p.portion);
        chains.control = portions + at / p.portion * kPortionWords;
        chains.next = portions + at / p.portion * kPortionWords + kPortionNext;
        rc = rns_chains(ctx, mh, chains, count, count, st);
        if (rc != HAFLO_OK) return rc;
        chains.chains += count * 4;
        const u32* places = p.seg_shift ? nullptr : order;
        const LaunchShape sh = launch_shape(ctx, count, lanes, 8);
#define CALL(LPT, T)                                                                                            \
  HAFLO_LAUNCH((k_xw_leave<LPT, T>), sh, st, M, (const u32*)(mh.d_pairs + (size_t)kConstMStored * 2 * mh.nl),  \
               (const long long*)(ws + p.off_columns), rns_columns(mh), count, places, at, filled, ctx->N.ref().r1, (u32*)d_out)
        HAFLO_DISPATCH_PAIRS(mh, CALL);
#undef CALL
      }
      return hip_status(hipGetLastError());
    }
    {
      const LaunchShape sh = launch_shape(ctx, rows << p.seg_shift, lanes, 3);
#define CALL(LPT, T)                                                                                            \
  HAFLO_LAUNCH((k_xw_main<LPT, T, true>), sh, st, M, one, leave, rows, cols * (size_t)kMaxPos, (const u32*)lists, \
               (const u32*)cnt, (const u32*)order, (const u32*)tables, ws + 1, p.seg_shift, partial, (u32*)d_out)
      HAFLO_DISPATCH_PAIRS(mh, CALL);
#undef CALL
    }
    if (p.seg_shift) {
      const LaunchShape sh = launch_shape(ctx, rows, lanes, 8);
#define CALL(LPT, T) \
  HAFLO_LAUNCH((k_xw_combine<LPT, T, true>), sh, st, M, leave, rows, p.seg_shift, (const u32*)partial, (u32*)d_out)
      HAFLO_DISPATCH_PAIRS(mh, CALL);
#undef CALL
    }
  }
  return hip_status(hipGetLastError());
}

int haflo_cipher_sum(const haflo_ctx* ctx, const void* d_c, size_t count, void* d_out, void* d_workspace,
                     size_t workspace_bytes, void* stream) {
  if (!ctx || !d_out || (count && !d_c)) return HAFLO_EINVAL;
  const ModHost& m = ctx->N;
  hipStream_t st = (hipStream_t)stream;
  const int nb = sum_blocks(ctx, count);
  // partial products of the first level, then of every further level, ping-pong in the workspace
  const int gpw = kBlockThreads / haflo_wide_lanes(m);  // groups per block of the later levels
  const size_t second = (size_t)(nb + gpw - 1) / gpw;
  if (!d_workspace || workspace_bytes < ((size_t)nb + second) * m.nl * 4) return HAFLO_EINVAL;
  u32* buf[2] = {(u32*)d_workspace, (u32*)d_workspace + (size_t)nb * m.nl};
  LaunchShape sh;
  sh.threads = kBlockThreads;
  sh.gpb = kBlockThreads / m.t;
  sh.blocks = nb;
  if (nb == 1) {
#define CALL(LPT, T) HAFLO_LAUNCH((k_sum<LPT, T>), sh, st, m.ref(), (const u32*)d_c, count, (u32*)d_out, 1)
    HAFLO_DISPATCH_GEOMETRY(m, CALL);
#undef CALL
    return hip_status(hipGetLastError());
  }
#define CALL(LPT, T) HAFLO_LAUNCH((k_sum<LPT, T>), sh, st, m.ref(), (const u32*)d_c, count, buf[0], 0)
  HAFLO_DISPATCH_GEOMETRY(m, CALL);
#undef CALL
  // Further levels: one partial per lane group and a tree inside the block, in the wide geometry
  // (few integers are left and every level is a chain of only log2(groups) + 1 products).
  size_t n = (size_t)nb;
  int from = 0;
  while (n > 1) {
    LaunchShape lv;
    lv.threads = kBlockThreads;
    lv.gpb = gpw;
    lv.blocks = (int)((n + gpw - 1) / gpw);
    const bool last = lv.blocks == 1;
    u32* dst = last ? (u32*)d_out : buf[from ^ 1];
    const u32* src = buf[from];
#define CALL(LPT, T) HAFLO_LAUNCH((k_sum<LPT, T>), lv, st, m.ref(), src, n, dst, last ? 1 : 0)
    HAFLO_DISPATCH_GEOMETRY_WIDE(m, CALL);
#undef CALL
    n = (size_t)lv.blocks;
    from ^= 1;
  }
  return hip_status(hipGetLastError());
}

int haflo_cipher_sum_segments(const haflo_ctx* ctx, const void* d_c, size_t count, const uint32_t* d_offsets,
                              size_t nseg, void* d_out, uint32_t* d_status, void* d_workspace, size_t workspace_bytes,
                              void* stream) {
  if (!ctx || count >= (1ull << 32) || nseg >= (1ull << 24)) return HAFLO_EINVAL;
  if (nseg == 0) return HAFLO_OK;
  if (!d_offsets || !d_out || (count && !d_c)) return HAFLO_EINVAL;
  if (!d_workspace || workspace_bytes < seg_sum_plan(ctx, count, nseg).total * 4) return HAFLO_EINVAL;
  return seg_sum(ctx, (const u32*)d_c, d_offsets, count, nseg, (u32*)d_out, d_status, (u32*)d_workspace,
                 (hipStream_t)stream);
}

}  // extern "C"
