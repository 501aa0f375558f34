// Exponentiation modulo s^2 on pairs of residues modulo s in a residue number system, with the Montgomery
// reductions as matrix products of bytes on the matrix cores.
//
// A pair product (see pairmul_core) is two Montgomery reductions modulo s with the same quotient digits fed from
// the first into the second. In base A (primes a_i, radix M_A) and base B (primes b_j), rns.hpp, one of them is
//     q_i = T_i (-1/s) mod a_i,  sigma_i = q_i / (M_A / a_i) mod a_i          one residue product per prime
//     t_j = (T_j + s sum_i sigma_i M_A / a_i) / M_A mod b_j                   a constant matrix times sigma
//     t_i = sum_j rho_j M_B / b_j - alpha M_B mod a_i, rho_j = t_j / (M_B / b_j) mod b_j, alpha = round(sum rho_j / 2^30)
//                                                                             a constant matrix times rho
// (sum sigma_i M_A / a_i may exceed the quotient by a multiple of M_A: t then exceeds the reduced value by a small
// multiple of s, which M_A's 14 to 28 spare bits absorb. The second extension is exact: t is below 600 s, M_B above
// 2^14 s and the b_j within 2^-16 of 2^30, so the sum lies less than 2^-4.6 above an integer.)
// The word-serial pair product takes 3.6 (5 for a product of two elements) NL^2 multiply-adds per element; here the
// NL^2 part are four products with constant matrices over a whole batch, which the matrix cores do on the residues'
// bytes, and the vector unit is left with about 42 instructions per prime and pair squared. It issues one of them per four
// cycles, whatever it is, and loses two such slots to every matrix instruction: their number is what the kernels are built
// around. Residues are signed and reduced only as far as one Montgomery reduction goes, and the byte rows of a matrix are
// weighted so that a product's sums are the two words of what is to be reduced (rns::Matrix).
//
// Layout. Lane l of a wavefront holds a quarter (g = l / 16) of the residues of element l % 16: channel slot 4 i + g in
// register i. With the constant matrix as the first operand of v_mfma_i32_16x16x64_i8 and the residues' bytes as the
// second, four consecutive rows of a result belong to one lane: the four byte rows of one destination slot.
#include "kernels_common.hpp"
#include "rns.hpp"

using namespace haflo;
using namespace haflo::dev;

namespace {

typedef u32 Quad __attribute__((vector_size(16)));
typedef u32 Twin __attribute__((vector_size(8)));
typedef int Acc __attribute__((vector_size(16)));  // also a matrix operand of 16 bytes

template <int N>
struct QuadSet {
  Acc q[N];
};

constexpr int kRnsInline = 96;  // instructions that travel with the launch: 90 at most for a 63-bit scalar
struct RnsJob {
  const u32* tables;  // rns.hpp's device layout
  const u32* prog;    // null: `ins`; ENG_SQ, ENG_MUL_T, ENG_MUL_T_ST, ENG_STORE_T, ENG_LOAD_T only
  int len;
  // Per element [x0: nl limbs][x1: nl limbs], lazy: limbs below 2^29 + 2^8. They go into the matrix product as they are, the top
  // byte as a signed one, and the bounds of its sums (tests/test_rns_tables.py) take limbs of that size.
  const u32* in;
  int nl;
  long long* out;     // per element [x0: columns][x1: columns] of weight 2^(29 l), signed
  u32* slots;         // window tables: 4 NR dwords per lane and entry
  int entries;
  u32 ins[kRnsInline];
};

__device__ __forceinline__ s64 smad(u32 a, u32 b, s64 c) { return (s64)(s32)a * (s64)(s32)b + c; }
// 2 a b, which may take 33 bits of a factor: two multiply-adds, hidden from the compiler, which would shift a wider one
__device__ __forceinline__ s64 twice(u32 a, u32 b) {
  s64 t = smad(a, b, 0);
  asm("" : "+v"(t));
  return smad(a, b, t);
}
// T 2^-32 mod p, signed: (T + m p) / 2^32 for an m between -2^31 and 2^31
__device__ __forceinline__ u32 reduce(s64 t, u32 p, u32 pinv) {
  const u32 m = (u32)t * pinv;
  u32 r = (u32)((u64)smad(m, p, t) >> 32);
  asm("" : "+v"(r));  // a register of its own: the compiler would carry the dead low word along with it
  return r;
}

// What the sums of a tile's products start from: 2^31 in every column's lower word, which then is not negative
__device__ __forceinline__ Acc start_sums(bool kept = true) {
  Acc a = {0, rns::kStart, 0, 0};
  if (kept) asm volatile("" : "+v"(a));
  return a;
}
// the four byte rows of a slot as one number, see rns::Matrix
__device__ __forceinline__ s64 column(const Acc& acc) {
  const u32 lo = ((u32)acc[1] << 8) + (u32)acc[0];
  const u32 hi = ((u32)acc[3] << 8) + (u32)acc[2];
  s64 v = (s64)((u64)hi << 32 | lo);
  asm("" : "+v"(v));  // a pair of registers as it is: the compiler would add its halves one by one to what it is added to
  return v;
}
// the same for rows of radix 256 and sums from zero
__device__ __forceinline__ s64 integer(const Acc& acc) {
  return (((s64)acc[3] * 256 + acc[2]) * 256 + acc[1]) * 256 + acc[0];
}
// alpha, the multiple of M_B, from what it is the rounded quotient of (by 2^14), as two bytes: modulo 128 and the rest
__device__ __forceinline__ u32 alpha_bytes(u32 sum) {
  const s32 a = (s32)sum >> 14;
  return ((u32)a & 127u) | ((u32)(a >> 7) & 255u) << 8;
}

// One or two sets of 16 elements, which a wavefront works on side by side, so that a fragment of a matrix read from LDS serves
// both: the residues of x0 and x1 (PAIR; else of one value, x0) in one base, in the registers that the matrix products take
// them from: full quads of each, and one quad per set with the last two of both.
template <int NR, bool PAIR, int kSets>
struct Residues {
  static_assert(NR % 4 == 2, "full blocks and a half one");
  static constexpr int kFull = NR / 4, kHalves = PAIR ? 2 : 1;
  Quad q[kSets][kHalves][kFull];
  Quad h[kSets];
  __device__ __forceinline__ u32 get(int s, int x, int i) const {
    return i < 4 * kFull ? q[s][x][i / 4][i % 4] : h[s][2 * x + i % 4];
  }
  __device__ __forceinline__ void set(int s, int x, int i, u32 v) {
    if (i < 4 * kFull) q[s][x][i / 4][i % 4] = v;
    else h[s][2 * x + i % 4] = v;
  }
  // Gathers quad k in its registers now: left alone, the compiler keeps the values in the 64-bit results they are the
  // upper words of until all are there.
  __device__ __forceinline__ void gather(int k) {
#pragma unroll
    for (int s = 0; s < kSets; ++s) {
      if (k < kFull) {
        asm("" : "+v"(q[s][0][k]));
        if constexpr (PAIR) asm("" : "+v"(q[s][1][k]));
      } else {
        asm("" : "+v"(h[s]));
      }
    }
  }
};
template <int NR, bool PAIR, int kSets>
struct RnsState {
  Residues<NR, PAIR, kSets> a, b;
};

// The operand of a matrix product: the half block's words of x0 and of x1 in quads of their own, zeros behind them.
template <int NR, bool PAIR, int kSets>
struct Operand {
  static constexpr int kFull = NR / 4, kHalves = PAIR ? 2 : 1;
  Residues<NR, PAIR, kSets>& d;
  Quad o[kSets][kHalves];
  __device__ __forceinline__ explicit Operand(Residues<NR, PAIR, kSets>& d_) : d(d_) {
#pragma unroll
    for (int s = 0; s < kSets; ++s)
#pragma unroll
      for (int x = 0; x < kHalves; ++x) {
        o[s][x] = Quad{d.h[s][2 * x], d.h[s][2 * x + 1], 0, 0};
        asm("" : "+v"(o[s][x]));  // made once, not for every tile
      }
  }
  __device__ __forceinline__ Acc get(int s, int x, int k) const { return (Acc)(k < kFull ? d.q[s][x][k < kFull ? k : 0] : o[s][x]); }
  // back to the residues' own form
  __device__ __forceinline__ void release() {
#pragma unroll
    for (int s = 0; s < kSets; ++s)
      d.h[s] = Quad{o[s][0][0], o[s][0][1], PAIR ? o[s][kHalves - 1][0] : 0u, PAIR ? o[s][kHalves - 1][1] : 0u};
  }
};

// A modular product is two matrix products, sigma to base B and rho to base A, tile by tile (four slots, one per lane
// group). A lane gets whole residues from one, works on them alone and feeds them to the next as they are: no lane
// exchange, no LDS traffic but the matrices' and the constants', no barrier. While the matrix unit works on one tile, the
// vector unit finishes the one before.
// Between operations base A is held as residues (in a run of squarings as the next one's sigma), base B as bytes, with
// the extra sources of the last way back in their slots.
template <int NR, bool PAIR, int kSets>
struct RnsEngine {
  static constexpr int kHalves = PAIR ? 2 : 1;
  static constexpr int kFull = rns::full_blocks(NR);
  static constexpr int kTiles = rns::tiles(NR);  // also the registers that hold primes
  static constexpr int kTileBytes = rns::tile_bytes(NR, 16);
  using Res = Residues<NR, PAIR, kSets>;
  using State = RnsState<NR, PAIR, kSets>;
  using Op = Operand<NR, PAIR, kSets>;
  struct Frags {  // of a tile; of the half block only 8 bytes of a row are stored, the rest meets the operand's zeros
    Acc q[kFull + 1];
  };
  struct Sums {  // of one set
    Acc r[kHalves];
  };
  const char* lds;
  int lane, g;
  Acc start;
  // An LDS read adds at most 64 KB to an address, a matrix of 2048-bit moduli is 78 KB: two windows.
  static constexpr int kWindow = 1 << 16, kWindows = rns::lds_matrix_bytes(NR, 1) > kWindow ? 2 : 1;
  int at[kWindows], at_half[kWindows];  // this lane's part of a matrix's fragments; of half blocks
  int at_cst;                           // of this lane group's constants in a row of four slots

  __device__ __forceinline__ RnsEngine(const void* lds_)
      : lds((const char*)lds_), lane((int)(threadIdx.x & (WAVE - 1))), g(lane >> 4), start(start_sums()) {
    use_matrix<0>();
  }
  // What a wavefront reads from LDS is constant over the launch: with addresses that are made anew for each matrix
  // product the compiler does not read it once and run out of registers for it.
  template <int MATRIX>
  __device__ __forceinline__ void use_matrix() {
    int l = lane;
    asm volatile("" : "+v"(l));
#pragma unroll
    for (int w = 0; w < kWindows; ++w) {
      at[w] = MATRIX * rns::lds_matrix_bytes(NR, 0) + w * kWindow + 16 * l;
      at_half[w] = MATRIX * rns::lds_matrix_bytes(NR, 0) + w * kWindow + 8 * l;
      asm volatile("" : "+v"(at[w]), "+v"(at_half[w]));
    }
    at_cst = rns::lds_matrices_bytes(NR) + (l & 48);
    asm volatile("" : "+v"(at_cst));
  }
  // the constants of base A (0), base B's products (1) and its sums (2)
  __device__ __forceinline__ Quad cst(int base, int i) const {
    return *(const Quad*)(lds + at_cst + (base * rns::slots(NR) + 4 * i) * 16);
  }
  static __device__ __forceinline__ Acc half_fragment(const void* p) {
    const Twin h = *(const Twin*)p;
    int any0 = 0, any1 = 0;
#if defined(__HIP_DEVICE_COMPILE__)
    asm("" : "=v"(any0), "=v"(any1));
#endif
    return Acc{(int)h[0], (int)h[1], any0, any1};
  }
  template <int MATRIX>
  __device__ __forceinline__ void fragments(Frags& m, int t) const {
    constexpr int kRows = rns::last_rows(NR, MATRIX);
    if (t == kTiles - 1 && kRows != 16) {
      const char* p = lds + MATRIX * rns::lds_matrix_bytes(NR, 0) + t * kTileBytes;
      int row = (lane >> 4) * kRows + (lane & (kRows - 1));
      asm volatile("" : "+v"(row));
#pragma unroll
      for (int k = 0; k < kFull; ++k) m.q[k] = *(const Acc*)(p + k * kRows * 64 + 16 * row);
      m.q[kFull] = half_fragment(p + kFull * kRows * 64 + 8 * row);
      return;
    }
#pragma unroll
    for (int k = 0; k < kFull; ++k) {
      const int o = t * kTileBytes + k * 1024;
      m.q[k] = *(const Acc*)(lds + at[o / kWindow] + o % kWindow);
    }
    const int o = t * kTileBytes + kFull * 1024;
    m.q[kFull] = half_fragment(lds + at_half[o / kWindow] + o % kWindow);
  }
  static __device__ __forceinline__ Sums sums(const Frags& m, const Op& d, int s, const Acc& from) {
    Sums v;
#pragma unroll
    for (int x = 0; x < kHalves; ++x) v.r[x] = from;
#pragma unroll
    for (int k = 0; k <= kFull; ++k)
#pragma unroll
      for (int x = 0; x < kHalves; ++x)
        v.r[x] = __builtin_amdgcn_mfma_i32_16x16x64_i8(m.q[k], d.get(s, x, k), v.r[x], 0, 0, 0);
    return v;
  }
  // The order that one set's products of a tile are issued in: a matrix instruction keeps its unit busy for 16 cycles and
  // the issue slot for 8; the vector unit's work on the set before goes between, as do the next fragments' reads.
  template <int VALU, bool READ>
  static __device__ __forceinline__ void interleave() {
#pragma unroll
    for (int k = 0; k <= kFull; ++k)
#pragma unroll
      for (int x = 0; x < kHalves; ++x) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        if (READ && x == kHalves - 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x2, VALU, 0);
      }
    __builtin_amdgcn_sched_barrier(0);
  }

  // the residue products of register i with v0, v1: of base A (sigma) or base B (z, w)
  static __device__ __forceinline__ void product(u32& r0, u32& r1, u32 u0, u32 u1, u32 v0, u32 v1, u32 p, u32 pinv, u32 e) {
    r0 = reduce(smad(u0, v0, 0), p, pinv);
    if constexpr (PAIR) r1 = reduce(smad(r0, e, smad(u0, v1, smad(u1, v0, 0))), p, pinv);
  }
  static __device__ __forceinline__ void square(u32& r0, u32& r1, u32 u0, u32 u1, u32 p, u32 pinv, u32 e) {
    r0 = reduce(smad(u0, u0, 0), p, pinv);
    if constexpr (PAIR) r1 = reduce(smad(r0, e, twice(u0, u1)), p, pinv);
  }
  // sigma, as bytes, of the square of base A's residues
  __device__ __forceinline__ void square_a(Res& a) {
    use_matrix<0>();
#pragma unroll
    for (int i = 0; i < kTiles; ++i) {
      if (i % 4 == 0) __builtin_amdgcn_sched_barrier(0);
      const Quad k = cst(0, i);
#pragma unroll
      for (int s = 0; s < kSets; ++s) {
        u32 r0, r1 = 0;
        square(r0, r1, a.get(s, 0, i), PAIR ? a.get(s, 1, i) : 0u, k[0], k[1], k[2]);
        a.set(s, 0, i, r0 ^ rns::kOmega);
        if constexpr (PAIR) a.set(s, 1, i, r1 ^ rns::kOmega);
      }
      if (i % 4 == 3 || i == kTiles - 1) a.gather(i / 4);
    }
  }
  // Sigma, and z and w, of the product with a table entry, which comes from memory: the next kAhead quads of four
  // registers are on their way.
  struct EntryQuad {
    Quad q[kSets][kHalves];
  };
  static constexpr int kAhead = kSets == 1 ? 1 : 3;
  __device__ __forceinline__ EntryQuad load_quad(const u32* entry, int j) const {
    const int base = j / (kFull + 1), k = j % (kFull + 1);
    const Quad* p = (const Quad*)(entry + base * kArray) + lane;
    EntryQuad r;
#pragma unroll
    for (int s = 0; s < kSets; ++s) {
      if (k == kFull) {
        const Quad h = p[(kSets * kHalves * kFull + s) * WAVE];
        r.q[s][0] = h;
        r.q[s][kHalves - 1] = PAIR ? Quad{h[2], h[3], 0, 0} : h;
      } else {
#pragma unroll
        for (int x = 0; x < kHalves; ++x) r.q[s][x] = p[((kSets * k + s) * kHalves + x) * WAVE];
      }
    }
    return r;
  }
  __device__ __forceinline__ void multiply_residues(State& x, const u32* entry) {
    use_matrix<0>();
    constexpr int kSteps = 2 * (kFull + 1);
    EntryQuad y[kAhead];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) y[j] = load_quad(entry, j);
#pragma unroll
    for (int j = 0; j < kSteps; ++j) {
      const int base = j / (kFull + 1), k4 = j % (kFull + 1);
      Res& d = base ? x.b : x.a;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 4 * k4; i < 4 * k4 + 4 && i < kTiles; ++i) {
        const Quad k = cst(base, i);
#pragma unroll
        for (int s = 0; s < kSets; ++s) {
          const u32 flip = base ? rns::kOmega : 0u;
          u32 r0, r1 = 0;
          product(r0, r1, d.get(s, 0, i) ^ flip, PAIR ? d.get(s, 1, i) ^ flip : 0u, y[j % kAhead].q[s][0][i % 4],
                  PAIR ? y[j % kAhead].q[s][kHalves - 1][i % 4] : 0u, k[0], k[1], k[2]);
          d.set(s, 0, i, base ? r0 : r0 ^ rns::kOmega);
          if constexpr (PAIR) d.set(s, 1, i, base ? r1 : r1 ^ rns::kOmega);
        }
      }
      d.gather(k4);
      __builtin_amdgcn_sched_barrier(0);
      if (j + kAhead < kSteps) y[j % kAhead] = load_quad(entry, j + kAhead);
    }
  }

  // the constant 1 of the bias in its slot, and nothing in alpha's yet
  __device__ __forceinline__ void set_extra(Res& d) const {
    const bool alpha = g == rns::alpha_group(NR), bias = g == rns::bias_group(NR);
#pragma unroll
    for (int s = 0; s < kSets; ++s)
#pragma unroll
      for (int x = 0; x < kHalves; ++x) d.h[s][2 * x + 1] = alpha ? 0u : bias ? 1u : d.h[s][2 * x + 1];
  }
  // Base B of a register's reduced value, as bytes, from a tile's sums and z, w
  static __device__ __forceinline__ void finish_b(Res& b, int i, int s, const Sums& v, const Quad& k) {
    const u32 t0 = reduce(smad(b.get(s, 0, i), k[2], column(v.r[0])), k[0], k[1]);
    b.set(s, 0, i, t0 ^ rns::kOmega);
    if constexpr (PAIR) {
      s64 col = smad(b.get(s, 1, i), k[2], column(v.r[1]));
      asm("" : "+v"(col));  // multiply-adds one after the other
      b.set(s, 1, i, reduce(smad(t0, k[3], col), k[0], k[1]) ^ rns::kOmega);
    }
    if (s == kSets - 1 && (i % 4 == 3 || i == kTiles - 1)) b.gather(i / 4);
  }
  // z and w of the square of a register, in place of its bytes
  static __device__ __forceinline__ void square_b(Res& b, int i, int s, const Quad& k) {
    u32 r0, r1 = 0;
    square(r0, r1, b.get(s, 0, i) ^ rns::kOmega, PAIR ? b.get(s, 1, i) ^ rns::kOmega : 0u, k[0], k[1], 0u - k[3]);
    b.set(s, 0, i, r0);
    if constexpr (PAIR) b.set(s, 1, i, r1);
  }
  // Base B of the reduced pair, as bytes, from sigma in base A; SQ: of a square, whose z and w are made on the way from
  // base B's bytes, else from those.
  template <bool SQ>
  __device__ __forceinline__ void extend_to_b(State& x) {
    use_matrix<0>();
    set_extra(x.a);
    Op d(x.a);
    Frags m;
    Sums v0, v1;
    Quad k = {}, k_before = {}, k_next = cst(2, 0);
    fragments<0>(m, 0);
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      __builtin_amdgcn_sched_barrier(0);
      k = k_next;
      v0 = sums(m, d, 0, start);
      if (kSets == 1 && t + 1 < kTiles) {
        fragments<0>(m, t + 1);
        k_next = cst(2, t + 1);
      }
      if (t > 0) finish_b(x.b, t - 1, kSets - 1, v1, k_before);
      if (SQ) square_b(x.b, t, 0, k);
      interleave<2, kSets == 1>();
      if constexpr (kSets == 2) {
        v1 = sums(m, d, 1, start);
        if (t + 1 < kTiles) {
          fragments<0>(m, t + 1);
          k_next = cst(2, t + 1);
        }
        finish_b(x.b, t, 0, v0, k);
        if (SQ) square_b(x.b, t, 1, k);
        interleave<2, true>();
      } else {
        v1 = v0;
      }
      k_before = k;
    }
    finish_b(x.b, kTiles - 1, kSets - 1, v1, k_before);
    set_extra(x.b);
  }

  // base A of a register from a tile's sums; NEXT: and sigma of its square, as bytes
  template <bool NEXT>
  static __device__ __forceinline__ void finish_a(Res& a, int i, int s, const Sums& v, const Quad& k) {
    u32 u0 = reduce(column(v.r[0]), k[0], k[1]), u1 = 0;
    if constexpr (PAIR) u1 = reduce(column(v.r[kHalves - 1]), k[0], k[1]);
    if (NEXT) {
      u32 r0, r1 = 0;
      square(r0, r1, u0, u1, k[0], k[1], k[2]);
      u0 = r0 ^ rns::kOmega;
      u1 = r1 ^ rns::kOmega;
    }
    a.set(s, 0, i, u0);
    if constexpr (PAIR) a.set(s, 1, i, u1);
    if (s == kSets - 1 && i % 4 == 3) a.gather(i / 4);
  }
  // base A from base B's bytes, NEXT: as sigma of the square; alpha stays in its slot of base B
  template <bool NEXT>
  __device__ __forceinline__ void extend_to_a(State& x) {
    use_matrix<1>();
    Op d(x.b);
    Frags m;
    fragments<1>(m, kTiles - 1);
    Quad k_before = cst(0, kTiles - 1), k_next = cst(0, 0);
    // the tile that has alpha's row: its own primes take alpha afterwards
    Sums v0 = sums(m, d, 0, start), v1;
    if constexpr (kSets == 2) v1 = sums(m, d, 1, start);
    const Acc half = m.q[kFull];
    fragments<1>(m, 0);
#pragma unroll
    for (int s = 0; s < kSets; ++s)
#pragma unroll
      for (int i = 0; i < kHalves; ++i) {
        Acc& r = s == 1 ? v1.r[i] : v0.r[i];
        const u32 a = g == rns::alpha_group(NR) ? alpha_bytes((u32)column(r) + rns::alpha_round(NR)) : 0u;
        const Quad only = {0, a, 0, 0};
        r = __builtin_amdgcn_mfma_i32_16x16x64_i8(half, (Acc)only, r, 0, 0, 0);
        d.o[s][i][1] |= a;
      }
    if constexpr (kSets == 2) finish_a<NEXT>(x.a, kTiles - 1, 0, v0, k_before);
    else v1 = v0;
#pragma unroll
    for (int t = 0; t < kTiles - 1; ++t) {
      __builtin_amdgcn_sched_barrier(0);
      const Quad k = k_next;
      v0 = sums(m, d, 0, start);
      if (kSets == 1 && t + 2 < kTiles) {
        fragments<1>(m, t + 1);
        k_next = cst(0, t + 1);
      }
      finish_a<NEXT>(x.a, t == 0 ? kTiles - 1 : t - 1, kSets - 1, v1, k_before);
      interleave<2, kSets == 1>();
      if constexpr (kSets == 2) {
        v1 = sums(m, d, 1, start);
        if (t + 2 < kTiles) {
          fragments<1>(m, t + 1);
          k_next = cst(0, t + 1);
        }
        finish_a<NEXT>(x.a, t, 0, v0, k);
        interleave<2, true>();
      } else {
        v1 = v0;
      }
      k_before = k;
    }
    finish_a<NEXT>(x.a, kTiles - 2, kSets - 1, v1, k_before);
    if ((kTiles - 2) / 4 < kFull) x.a.gather((kTiles - 2) / 4);
    x.a.gather(kFull);
    d.release();
  }

  // one tile of a matrix in global memory, with all rows
  __device__ __forceinline__ Frags global_fragments(const char* matrix, int t) const {
    Frags m;
    const char* p = matrix + t * kTileBytes;
#pragma unroll
    for (int k = 0; k < kFull; ++k) m.q[k] = *(const Acc*)(p + k * 1024 + lane * 16);
    m.q[kFull] = half_fragment(p + kFull * 1024 + lane * 8);
    return m;
  }
  // the pairs whose limbs are at `src` (`left` of them, then zeros) into both bases
  __device__ __forceinline__ void load(State& x, const u32* src, unsigned left, int nl, const char* matrix) {
    x = State();
#pragma unroll
    for (int s = 0; s < kSets; ++s) {
      const bool active = (unsigned)((lane & 15) + 16 * s) < left;
      const u32* p = src + ((lane & 15) + 16 * s) * 2 * nl;
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const int l = 4 * i + g;
        const bool ok = active && l < nl;
        x.a.set(s, 0, i, (ok ? p[l] : 0u) ^ rns::kOmega);
        if constexpr (PAIR) x.a.set(s, 1, i, (ok ? p[nl + l] : 0u) ^ rns::kOmega);
      }
    }
    if (g == rns::bias_group(NR)) {  // in place of a limb that is zero
#pragma unroll
      for (int s = 0; s < kSets; ++s)
#pragma unroll
        for (int i = 0; i < kHalves; ++i) x.a.set(s, i, NR - 1, 1);
    }
    use_matrix<0>();
    Op d(x.a);
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      __builtin_amdgcn_sched_barrier(0);
      const Frags m = global_fragments(matrix, t);
      const Quad k = cst(1, t);
#pragma unroll
      for (int s = 0; s < kSets; ++s) {
        const Sums v = sums(m, d, s, start);
#pragma unroll
        for (int i = 0; i < kHalves; ++i) x.b.set(s, i, t, reduce(column(v.r[i]), k[0], k[1]) ^ rns::kOmega);
      }
      if (t % 4 == 3 || t == kTiles - 1) x.b.gather(t / 4);
    }
    set_extra(x.b);
    extend_to_a<false>(x);
  }
  // the pairs as two integers each in columns of weight 2^(29 l), from base B
  __device__ __forceinline__ void store(State& x, long long* dst, unsigned left, const char* matrix) {
    Op d(x.b);
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      __builtin_amdgcn_sched_barrier(0);
      const Frags m = global_fragments(matrix, t);
#pragma unroll
      for (int s = 0; s < kSets; ++s) {
        const Sums v = sums(m, d, s, Acc{0, 0, 0, 0});
        const unsigned e = (unsigned)((lane & 15) + 16 * s);
        if (e < left) {
          long long* p = dst + e * (8 * kTiles) + 4 * t + g;
          p[0] = integer(v.r[0]);
          p[4 * kTiles] = PAIR ? integer(v.r[kHalves - 1]) : 0;
        }
      }
    }
  }

  // Window tables: an entry holds the residues of base A and of base B one after the other, each as
  // [quad][set][x0, x1][lane], the last quad for both halves.
  static constexpr int kArray = kSets * (kHalves * kFull + 1) * 4 * WAVE;  // dwords
  // quads `from` to `to` of one base
  __device__ __forceinline__ void load_entry(Res& d, const u32* entry, int base, int from, int to) const {
    const Quad* p = (const Quad*)(entry + base * kArray) + lane;
#pragma unroll
    for (int k = from; k < to; ++k)
#pragma unroll
      for (int s = 0; s < kSets; ++s) {
        if (k == kFull) {
          d.h[s] = p[(kSets * kHalves * kFull + s) * WAVE];
          continue;
        }
#pragma unroll
        for (int x = 0; x < kHalves; ++x) d.q[s][x][k < kFull ? k : 0] = p[((kSets * k + s) * kHalves + x) * WAVE];
      }
  }
  __device__ __forceinline__ void store_entry(const Res& d, u32* entry, int base, u32 flip) const {
    Quad* p = (Quad*)(entry + base * kArray) + lane;
#pragma unroll
    for (int s = 0; s < kSets; ++s) {
#pragma unroll
      for (int k = 0; k < kFull; ++k)
#pragma unroll
        for (int x = 0; x < kHalves; ++x) p[((kSets * k + s) * kHalves + x) * WAVE] = d.q[s][x][k] ^ flip;
      p[(kSets * kHalves * kFull + s) * WAVE] = d.h[s] ^ flip;
    }
  }
  __device__ __forceinline__ void load_state(State& x, const u32* entry) const {
    load_entry(x.a, entry, 0, 0, kFull + 1);
    load_entry(x.b, entry, 1, 0, kFull + 1);
#pragma unroll
    for (int s = 0; s < kSets; ++s) {
#pragma unroll
      for (int k = 0; k < kFull; ++k)
#pragma unroll
        for (int i = 0; i < kHalves; ++i) x.b.q[s][i][k] ^= rns::kOmega;
      x.b.h[s] ^= rns::kOmega;
    }
  }
  __device__ __forceinline__ void store_state(const State& x, u32* entry) const {
    store_entry(x.a, entry, 0, 0u);
    store_entry(x.b, entry, 1, rns::kOmega);
  }
};

// Wavefronts per SIMD: two with 256 registers each for two sets, three with 168 for one. Measured against wavefronts of one
// set, four to a SIMD, whose phases did not overlap within a wavefront and which spent 54 instructions per prime: 65536
// encryptions at a 1024-bit key 9.8 -> 8.4 ms, 32768 decryptions at a 2048-bit key 10.0 -> 8.7, 8192 of them 3.47 -> 2.58,
// 20001 key-owner encryptions 11.2 -> 9.8. Per squaring of 32 elements at 1024 bits: 790 vector and 218 matrix instructions,
// 7.0 k cycles for a SIMD's only wavefront and 9 - 10 k for two together. The clock gives way under it (2.0 GHz with one
// wavefront per SIMD, 1.5 - 1.65 with two, and up to 6 % apart between the dies): more instructions in flight no longer help.
// What spills (99 registers in the pair form of 1024 bits) does so outside the run of squarings.
constexpr int rns_waves_per_simd(int sets) { return sets == 1 ? 3 : 2; }
// Every wavefront runs the program on its sets at a time. The first `split` blocks run j0, the others j1.
template <int NR, bool PAIR, int kSets>
__global__ __launch_bounds__(rns_waves_per_simd(kSets) * 256, rns_waves_per_simd(kSets)) void k_rns(RnsJob j0, RnsJob j1, unsigned split, size_t count) {
  constexpr int kElements = 16 * kSets;
  __shared__ __align__(16) u32 lds[rns::lds_bytes(NR) / 4];
  const bool second = blockIdx.x >= split;
  const RnsJob& j = second ? j1 : j0;
  const unsigned block = second ? blockIdx.x - split : blockIdx.x;
  const unsigned nblocks = second ? gridDim.x - split : split;
  for (int i = (int)threadIdx.x; i < rns::lds_bytes(NR) / 16; i += (int)blockDim.x)
    ((Quad*)lds)[i] = ((const Quad*)j.tables)[i];
  __syncthreads();
  const char* in_matrix = (const char*)j.tables + rns::lds_bytes(NR);
  const char* out_matrix = in_matrix + rns::in_matrix_bytes(NR);
  RnsEngine<NR, PAIR, kSets> e(lds);
  const unsigned waves = blockDim.x / 64;
  // the same for the whole wavefront, so that what follows from it stays in scalar registers
  const size_t wave = (size_t)block * waves + (unsigned)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
  constexpr size_t kEntry = 2 * RnsEngine<NR, PAIR, kSets>::kArray;
  const u32* prog = j.prog ? j.prog : j.ins;
  const int len = __builtin_amdgcn_readfirstlane(j.len);
  u32* table = j.slots + wave * (size_t)j.entries * kEntry;
  for (size_t tile = wave; tile * kElements < count; tile += (size_t)nblocks * waves) {
    const unsigned left = (unsigned)std::min(count - tile * kElements, (size_t)kElements);
    RnsState<NR, PAIR, kSets> x;
    e.load(x, j.in + tile * (size_t)(kElements * 2 * j.nl), left, j.nl, in_matrix);
    for (int pc = 0; pc < len;) {
      const u32 ins = (u32)__builtin_amdgcn_readfirstlane((int)prog[pc++]);
      const u32 op = ins & 0xFFu, a = (ins >> 8) & 0xFFFu, b = ins >> 20;
      u32* entry = table + (size_t)a * kEntry;
      if (op == ENG_STORE_T) {
        e.store_state(x, entry);
        continue;
      }
      if (op == ENG_LOAD_T) {
        e.load_state(x, entry);
        continue;
      }
      if (op == ENG_SQ) {  // a run of them, nine tenths of a program, each but the last with the next one's sigma
        e.square_a(x.a);
        e.template extend_to_b<true>(x);
#pragma unroll 1
        while (pc < len && (u32)__builtin_amdgcn_readfirstlane((int)prog[pc]) == ENG_SQ) {
          ++pc;

          e.template extend_to_a<true>(x);
          e.template extend_to_b<true>(x);
        }
      } else {
        e.multiply_residues(x, entry);
        e.template extend_to_b<false>(x);
      }
      e.template extend_to_a<false>(x);
      if (op == ENG_MUL_T_ST) e.store_state(x, table + (size_t)b * kEntry);
    }
    e.store(x, j.out + tile * (size_t)(kElements * 8 * rns::tiles(NR)), left, out_matrix);
  }
}

// The same for pairs of 2048-bit halves: 16 elements per wavefront and four wavefronts per SIMD, whose 128 registers hold
// the 72 of an element set's state, and each phase of a product after the other, without the next one's work in between.
// 65536 encryptions at a 2048-bit key take 48.5 ms with it (49.2 with the residues of before, kept below 2^31 by 54
// instructions per prime instead of 47), 52.4 with k_rns's two sets of which every wavefront's 256 registers are full:
// tables and spilled registers then wait for memory, two wavefronts per SIMD are too few to hide it. k_rns's one set with three
// wavefronts of 168 registers, which lies between, spills 348 of them: 49152 elements 39.4 ms against 37.8. This kernel with three
// wavefronts of 154, without a spill, takes 36.8 for those, but for 65536, 1.33 passes then, 64.8.
// The residues of x0 and x1 of a lane in one base: full quads of each, and one quad with the last two of both.
template <int NR>
struct OneResidues {
  static_assert(NR % 4 == 2, "full blocks and a half one");
  static constexpr int kFull = NR / 4;
  Quad q[2][kFull];
  Quad h;
  template <int X>
  __device__ __forceinline__ u32 get(int i) const {
    return i < 4 * kFull ? q[X][i / 4][i % 4] : h[2 * X + i % 4];
  }
  template <int X>
  __device__ __forceinline__ void set(int i, u32 v) {
    if (i < 4 * kFull) q[X][i / 4][i % 4] = v;
    else h[2 * X + i % 4] = v;
  }
  // Gathers quad k of both halves in its registers now: left alone, the compiler keeps the values in the 64-bit results
  // they are the upper words of until all are there.
  __device__ __forceinline__ void gather(int k) {
    if (k < kFull) {
      asm("" : "+v"(q[0][k]));
      asm("" : "+v"(q[1][k]));
    } else {
      asm("" : "+v"(h));
    }
  }
  // Hides where the values come from: the compiler would widen what is multiplied later to 64 bits where it is made
  // and carry the zero upper words along.
  __device__ __forceinline__ void forget() {
#pragma unroll
    for (int k = 0; k <= kFull; ++k) gather(k);
  }
};
template <int NR>
struct OneState {
  OneResidues<NR> a, b;
};

// A residue as the bytes the matrix products take (each 128 less), and back. Hidden from the compiler, which would
// otherwise keep the residue beside its bytes instead of taking it back from them.
__device__ __forceinline__ u32 to_bytes(u32 v) {
  v ^= rns::kOmega;
  asm("" : "+v"(v));
  return v;
}

// Where this lane's part of a fragment lies in a tile of 16 (kept) rows: of a full one, and of the half one
struct OneFragmentAt {
  int full, half;  // bytes
  __device__ __forceinline__ OneFragmentAt(int lane, int rows) {
    full = ((lane >> 4) * rows + (lane & (rows - 1))) * 16;
    half = full / 2;
  }
  // read again for each product: held in registers, the matrix would not fit them
  __device__ __forceinline__ void forget() { asm volatile("" : "+v"(full), "+v"(half)); }
};

// The operand of a matrix product: the half block's words of x0 and of x1 in a quad of their own, zeros behind them.
template <int NR>
struct OneOperand {
  OneResidues<NR>& d;
  Quad h0, h1;
  __device__ __forceinline__ explicit OneOperand(OneResidues<NR>& d_)
      : d(d_), h0(Quad{d_.h[0], d_.h[1], 0, 0}), h1(Quad{d_.h[2], d_.h[3], 0, 0}) {
    asm("" : "+v"(h0));  // made once, not for every tile
    asm("" : "+v"(h1));
  }
  // back to the residues' own form
  __device__ __forceinline__ void release() { d.h = Quad{h0[0], h0[1], h1[0], h1[1]}; }
};

// One tile (4 destination slots, one per lane) of a matrix times both halves of a pair. Of the half block only 8 bytes
// of a row are stored: what lies in the other registers meets the operand's zeros. (A version with
// v_mfma_i32_16x16x32_i8 for the half block, accumulated onto the 16x16x64 products, gave wrong sums. Why is not
// understood: neither a wrong idea of its operands' layout nor a missing wait was excluded.)
template <int NR>
__device__ __forceinline__ void tile_products(Acc& r0, Acc& r1, const void* tile, int rows, const OneFragmentAt& at,
                                              const OneOperand<NR>& d, const Acc& start, Acc* half = nullptr) {
  constexpr int F = rns::full_blocks(NR);
  const char* p = (const char*)tile;
  Acc m[F + 1];
#pragma unroll
  for (int k = 0; k < F; ++k) m[k] = *(const Acc*)(p + k * rows * 64 + at.full);
  const Twin h = *(const Twin*)(p + F * rows * 64 + at.half);
  int any0 = 0, any1 = 0;
#if defined(__HIP_DEVICE_COMPILE__)
  asm("" : "=v"(any0), "=v"(any1));
#endif
  m[F] = Acc{(int)h[0], (int)h[1], any0, any1};
  if (half) *half = m[F];
  r0 = r1 = start;
#pragma unroll
  for (int k = 0; k <= F; ++k) {
    r0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(m[k], (Acc)(k < F ? d.d.q[0][k < F ? k : 0] : d.h0), r0, 0, 0, 0);
    r1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(m[k], (Acc)(k < F ? d.d.q[1][k < F ? k : 0] : d.h1), r1, 0, 0, 0);
  }
}

template <int NR>
struct OneEngine {
  static constexpr int kTiles = rns::tiles(NR);  // also the registers that hold primes
  static constexpr int kGroup = 3;               // tiles the compiler may mix
  static constexpr int kTileBytes = rns::tile_bytes(NR, 16);
  const char* lds;
  int lane, g;
  Acc start;
  OneFragmentAt at, at_last0, at_last1;  // of a tile, and of the last one of either matrix
  int cst_at;                         // of this lane group's constants in a row of four slots
  u32 keep, mine, one;                // masks of set_extra and set_alpha

  __device__ __forceinline__ OneEngine(const void* lds_)
      : lds((const char*)lds_), lane((int)(threadIdx.x & (WAVE - 1))), g(lane >> 4), start(start_sums()), at(lane, 16),
        at_last0(lane, rns::last_rows(NR, 0)), at_last1(lane, rns::last_rows(NR, 1)), cst_at(16 * g),
        keep(g == rns::alpha_group(NR) || g == rns::bias_group(NR) ? 0u : ~0u), mine(g == rns::alpha_group(NR) ? ~0u : 0u),
        one(g == rns::bias_group(NR) ? 1u : 0u) {
    asm volatile("" : "+v"(keep), "+v"(mine), "+v"(one));  // no branches
  }
  // Everything a wavefront reads from LDS is constant over the launch: without these the compiler would read it once
  // and not have the registers for it. They also bound what it may mix.
  __device__ __forceinline__ void forget() {
    __builtin_amdgcn_sched_barrier(0);
    at.forget();
    if (rns::last_rows(NR, 0) != 16) {
      at_last0.forget();
      at_last1.forget();
    }
    asm volatile("" : "+v"(cst_at));
  }
  // of base A (0), base B's products (1) and its sums (2)
  __device__ __forceinline__ Quad cst(int base, int i) const {
    return *(const Quad*)(lds + rns::lds_matrices_bytes(NR) + (base * rns::slots(NR) + 4 * i) * 16 + cst_at);
  }
  template <int MATRIX>
  __device__ __forceinline__ void lds_products(Acc& r0, Acc& r1, int t, const OneOperand<NR>& d, Acc* half = nullptr) const {
    constexpr int kLast = rns::last_rows(NR, MATRIX);
    const char* p = lds + MATRIX * rns::lds_matrix_bytes(NR, 0) + t * kTileBytes;
    if (t == kTiles - 1) tile_products<NR>(r0, r1, p, kLast, kLast == 16 ? at : MATRIX ? at_last1 : at_last0, d, start, half);
    else tile_products<NR>(r0, r1, p, 16, at, d, start);
  }

  // The residue products of one base of a square (y null) or of a product with the table entry y: bytes of sigma in
  // base A (BASE 0), z and w in base B. The entry's quads are on their way one step ahead.
  template <int BASE, bool SQ, int STEP>
  __device__ __forceinline__ void base_products(OneResidues<NR>& x, const u32* y) {
    constexpr int kQuads = NR / 4 + 1;
    const Quad* p = quads<STEP>(y, BASE);
    x.forget();
    Quad n0 = {}, n1 = {};
    if (!SQ) {
      n0 = p[0];
      n1 = p[STEP];
    }
#pragma unroll
    for (int q = 0; q < kQuads; ++q) {
      const Quad y0 = n0, y1 = n1;
      forget();
      if (!SQ && q + 1 < kQuads) {
        n0 = p[2 * (q + 1) * STEP];
        if (q + 2 < kQuads) n1 = p[(2 * (q + 1) + 1) * STEP];
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int i = 4 * q + c;
        if (i >= kTiles || i >= NR) continue;
        const Quad k = cst(BASE, i);
        const u32 u0 = x.template get<0>(i), v0 = SQ ? u0 : y0[c];
        const u32 s0 = reduce(smad(u0, v0, 0), k[0], k[1]);
        x.template set<0>(i, BASE ? s0 : to_bytes(s0));
        {
          const u32 u1 = x.template get<1>(i), v1 = SQ ? u1 : (q + 1 < kQuads ? y1[c] : y0[(2 + c) % 4]);
          const s64 cross = SQ ? twice(u0, u1) : smad(u0, v1, smad(u1, v0, 0));
          const u32 s1 = reduce(smad(s0, k[2], cross), k[0], k[1]);
          x.template set<1>(i, BASE ? s1 : to_bytes(s1));
        }
      }
      x.gather(q);
    }
  }
  template <bool SQ, int STEP>
  __device__ __forceinline__ void products(OneState<NR>& x, const u32* y) {
    base_products<0, SQ, STEP>(x.a, y);
    base_products<1, SQ, STEP>(x.b, y);
  }

  // the constant 1 of the bias in its slot, and nothing in alpha's yet
  __device__ __forceinline__ void set_extra(OneResidues<NR>& d) const {
    d.h[1] = (d.h[1] & keep) | one;
    d.h[3] = (d.h[3] & keep) | one;
  }

  // Base B of the reduced pair from sigma (bytes, in base A) and the products z, w (in base B); leaves base B as bytes
  // for the way back.
  __device__ __forceinline__ void extend_to_b(OneState<NR>& x) {
    x.b.forget();
    set_extra(x.a);
    OneOperand<NR> d(x.a);
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      if (t % kGroup == 0) forget();
      Acc r0, r1;
      lds_products<0>(r0, r1, t, d);
      const Quad k = cst(2, t);
      const u32 t0 = reduce(smad(x.b.template get<0>(t), k[2], column(r0)), k[0], k[1]);
      {
        const s64 col = smad(x.b.template get<1>(t), k[2], column(r1));
        x.b.template set<1>(t, to_bytes(reduce(smad(t0, k[3], col), k[0], k[1])));
      }
      x.b.template set<0>(t, to_bytes(t0));
      if (t % 4 == 3) x.b.gather(t / 4);
    }
    set_extra(x.b);
  }
  // base A from base B's bytes; turns base B back to residues, with alpha in its slot
  __device__ __forceinline__ void extend_to_a(OneState<NR>& x) {
    OneOperand<NR> d(x.b);
#pragma unroll
    for (int i = 0; i < kTiles; ++i) {
      const int t = i == 0 ? kTiles - 1 : i - 1;
      if (i % kGroup == 0) forget();
      Acc r0, r1;
      if (i == 0) {  // the tile that has alpha's row: its own primes take alpha afterwards
        Acc half;
        lds_products<1>(r0, r1, t, d, &half);
        const Quad a0 = {0, alpha_bytes((u32)column(r0) + rns::alpha_round(NR)) & mine, 0, 0};
        r0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(half, (Acc)a0, r0, 0, 0, 0);
        d.h0[1] |= a0[1];
        {
          const Quad a1 = {0, alpha_bytes((u32)column(r1) + rns::alpha_round(NR)) & mine, 0, 0};
          r1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(half, (Acc)a1, r1, 0, 0, 0);
          d.h1[1] |= a1[1];
        }
      } else {
        lds_products<1>(r0, r1, t, d);
      }
      const Quad k = cst(0, t);
      x.a.template set<0>(t, reduce(column(r0), k[0], k[1]));
      x.a.template set<1>(t, reduce(column(r1), k[0], k[1]));
      if (t % 4 == 3) x.a.gather(t / 4);
    }
    d.release();
    flip(x.b);
  }
  // residues <-> bytes
  static __device__ __forceinline__ void flip(OneResidues<NR>& d) {
#pragma unroll
    for (int k = 0; k < NR / 4; ++k) {
      d.q[0][k] ^= rns::kOmega;
      d.q[1][k] ^= rns::kOmega;
    }
    d.h ^= rns::kOmega;
  }

  // the pairs whose limbs are at `src` (`left` of them, then zeros) into both bases
  __device__ __forceinline__ void load(OneState<NR>& x, const u32* src, unsigned left, int nl, const char* matrix) {
    const bool active = (unsigned)(lane & 15) < left;
    src += (lane & 15) * 2 * nl;
    x = OneState<NR>();
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int l = 4 * i + g;
      const bool ok = active && l < nl;
      x.a.template set<0>(i, (ok ? src[l] : 0u) ^ rns::kOmega);
      x.a.template set<1>(i, (ok ? src[nl + l] : 0u) ^ rns::kOmega);
    }
    if (one) {  // in place of a limb that is zero
      x.a.template set<0>(NR - 1, 1);
      x.a.template set<1>(NR - 1, 1);
    }
    OneOperand<NR> d(x.a);
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      forget();
      Acc r0, r1;
      tile_products<NR>(r0, r1, matrix + t * kTileBytes, 16, at, d, start);
      const Quad k = cst(1, t);
      x.b.template set<0>(t, to_bytes(reduce(column(r0), k[0], k[1])));
      x.b.template set<1>(t, to_bytes(reduce(column(r1), k[0], k[1])));
    }
    set_extra(x.b);
    extend_to_a(x);
  }
  // The pairs as two integers each in columns of weight 2^(29 l), this lane's to element `own` behind `dst`. Base B still
  // holds what the way back left there, alpha and the bias among it.
  __device__ __forceinline__ void store(OneState<NR>& x, long long* dst, unsigned own, bool active, const char* matrix) {
    dst += own * (8 * kTiles);
    flip(x.b);
    OneOperand<NR> d(x.b);
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      forget();
      Acc r0, r1;
      tile_products<NR>(r0, r1, matrix + t * kTileBytes, 16, at, d, Acc{0, 0, 0, 0});
      if (active) {
        dst[4 * t + g] = integer(r0);
        dst[4 * kTiles + 4 * t + g] = integer(r1);
      }
    }
  }

  // In memory the registers of base A and of base B lie one after the other, a lane's quads STEP apart: WAVE in a window
  // table's entry of 16 elements, where a lane's first is quad `lane`, and 4 in an element by itself (quad `g`), whose
  // place each lane knows.
  template <int STEP>
  static constexpr int kArray = (2 * (NR / 4) + 1) * 4 * STEP;  // dwords of one base
  template <int STEP>
  __device__ __forceinline__ const Quad* quads(const u32* y, int base) const {
    return (const Quad*)(y + base * kArray<STEP>) + (STEP == WAVE ? lane : g);
  }
  template <int STEP>
  __device__ __forceinline__ void load_array(OneResidues<NR>& d, const u32* y, int base) const {
    const Quad* p = quads<STEP>(y, base);
#pragma unroll
    for (int k = 0; k < NR / 4; ++k) {
      d.q[0][k] = p[2 * k * STEP];
      d.q[1][k] = p[(2 * k + 1) * STEP];
    }
    d.h = p[2 * (NR / 4) * STEP];
  }
  template <int STEP>
  __device__ __forceinline__ void store_array(const OneResidues<NR>& d, u32* y, int base) const {
    Quad* p = (Quad*)quads<STEP>(y, base);
#pragma unroll
    for (int k = 0; k < NR / 4; ++k) {
      p[2 * k * STEP] = d.q[0][k];
      p[(2 * k + 1) * STEP] = d.q[1][k];
    }
    p[2 * (NR / 4) * STEP] = d.h;
  }
  template <int STEP>
  __device__ __forceinline__ void load_state(OneState<NR>& x, const u32* y) const {
    load_array<STEP>(x.a, y, 0);
    load_array<STEP>(x.b, y, 1);
  }
  template <int STEP>
  __device__ __forceinline__ void store_state(const OneState<NR>& x, u32* y) const {
    store_array<STEP>(x.a, y, 0);
    store_array<STEP>(x.b, y, 1);
  }
};

// Every wavefront runs the program on 16 elements at a time. The first `split` blocks run j0, the others j1.
template <int NR>
__global__ __launch_bounds__(1024, 4) void k_rns_one(RnsJob j0, RnsJob j1, unsigned split, size_t count) {
  __shared__ __align__(16) u32 lds[rns::lds_bytes(NR) / 4];
  const bool second = blockIdx.x >= split;
  const RnsJob& j = second ? j1 : j0;
  const unsigned block = second ? blockIdx.x - split : blockIdx.x;
  const unsigned nblocks = second ? gridDim.x - split : split;
  for (int i = (int)threadIdx.x; i < rns::lds_bytes(NR) / 16; i += (int)blockDim.x)
    ((Quad*)lds)[i] = ((const Quad*)j.tables)[i];
  __syncthreads();
  const char* in_matrix = (const char*)j.tables + rns::lds_bytes(NR);
  const char* out_matrix = in_matrix + rns::in_matrix_bytes(NR);
  OneEngine<NR> e(lds);
  const unsigned waves = blockDim.x / 64;
  // the same for the whole wavefront, so that what follows from it stays in scalar registers
  const size_t wave = (size_t)block * waves + (unsigned)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
  constexpr size_t kEntry = 2 * OneEngine<NR>::template kArray<WAVE>;
  const u32* prog = j.prog ? j.prog : j.ins;
  const int len = __builtin_amdgcn_readfirstlane(j.len);
  u32* table = j.slots + wave * (size_t)j.entries * kEntry;
  for (size_t tile = wave; tile * 16 < count; tile += (size_t)nblocks * waves) {
    const unsigned left = (unsigned)std::min(count - tile * 16, (size_t)16);
    OneState<NR> x;
    e.load(x, j.in + tile * (size_t)(16 * 2 * j.nl), left, j.nl, in_matrix);
    for (int pc = 0; pc < len;) {
      u32 ins = (u32)__builtin_amdgcn_readfirstlane((int)prog[pc]);
      // a run of squarings (nine tenths of a program) in a loop of its own, where the state stays in registers
#pragma unroll 1
      while (ins == ENG_SQ) {
        e.template products<true, WAVE>(x, nullptr);
        e.extend_to_b(x);
        e.extend_to_a(x);
        ins = ++pc < len ? (u32)__builtin_amdgcn_readfirstlane((int)prog[pc]) : ~0u;
      }
      if (pc++ >= len) break;
      const u32 op = ins & 0xFFu, a = (ins >> 8) & 0xFFFu, b = ins >> 20;
      u32* entry = table + (size_t)a * kEntry;
      if (op == ENG_STORE_T) {
        e.template store_state<WAVE>(x, entry);
      } else if (op == ENG_LOAD_T) {
        e.template load_state<WAVE>(x, entry);
      } else {
        e.template products<false, WAVE>(x, entry);
        e.extend_to_b(x);
        e.extend_to_a(x);
        if (op == ENG_MUL_T_ST) e.template store_state<WAVE>(x, table + (size_t)b * kEntry);
      }
    }
    e.store(x, j.out + tile * (size_t)(16 * 8 * rns::tiles(NR)), e.lane & 15, (unsigned)(e.lane & 15) < left, out_matrix);
  }
}

// Products of lists of elements, each in memory by itself as [base A, base B][quad][lane group] (rns_item_words()): a lane
// group's four lanes read 64 consecutive bytes, 18 times, from wherever the element lies.
// Into that form: lazy limb pairs as in RnsJob::in.
template <int NR>
__global__ __launch_bounds__(1024, 4) void k_rns_enter(const u32* __restrict__ tables, const u32* __restrict__ in,
                                                       size_t count, int nl, u32* __restrict__ items) {
  __shared__ __align__(16) u32 lds[rns::lds_bytes(NR) / 4];
  for (int i = (int)threadIdx.x; i < rns::lds_bytes(NR) / 16; i += (int)blockDim.x)
    ((Quad*)lds)[i] = ((const Quad*)tables)[i];
  __syncthreads();
  OneEngine<NR> e(lds);
  const unsigned waves = blockDim.x / WAVE;
  const size_t wave = (size_t)blockIdx.x * waves + (unsigned)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
  for (size_t tile = wave; tile * 16 < count; tile += (size_t)gridDim.x * waves) {
    const size_t own = tile * 16 + (threadIdx.x & 15);
    OneState<NR> x;
    e.load(x, in + tile * (size_t)(16 * 2 * nl), (unsigned)std::min(count - tile * 16, (size_t)16), nl, (const char*)tables + rns::lds_bytes(NR));
    if (own < count) e.template store_state<4>(x, items + own * (size_t)rns::item_words(NR));
  }
}

// Every wavefront multiplies 16 lists side by side, up to the longest of them. A factor's quads are on their way one step
// ahead, its place two products ahead. What bounds it are the matrix products and the vector unit's work between them, one
// after the other within a wavefront: 2.9 x 10^6 products a ms, matrix cores 59 % and vector issue 54 % of the cycles, with three
// wavefronts of 168 registers per SIMD; with four of 128, which spill 88 of them, 8 % less (65536 by 32 entries' gradient 2.81 /
// 3.19 ms). The limb arithmetic forms 1.0 x 10^6.
template <int NR>
__global__ __launch_bounds__(768, 3) void k_rns_chains(RnsChains j) {
  __shared__ __align__(16) u32 lds[rns::lds_bytes(NR) / 4];
  const u32 total = j.control[kChainsTotal];
  if (total == 0) return;
  for (int i = (int)threadIdx.x; i < rns::lds_bytes(NR) / 16; i += (int)blockDim.x)
    ((Quad*)lds)[i] = ((const Quad*)j.tables)[i];
  __syncthreads();
  const bool columns = j.control[kChainsColumns] != 0;
  OneEngine<NR> e(lds);
  const unsigned waves = blockDim.x / WAVE;
  // The first runs, the longest, are spread over all compute units; the wavefronts draw the ones behind them from a counter.
  u32 at = ((unsigned)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE)) * gridDim.x + blockIdx.x) * 16;
  const u32 drawn_from = gridDim.x * waves * 16;
  while (at < total) {
    const u32 own = at + (threadIdx.x & 15);
    const bool active = own < total;
    const Quad c = active ? ((const Quad*)j.chains)[own] : Quad{0, 0, 0, 0};
    const u32 first = c[1], len = c[2];
    // an element whose list has ended is multiplied by one
    const auto item = [&](u32 i) -> u32 { return i < len ? j.index ? j.index[first + i] : first + i : 0u; };
    const auto element = [&](u32 i, u32 at) {
      return i < len ? j.items + (size_t)at * rns::item_words(NR) : j.one;
    };
    u32 longest = (u32)__builtin_amdgcn_readfirstlane((int)wave_max(len));
    // An element as it lies in memory need not have alpha in its slot, which the way out takes: what leaves has been a product.
    if (columns && longest < 2) longest = 2;
    OneState<NR> x;
    e.template load_state<4>(x, element(0, item(0)));
    u32 next = item(1);
#pragma unroll 1
    for (u32 i = 1; i < longest; ++i) {
      const u32* y = element(i, next);
      next = item(i + 1);
      e.template products<false, 4>(x, y);
      e.extend_to_b(x);
      e.extend_to_a(x);
    }
    if (columns) {
      e.store(x, j.columns + (size_t)c[0] * (8 * rns::tiles(NR)), 0, active, (const char*)j.tables + rns::lds_bytes(NR) + rns::in_matrix_bytes(NR));
    } else if (active) {
      e.template store_state<4>(x, j.out + (size_t)c[0] * rns::item_words(NR));
    }
    u32 drawn = 0;
    if (e.lane == 0) drawn = atomicAdd(j.next, 16u);
    at = drawn_from + (u32)__builtin_amdgcn_readfirstlane((int)drawn);
  }
}

// What the wavefronts of a block of k_rns_group share, whichever tiles they have.
// LISTS: of k_rns_lists, whose registers go to two values and an operand on its way: its constants lie in LDS.
template <int NR, int HALVES, bool LISTS>
struct GroupShared {
  static constexpr int kBlocks = (NR + 3) / 4;  // of 64 bytes, the last one partly empty
  static constexpr bool kHeldCst = !LISTS;
  Quad bytes[2][HALVES][kBlocks][WAVE];  // [sigma, rho][x0, x1][block][lane]
  Quad sum[3][HALVES][16];               // alpha's sums over lane group 0 .. 3's slots, of the last, the present and the next rho
  Quad cst[kHeldCst ? 0 : 2][rns::slots(NR)];
};

// The same arithmetic with the slots of 16 elements spread over the W wavefronts of a block, TW tiles each, for batches that
// would leave most of the chip idle with a wavefront per 16 elements. A wavefront keeps the residues of its own slots and
// multiplies and reduces them alone; what every wavefront needs of the others, the bytes of all residues, goes through LDS (16
// bytes per lane and block of 64, as the matrix product reads its operand), one barrier before each of the two matrix products
// of a modular product. The matrices stay in registers, 16 to 80 of them. What bounds it is one wavefront's chain from barrier
// to barrier and the SIMD with the most tiles (three of a 1024-bit modulus's nine): on blocks of 8 elements a product takes
// some 1450 and 2100 cycles of 2.4 GHz (1024 and 2048 bits). Measured against the limb arithmetic on one wavefront per integer,
// the version before blocks of 8 elements and weighted rows, and the one before the program's words were kept in registers, a
// square's lanes of x1 took a second multiply-add instead of a 64-bit factor, and alpha's sums were cleared off the first SIMD:
// 1024 encryptions at a 1024-bit key 2.67, 1.06, 0.85 -> 0.73 ms, 256 at 2048 bits 8.5, 3.9, 2.30 -> 2.08; 3072 decryptions at
// 1024 bits 1.33, 0.55, 0.51 -> 0.47 ms, 100 at 2048 bits (the last two) 0.89 -> 0.77, 64 at 4096 bits 8.63, 4.01, 2.38 ->
// 2.14.
//
// FOLD: 8 elements to a block, x0 in columns 0 to 7 of the matrix products and x1 in columns 8 to 15, for batches that do
// not fill the chip with blocks of 16: half the matrix instructions and operand reads per product. A lane then has one half
// of a pair; x1's lanes take the first half's values by DPP, x0's run through the same instructions with zeros in place.
// W wavefronts, TILES tiles in all.
template <int NR, int TW, int W, int TILES, bool PAIR, bool FOLD, bool LISTS = false>
struct RnsGroup {
  static constexpr bool kBoth = PAIR && !FOLD;  // x0 and x1 in one lane
  static constexpr int kHalves = kBoth ? 2 : 1;
  static constexpr int kElements = FOLD ? 8 : 16;
  static constexpr int kRegs = NR, kOwn = TW;
  static constexpr int kTiles = rns::tiles(NR);
  static constexpr int kLimbTiles = rns::limb_tiles(NR);
  static constexpr bool kClearLate = NR <= 10;  // where alpha's old sums are cleared, see publish()
  using Shared = GroupShared<NR, kHalves, LISTS>;
  static constexpr int kBlocks = Shared::kBlocks;
  static constexpr int kFull = rns::full_blocks(NR);
  static constexpr int kTileBytes = rns::tile_bytes(NR, 16);
  static constexpr bool kHeldCst = Shared::kHeldCst;
  static_assert(TILES >= kLimbTiles, "every tile has a wavefront");
  static_assert(!LISTS || (PAIR && FOLD), "elements in memory by themselves are taken by halves");
  struct State {
    u32 a0[TW], a1[TW], b0[TW], b1[TW];
  };
  using Frags = QuadSet<TW * kBlocks>;
  Shared& sh;
  const char* tables;
  int lane, g, wave, own_tile, turn;  // own_tile: the first of TW
  Acc start;
  Quad held_cst[2][kHeldCst ? TW : 1];  // the constants of this lane's slots in base A and base B
  u32 second;           // FOLD: all ones in x1's lanes
  Frags held[2];

  __device__ __forceinline__ bool mine(int i, int tiles = kTiles) const { return own_tile + i < tiles; }
  // a wavefront without a tile of its own repeats the last one and keeps the result to itself
  __device__ __forceinline__ int tile(int i, int tiles = kTiles) const { return mine(i, tiles) ? own_tile + i : tiles - 1; }
  // this lane holds a prime's residue (not one of the extra values) in tile i
  __device__ __forceinline__ bool owns(int i) const { return mine(i) && 4 * tile(i) + g < rns::primes_for(NR); }

  __device__ __forceinline__ Quad cst(int base, int i) const { return kHeldCst ? held_cst[base][kHeldCst ? i : 0] : sh.cst[kHeldCst ? 0 : base][4 * tile(i) + g]; }

  // FOLD: x0's value for both halves; and for x1's lanes only, zero in x0's
  static __device__ __forceinline__ u32 of_first(u32 v) {
    return (u32)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x118 /* row_shr:8 */, 0xf, 0xc, false);
  }
  static __device__ __forceinline__ u32 from_first(u32 v) {
    return (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x118 /* row_shr:8 */, 0xf, 0xf, true);
  }

  // `l`: the lane
  __device__ __forceinline__ Acc fragment(const char* matrix, int tiles, int last, int i, int k, unsigned l) const {
    const int t = tile(i, tiles), rows = t == tiles - 1 ? last : 16;
    const char* p = matrix + t * kTileBytes + k * rows * 64;
    const unsigned at = ((l >> 4) * (unsigned)rows + (l & (unsigned)(rows - 1))) * 16;
    if (k < kFull) return *(const Acc*)(p + at);
    const Twin h = *(const Twin*)(p + at / 2);
    return Acc{(int)h[0], (int)h[1], 0, 0};
  }

  __device__ __forceinline__ RnsGroup(Shared& shared, const u32* tables_, int own_tile_)
      : sh(shared), tables((const char*)tables_), lane((int)(threadIdx.x & (WAVE - 1))), g(lane >> 4),
        wave(__builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE))), own_tile(own_tile_), turn(0), start(start_sums()),
        second(FOLD && (threadIdx.x & 8) ? ~0u : 0u) {
    const char* from = tables + rns::lds_matrices_bytes(NR);
    if (kHeldCst)
#pragma unroll
      for (int i = 0; i < TW; ++i)
#pragma unroll
        for (int b = 0; b < 2; ++b) held_cst[b][kHeldCst ? i : 0] = *(const Quad*)(from + (2 * b * rns::slots(NR) + 4 * tile(i) + g) * 16);
#pragma unroll
    for (int mat = 0; mat < 2; ++mat)
#pragma unroll
      for (int i = 0; i < TW; ++i)
#pragma unroll
        for (int k = 0; k < kBlocks; ++k)
          held[mat].q[i * kBlocks + k] = fragment(tables + mat * rns::lds_matrix_bytes(NR, 0), kTiles, rns::last_rows(NR, mat), i, k, (unsigned)lane);
    for (int i = (int)threadIdx.x; i < (int)(sizeof(Shared) / 4); i += (int)blockDim.x) ((u32*)&sh)[i] = 0;
    __syncthreads();
    if (!kHeldCst)
      for (int i = (int)threadIdx.x; i < 2 * rns::slots(NR); i += (int)blockDim.x)
        sh.cst[kHeldCst ? 0 : i / rns::slots(NR)][i % rns::slots(NR)] = *(const Quad*)(from + (i + i / rns::slots(NR) * rns::slots(NR)) * 16);
    set_bias();
  }
  // A residue's bytes to where the other wavefronts read them. All lanes write: what has no prime meets zeros in the matrix,
  // a wavefront that repeats a tile writes what its owner does, and the bias stays 1 where it shares a register with primes.
  __device__ __forceinline__ void put(int buffer, int x, int i, u32 v) const {
    v ^= rns::kOmega;
    if (rns::tiles(NR) == NR && tile(i) == NR - 1) v = g == rns::bias_group(NR) ? 1u : v;
    word(buffer, x, tile(i), lane) = v;
  }
  // the constant 1 of the bias: a lane group of the last register, which no wavefront writes
  __device__ __forceinline__ void set_bias() {
    if (threadIdx.x < 16)
      for (int b = 0; b < 2; ++b)
        for (int x = 0; x < kHalves; ++x) word(b, x, NR - 1, 16 * rns::bias_group(NR) + (int)threadIdx.x) = 1;
  }
  __device__ __forceinline__ u32& word(int buffer, int x, int i, int l) const {
    return ((u32*)&sh.bytes[buffer][x][i / 4][l])[i % 4];
  }

  // r = the tiles' products with the bytes in `buffer`, after all wavefronts have written theirs. MATRIX 0, 1: the two
  // of the modular product; ALPHA: its lane group of the last register takes alpha.
  template <int MATRIX, bool ALPHA>
  __device__ __forceinline__ void products(Acc (&r)[TW][kHalves], int buffer, const char* matrix, int tiles, int last, const Acc& from) {
    unsigned l = (unsigned)lane;
    asm volatile("" : "+v"(l));  // or the addresses of all fragments are kept in registers from one product to the next
    u32 alpha[kHalves];
    if (ALPHA) {
#pragma unroll
      for (int x = 0; x < kHalves; ++x) {
        const Quad q = sh.sum[turn == 0 ? 2 : turn - 1][x][lane & 15];
        alpha[x] = alpha_bytes(q[0] + q[1] + q[2] + q[3] + (1u << 13) + (u32)rns::primes_for(NR) / 2);
      }
    }
#pragma unroll
    for (int i = 0; i < TW; ++i)
#pragma unroll
      for (int x = 0; x < kHalves; ++x) r[i][x] = from;
    const auto block = [&](int k, const Acc* f) {
      Quad d[kHalves];
#pragma unroll
      for (int x = 0; x < kHalves; ++x) {
        d[x] = sh.bytes[buffer][x][k][lane];
        if (ALPHA && k == (NR - 1) / 4) d[x][(NR - 1) % 4] = g == rns::alpha_group(NR) ? alpha[x] : d[x][(NR - 1) % 4];
      }
#pragma unroll
      for (int i = 0; i < TW; ++i)
#pragma unroll
        for (int x = 0; x < kHalves; ++x)
          r[i][x] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f[i], (Acc)d[x], r[i][x], 0, 0, 0);
    };
#pragma unroll
    for (int k = 0; k < kBlocks; ++k) {
      if (MATRIX == 2 && k % 3 == 0) __builtin_amdgcn_sched_barrier(0);
      Acc f[TW];
#pragma unroll
      for (int i = 0; i < TW; ++i)
        f[i] = MATRIX < 2 ? held[MATRIX < 2 ? MATRIX : 0].q[i * kBlocks + k] : fragment(matrix, tiles, last, i, k, l);
      block(k, f);
    }
  }
  // base B's bytes and alpha's sums to the other wavefronts
  __device__ __forceinline__ void publish(const State& x) {
    u32 s0 = 0, s1 = 0;
#pragma unroll
    for (int i = 0; i < TW; ++i) {
      put(1, 0, i, x.b0[i]);
      if constexpr (kBoth) put(1, 1, i, x.b1[i]);
      s0 += owns(i) ? (u32)((s32)x.b0[i] >> 16) : 0u;
      if constexpr (kBoth) s1 += owns(i) ? (u32)((s32)x.b1[i] >> 16) : 0u;
    }
    u32* s = (u32*)&sh.sum[turn][0][lane & 15] + g;
    atomicAdd(s, s0);
    if (kBoth) atomicAdd(s + 64, s1);
    __syncthreads();
    turn = turn == 2 ? 0 : turn + 1;
    // At once, or after the matrix product: 1024 encryptions at a 1024-bit key 785 / 771 us, 256 at 2048 bits 2142 / 2198
    if (!kClearLate) clear_sums();
  }
  // The sums of the publish() before the last one, which were last read before its barrier, are next added to after the
  // barrier of the one that follows: called between the two.
  __device__ __forceinline__ void clear_sums() const {
    if (wave == 3)  // of a SIMD that has fewer tiles than the first one
#pragma unroll
      for (int x = 0; x < kHalves; ++x) ((u32*)&sh.sum[turn == 2 ? 0 : turn + 1][x][0])[lane] = 0;
  }
  // base A from what publish() left
  __device__ __forceinline__ void extend_to_a(State& x) {
    Acc r[TW][kHalves];
    products<1, true>(r, 1, tables + rns::lds_matrix_bytes(NR, 0), kTiles, rns::last_rows(NR, 1), start);
    if (kClearLate) clear_sums();
#pragma unroll
    for (int i = 0; i < TW; ++i) {
      const Quad k = cst(0, i);
      x.a0[i] = reduce(column(r[i][0]), k[0], k[1]);
      if constexpr (kBoth) x.a1[i] = reduce(column(r[i][kHalves - 1]), k[0], k[1]);
    }
  }
  // the residue products of one base of slot i: x0 y0 and x0 y1 + x1 y0 + e x0 y0 (e: of the reduced first one)
  template <bool SQ>
  __device__ __forceinline__ void residues(u32& r0, u32& r1, u32 u0, u32 u1, u32 v0, u32 v1, u32 p, u32 pinv, u32 e) const {
    if constexpr (FOLD) {
      s64 t;
      if constexpr (SQ) {  // x1's lanes twice, hidden from the compiler, which would multiply a wider sum of factors
        const u32 first = of_first(u0);
        t = smad(first, u0, 0);
        asm("" : "+v"(t));
        t = smad(first, u0 & second, t);
      } else {
        t = smad(of_first(u0), v0, smad(u0 & second, of_first(v0), 0));
      }
      r0 = reduce(smad(from_first(reduce(t, p, pinv)), e, t), p, pinv);
      r1 = 0;
    } else {
      r0 = reduce(smad(u0, v0, 0), p, pinv);
      r1 = 0;
      if constexpr (kBoth) r1 = reduce(smad(r0, e, SQ ? twice(u0, u1) : smad(u0, v1, smad(u1, v0, 0))), p, pinv);
    }
  }
  // x times the table entry y, or (null) squared
  template <bool SQ>
  __device__ __forceinline__ void multiply(State& x, const u32* y) {
    Quad v[TW];
#pragma unroll
    for (int i = 0; i < TW; ++i) v[i] = SQ ? own(x, i) : entry(y, i);
    multiply<SQ>(x, v, [] {});
  }
  __device__ __forceinline__ void begin() {}  // for run_lists(): all matrices are held, none on its way
  // `meanwhile` asks for what the next product takes, behind this one's first barrier
  template <bool SQ, class F>
  __device__ __forceinline__ void multiply(State& x, const Quad (&v)[TW], const F& meanwhile) {
    u32 z[TW], w[TW];
#pragma unroll
    for (int i = 0; i < TW; ++i) {
      const Quad k = cst(0, i);
      u32 s0, s1;
      residues<SQ>(s0, s1, x.a0[i], kBoth ? x.a1[i] : 0u, v[i][0], v[i][1], k[0], k[1], k[2]);
      put(0, 0, i, s0);
      if constexpr (kBoth) put(0, 1, i, s1);
    }
    __syncthreads();
    meanwhile();
    // base B's share is not needed before the matrix product's result
#pragma unroll
    for (int i = 0; i < TW; ++i) {
      const Quad k = cst(1, i);
      residues<SQ>(z[i], w[i], x.b0[i], kBoth ? x.b1[i] : 0u, v[i][2], v[i][3], k[0], k[1], 0u - k[3]);
    }
    Acc r[TW][kHalves];
    products<0, false>(r, 0, tables, kTiles, rns::last_rows(NR, 0), start);
#pragma unroll
    for (int i = 0; i < TW; ++i) {
      const Quad k = cst(1, i);
      s64 col = smad(z[i], k[2], column(r[i][0]));
      u32 t0 = reduce(col, k[0], k[1]);
      if constexpr (FOLD) t0 = reduce(smad(from_first(t0), k[3], col), k[0], k[1]);
      x.b0[i] = t0;
      if constexpr (kBoth) {
        col = smad(w[i], k[2], column(r[i][kHalves - 1]));
        x.b1[i] = reduce(smad(t0, k[3], col), k[0], k[1]);
      }
    }
    publish(x);
    extend_to_a(x);
  }
  // the pairs whose limbs are at `src` (`left` of them, then zeros) into both bases
  __device__ __forceinline__ void load(State& x, const u32* src, unsigned left, int nl) {
    const int e = lane & (kElements - 1), half = FOLD ? lane >> 3 & 1 : 0;
    __syncthreads();  // the bytes of the elements before have been read
    for (int i = wave; i < NR; i += W) {
      const int l = 4 * i + g;
      if (l == rns::bias_slot(NR)) continue;
      const bool ok = (unsigned)e < left && l < nl;
      const u32* p = src + (size_t)e * (2 * nl) + half * nl + l;
      word(0, 0, i, lane) = (ok ? p[0] : 0u) ^ rns::kOmega;
      if constexpr (kBoth) word(0, 1, i, lane) = (ok ? p[nl] : 0u) ^ rns::kOmega;
    }
    __syncthreads();
    Acc r[TW][kHalves];
    products<2, false>(r, 0, tables + rns::lds_bytes(NR), kTiles, 16, start);
#pragma unroll
    for (int i = 0; i < TW; ++i) {
      const Quad k = cst(1, i);
      x.b0[i] = reduce(column(r[i][0]), k[0], k[1]);
      if constexpr (kBoth) x.b1[i] = reduce(column(r[i][kHalves - 1]), k[0], k[1]);
    }
    publish(x);
    extend_to_a(x);
  }
  // the pairs as two integers each in columns of weight 2^(29 l)
  __device__ __forceinline__ void store(const State& x, long long* dst, unsigned left) {
    const unsigned e = (unsigned)(lane & (kElements - 1));
    store(x, dst, e, e < left);
  }
  // the same, this lane's to element `e` behind `dst`
  template <class I>
  __device__ __forceinline__ void store(const State& x, long long* dst, I e, bool active) {
    __syncthreads();  // the bytes of the last product have been read
    publish(x);
    Acc r[TW][kHalves];
    products<2, true>(r, 1, tables + rns::lds_bytes(NR) + rns::in_matrix_bytes(NR), kLimbTiles, 16, Acc{0, 0, 0, 0});
    if (kClearLate) clear_sums();
#pragma unroll
    for (int i = 0; i < TW; ++i) {
      const unsigned half = FOLD ? (unsigned)lane >> 3 & 1 : 0;
      if (active && mine(i, kLimbTiles)) {
        long long* d = dst + (size_t)e * (8 * kLimbTiles) + half * (4 * kLimbTiles) + 4 * tile(i, kLimbTiles) + g;
        d[0] = integer(r[i][0]);
        if (!FOLD) d[4 * kLimbTiles] = kBoth ? integer(r[i][kHalves - 1]) : 0;
      }
    }
  }
  // Window tables: [tile][lane] quads {x0, x1 in base A, in base B}, of one half alone {base A, base B}
  static constexpr int kWords = kBoth ? 4 : 2;
  static constexpr int kEntry = TILES * WAVE * kWords;  // dwords
  __device__ __forceinline__ u32* entry_at(const u32* entry, int i) const {
    return (u32*)entry + ((own_tile + i) * WAVE + lane) * kWords;
  }
  static __device__ __forceinline__ Quad own(const State& x, int i) {
    return Quad{x.a0[i], kBoth ? x.a1[i] : 0u, x.b0[i], kBoth ? x.b1[i] : 0u};
  }
  __device__ __forceinline__ Quad entry(const u32* entry, int i) const {
    if constexpr (kBoth) return *(const Quad*)entry_at(entry, i);
    const Twin v = *(const Twin*)entry_at(entry, i);
    return Quad{v[0], 0, v[1], 0};
  }
  // LISTS: the same of an element in memory by itself (see item_words): where the word of this lane's half is
  __device__ __forceinline__ int item_at(int base, int i) const {
    const int t = tile(i), half = lane >> 3 & 1;
    const int quad = t < 4 * kFull ? 2 * (t / 4) + half : 2 * kFull, word = t < 4 * kFull ? t % 4 : 2 * half + t % 4;
    return base * (rns::item_words(NR) / 2) + (quad * 4 + g) * 4 + word;
  }
  __device__ __forceinline__ void load_item(Quad (&v)[TW], const u32* item) const {
#pragma unroll
    for (int i = 0; i < TW; ++i) v[i] = Quad{item[item_at(0, i)], 0u, item[item_at(1, i)], 0u};
  }
  __device__ __forceinline__ void store_item(const State& x, u32* item) const {
#pragma unroll
    for (int i = 0; i < TW; ++i) {
      if (!mine(i)) continue;
      item[item_at(0, i)] = x.a0[i];
      item[item_at(1, i)] = x.b0[i];
    }
  }
  static __device__ __forceinline__ void set(State& x, const Quad (&v)[TW]) {
#pragma unroll
    for (int i = 0; i < TW; ++i) {
      x.a0[i] = v[i][0];
      x.b0[i] = v[i][2];
    }
  }
  __device__ __forceinline__ void store_state(const State& x, u32* entry) const {
#pragma unroll
    for (int i = 0; i < TW; ++i)
      if constexpr (kBoth) *(Quad*)entry_at(entry, i) = own(x, i);
      else *(Twin*)entry_at(entry, i) = Twin{x.a0[i], x.b0[i]};
  }
  __device__ __forceinline__ void load_state(State& x, const u32* y) const {
#pragma unroll
    for (int i = 0; i < TW; ++i) {
      const Quad v = entry(y, i);
      x.a0[i] = v[0];
      x.b0[i] = v[2];
      if constexpr (kBoth) {
        x.a1[i] = v[1];
        x.b1[i] = v[3];
      }
    }
  }
};

// The engine of 4096-bit moduli, whose matrices, 630 KB, fit neither a wavefront's registers nor the LDS: the slots of 16 (FOLD: 8)
// elements spread over a block of four wavefronts, one to a SIMD, each with all 512 of its registers and nine tiles. Against twelve
// wavefronts of three tiles, the form before:
// - the operand of a matrix product is read from LDS once by each of four wavefronts, and not of twelve: 144 KB instead of 432 for the
//   two matrix products of a modular one;
// - of the 18 blocks of both matrices a tile has, 10 stay on the compute unit instead of 6: 7 in registers, in the half that only
//   loads and the matrix unit reach, and three in LDS. 288 KB instead of 420 come from L2 for a modular product;
// - a matrix product goes tile by tile, with the vector unit's work on one tile between the matrix instructions of the next: the
//   phases of the twelve wavefronts lay one after the other between their barriers.
// ms before and now: encryption of 64 elements 17.8 / 12.6, 3001 21.7 / 18.8, 4096 25.5 / 21.4, 20000 125.6 / 105.1; gradient 20000 by
// 64 8.76 / 5.9, forward 4096 by 64 1.72 / 1.30. What bounds it is the issue of a SIMD's only wavefront (without the blocks that
// stream 64 and 3001 elements take 9.7 and 14.3) and the 64 bytes a clock that they come with; the entries of a window table are
// waited for.
template <bool FOLD>
struct WideShared {
  static constexpr int kNr = 36, kHalves = FOLD ? 1 : 2;
  Quad bytes[2][kHalves][rns::full_blocks(kNr)][WAVE];  // [sigma, rho][x0, x1][block][lane]
  Quad sum[3][kHalves][16];                             // see GroupShared
  Quad cst[2][rns::slots(kNr)];
  Acc resident[4][9][3][WAVE];                          // [wavefront][tile][block]: one address and constants reach all of a lane's
};
template <bool FOLD, int STREAM0, int STREAM1, int RING, bool HELD>
struct RnsWide {
  static constexpr int kRegs = 36, kOwn = 9, kWaves = 4;
  static constexpr bool kBoth = !FOLD;  // x0 and x1 in one lane
  static constexpr int kHalves = kBoth ? 2 : 1;
  static constexpr int kElements = FOLD ? 8 : 16;
  static constexpr int kTiles = rns::tiles(kRegs), kLimbTiles = rns::limb_tiles(kRegs);
  static constexpr int kBlocks = rns::full_blocks(kRegs), kTileBytes = rns::tile_bytes(kRegs, 16);
  static_assert(kRegs % 4 == 0 && kLimbTiles == kOwn * kWaves && kTiles == kLimbTiles - 1, "whole blocks, and a tile without primes");
  using Shared = WideShared<FOLD>;
  // A tile's blocks, in the order in which they are multiplied: every other one streams, so that the requests come evenly, up to
  // STREAM0 of the first matrix and STREAM1 of the second one. Of the rest, the first ones stay in registers, the last three of the
  // second matrix in LDS.
  static constexpr int kLds = 3;
  static constexpr int kStay0 = kBlocks - STREAM0, kStay1 = kBlocks - kLds - STREAM1;
  static __host__ __device__ constexpr int count(int m) { return m == 0 ? STREAM0 : STREAM1; }
  static __host__ __device__ constexpr bool streams(int m, int n) { return n % 2 == 0 && n / 2 < count(m); }
  static __host__ __device__ constexpr int rest(int m, int n) { return n - (n + 1 < 2 * count(m) ? (n + 1) / 2 : count(m)); }  // its number
  static __host__ __device__ constexpr int rest_block(int m, int r) { return r < count(m) ? 2 * r + 1 : r + count(m); }
  static_assert(2 * STREAM0 <= kBlocks && 2 * STREAM1 <= kBlocks && rest_block(0, rest(0, 8)) == 8 && rest_block(1, rest(1, 1)) == 1, "");
  // Tiles whose matrix products are issued in turn, with the vector unit's work on as many others between them: a step
  static constexpr int kStep = FOLD ? 2 : 1;
  static __host__ __device__ constexpr int stream_begin(int m) { return m == 0 ? 0 : kOwn * STREAM0; }  // in a product's
  static_assert(kOwn * (STREAM0 + STREAM1) % RING == 0 && RING <= kOwn * STREAM0 && RING <= kOwn * STREAM1, "a product begins where the last one ended");
  // The n-th block of tile i that streams, in the order in which they are multiplied: by steps, by blocks, by tiles
  static __host__ __device__ constexpr int step_tiles(int t) { return t + kStep <= kOwn ? kStep : kOwn - t; }
  static __host__ __device__ constexpr int stream_at(int m, int i, int n) { return i / kStep * kStep * count(m) + n * step_tiles(i / kStep * kStep) + i % kStep; }
  static __host__ __device__ constexpr int stream_step(int m, int s) { return s / (kStep * count(m)) * kStep; }
  static __host__ __device__ constexpr int stream_block(int m, int s) { return s % (kStep * count(m)) / step_tiles(stream_step(m, s)); }
  static __host__ __device__ constexpr int stream_tile(int m, int s) { return stream_step(m, s) + s % (kStep * count(m)) % step_tiles(stream_step(m, s)); }
  // HELD: a value's residues in base B are registers of its state. Else they are only where the other wavefronts read them, but
  // for the last tile's, which two wavefronts have: a lane reads its own back from there, and there are registers for more
  // blocks on their way.
  static constexpr int kHeldB = HELD ? kOwn : 1;
  struct State {
    u32 a0[kOwn], a1[kOwn], b0[kHeldB], b1[kHeldB];
  };
  struct Sums {
    Acc r[kHalves];
  };
  struct Words {  // x0's and x1's in one base
    Twin w[kOwn];
  };
  Shared& sh;
  const char* tables;
#if defined(__HIP_DEVICE_COMPILE__)
  __amdgpu_buffer_rsrc_t rows;  // of both matrices
#endif
  int lane, g, wave, turn;
  unsigned place;
  Acc start;
  u32 second;  // FOLD: all ones in x1's lanes
  u32 last;    // all ones where the ninth tile has a prime
  QuadSet<kOwn * kStay0> stay0;
  QuadSet<kOwn * kStay1> stay1;
  QuadSet<RING> ring;

  // Tile i of this wavefront: two blocks of four and one of the last block
  __device__ __forceinline__ int limb_tile(int i) const { return i < 8 ? 8 * wave + i : 32 + wave; }
  // of those with primes: the last wavefront repeats the last one and keeps the result to itself
  __device__ __forceinline__ bool mine(int i) const { return i < 8 || limb_tile(i) < kTiles; }
  __device__ __forceinline__ int tile(int i) const { return mine(i) ? limb_tile(i) : kTiles - 1; }
  __device__ __forceinline__ Quad cst(int base, int i) const { return sh.cst[base][4 * tile(i) + g]; }
  // FOLD: x0's value for both halves; and for x1's lanes only, zero in x0's
  static __device__ __forceinline__ u32 of_first(u32 v) {
    return (u32)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x118 /* row_shr:8 */, 0xf, 0xc, false);
  }
  static __device__ __forceinline__ u32 from_first(u32 v) {
    return (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x118 /* row_shr:8 */, 0xf, 0xf, true);
  }
  static __device__ __forceinline__ Acc fragment(const char* matrix, int tile, int k, unsigned at) {
    return *(const Acc*)(matrix + tile * kTileBytes + k * 1024 + at);
  }
  // Fragment n of those that stay, the first 63 in the half of the registers that only loads and the matrix unit reach: left alone,
  // the compiler copies what it keeps there to the other half for each use.
  static __device__ __forceinline__ Acc stays([[maybe_unused]] int n, Acc f) {
#if defined(__HIP_DEVICE_COMPILE__)
    if (n < 63) asm("" : "+a"(f));
#endif
    return f;
  }
  __device__ __forceinline__ const char* matrix(int m) const { return tables + m * rns::lds_matrix_bytes(kRegs, 0); }
  // this lane's place in a fragment, made anew: or the addresses of all fragments are kept in registers from one product to the next
  __device__ __forceinline__ unsigned fresh_place() const {
    unsigned l = place;
    asm volatile("" : "+v"(l));
    return l;
  }

  __device__ __forceinline__ RnsWide(Shared& shared, const u32* tables_)
      : sh(shared), tables((const char*)tables_), lane((int)(threadIdx.x & (WAVE - 1))), g(lane >> 4),
        wave(__builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE))), turn(0), place(16 * (threadIdx.x & (WAVE - 1))),
        start(start_sums()), second(FOLD && (threadIdx.x & 8) ? ~0u : 0u), last(mine(8) && 4 * tile(8) + g < rns::primes_for(kRegs) ? ~0u : 0u) {
#if defined(__HIP_DEVICE_COMPILE__)
    rows = __builtin_amdgcn_make_buffer_rsrc((void*)tables, 0, rns::lds_matrices_bytes(kRegs), 0x00020000 /* untyped words */);
#endif
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
#pragma unroll
      for (int k = 0; k < kStay0; ++k) stay0.q[i * kStay0 + k] = stays(i * kStay0 + k, fragment(matrix(0), tile(i), rest_block(0, k), place));
#pragma unroll
      for (int k = 0; k < kStay1; ++k)
        stay1.q[i * kStay1 + k] = stays(kOwn * kStay0 + i * kStay1 + k, fragment(matrix(1), tile(i), rest_block(1, k), place));
#pragma unroll
      for (int k = 0; k < kLds; ++k) sh.resident[wave][i][k][lane] = fragment(matrix(1), tile(i), rest_block(1, kStay1 + k), place);
    }
    constexpr int kClear = (int)(sizeof(sh.bytes) + sizeof(sh.sum)) / 4;
    for (int i = (int)threadIdx.x; i < kClear; i += (int)blockDim.x) ((u32*)&sh)[i] = 0;
    const char* from = tables + rns::lds_matrices_bytes(kRegs);
    for (int i = (int)threadIdx.x; i < 2 * rns::slots(kRegs); i += (int)blockDim.x)
      sh.cst[i / rns::slots(kRegs)][i % rns::slots(kRegs)] = *(const Quad*)(from + (i + i / rns::slots(kRegs) * rns::slots(kRegs)) * 16);
    __syncthreads();
    // the constant 1 of the bias: a lane group of the last register, which no wavefront writes
    if (threadIdx.x < 16)
      for (int b = 0; b < 2; ++b)
        for (int x = 0; x < kHalves; ++x) word(b, x, kRegs - 1, 16 * rns::bias_group(kRegs) + (int)threadIdx.x) = 1;
  }
  __device__ __forceinline__ u32& word(int buffer, int x, int i, int l) const {
    return ((u32*)&sh.bytes[buffer][x][i / 4][l])[i % 4];
  }
  // Residues' bytes to where the other wavefronts read them, once the value of tile i is there: four at a time. All lanes write,
  // what has no prime meets zeros in the matrix.
  __device__ __forceinline__ void put(int buffer, int x, int i, const u32 (&v)[kOwn]) const {
    if (i == 8) word(buffer, x, tile(8), lane) = v[8] ^ rns::kOmega;
    else if (i % 4 == 3) sh.bytes[buffer][x][2 * wave + i / 4][lane] = Quad{v[i - 3], v[i - 2], v[i - 1], v[i]} ^ rns::kOmega;
  }
  // Asks for block s of those of a matrix that stream. A lane's place in a fragment never changes and a tile's lies in a scalar
  // register, so that it takes one instruction.
  template <int MATRIX>
  __device__ __forceinline__ void ask(int s) {
    const int i = stream_tile(MATRIX, s), k = stream_block(MATRIX, s);
    const int tile_at = MATRIX * rns::lds_matrix_bytes(kRegs, 0) + (i < 8 ? 8 * wave + i : tile(8)) * kTileBytes;
    const unsigned at = place + (unsigned)k * 2048;
    Acc f;
#if defined(__HIP_DEVICE_COMPILE__)
    f = __builtin_amdgcn_raw_buffer_load_b128(rows, (int)at, tile_at, 0);
#else
    f = *(const Acc*)(tables + tile_at + at);
#endif
    ring.q[(s + stream_begin(MATRIX)) % RING] = f;
  }
  // before the first product of elements that load() did not bring in
  __device__ __forceinline__ void begin() {
#pragma unroll
    for (int s = 0; s < RING; ++s) ask<0>(s);
  }
  struct Operand {
    Acc q[kHalves][kBlocks];
  };
  // the bytes in `buffer`, after all wavefronts have written theirs; ALPHA: with alpha in its slot
  template <bool ALPHA>
  __device__ __forceinline__ void read(Operand& d, int buffer) const {
    u32 alpha[kHalves] = {};
    if (ALPHA) {
#pragma unroll
      for (int x = 0; x < kHalves; ++x) {
        const Quad q = sh.sum[turn == 0 ? 2 : turn - 1][x][lane & 15];
        alpha[x] = alpha_bytes(q[0] + q[1] + q[2] + q[3] + (1u << 13) + (u32)rns::primes_for(kRegs) / 2);
      }
    }
#pragma unroll
    for (int k = 0; k < kBlocks; ++k)
#pragma unroll
      for (int x = 0; x < kHalves; ++x) {
        Quad q = sh.bytes[buffer][x][k][lane];
        if (ALPHA && k == kBlocks - 1) q[3] = g == rns::alpha_group(kRegs) ? alpha[x] : q[3];
        d.q[x][k] = (Acc)q;
      }
  }
  // The matrix product of this wavefront's tiles, a step at a time. Between the matrix instructions of block n, work(i, n, k) is
  // piece n of what the vector unit can do for the step's tile i without its sums, and finish(i, n, k, sums) of what it does with
  // the sums of the step before; k: the constants of base 1 - MATRIX. ready(i) asks LDS for what work() takes of tile i, a step
  // ahead. The order is as it stands here, and the compiler's only within a block: left to itself it asks for blocks so late that
  // the next one waits for them, and leaves the vector unit's work to the end.
  template <int MATRIX, class R, class B, class F>
  __device__ __forceinline__ void sweep(const Operand& d, const R& ready, const B& work, const F& finish) {
    Sums v[2][kStep];
    Quad c[3][kStep];
#pragma unroll
    for (int j = 0; j < kStep; ++j) {
      c[0][j] = cst(1 - MATRIX, j);
      ready(j);
    }
#pragma unroll
    for (int t = 0; t < kOwn; t += kStep) {
      const int step = t / kStep, now = step % 2;
      Acc lds[kStep][kLds];
#pragma unroll
      for (int n = 0; n < kBlocks; ++n) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < kStep; ++j) {
          const int i = t + j;
          if (i >= kOwn) continue;
          const int r = streams(MATRIX, n) ? 0 : rest(MATRIX, n);
          Acc f;
          if (streams(MATRIX, n)) f = ring.q[(stream_at(MATRIX, i, n / 2) + stream_begin(MATRIX)) % RING];
          else if (MATRIX == 0) f = stay0.q[i * kStay0 + r];
          else if (r < kStay1) f = stay1.q[i * kStay1 + (r < kStay1 ? r : 0)];
          else f = lds[j][r < kStay1 ? 0 : r - kStay1];
#pragma unroll
          for (int x = 0; x < kHalves; ++x)
            v[now][j].r[x] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f, d.q[x][n], n == 0 ? start : v[now][j].r[x], 0, 0, 0);
          if (streams(MATRIX, n)) {
            const int s = stream_at(MATRIX, i, n / 2) + RING;
            if (s < kOwn * count(MATRIX)) ask<MATRIX>(s);
            else ask<1 - MATRIX>(s - kOwn * count(MATRIX));
          }
          if (MATRIX == 1 && n == 1)
#pragma unroll
            for (int k = 0; k < kLds; ++k) lds[j][k] = sh.resident[wave][i][k][lane];
          if (n == 2 && i + kStep < kOwn) {
            c[(step + 1) % 3][j] = cst(1 - MATRIX, i + kStep);
            ready(i + kStep);
          }
        }
#pragma unroll
        for (int j = 0; j < kStep; ++j)
          if (t + j < kOwn) work(t + j, n, c[step % 3][j]);
#pragma unroll
        for (int j = 0; j < kStep; ++j)
          if (t > 0) finish(t - kStep + j, n, c[(step + 2) % 3][j], v[1 - now][j]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    constexpr int kFrom = (kOwn - 1) / kStep * kStep;
#pragma unroll
    for (int i = kFrom; i < kOwn; ++i)
#pragma unroll
      for (int n = 0; n < kBlocks; ++n) finish(i, n, c[kFrom / kStep % 3][i - kFrom], v[kFrom / kStep % 2][i - kFrom]);
  }
  // the same with a matrix in global memory, for the ways in and out
  template <class F>
  __device__ __forceinline__ void sweep_global(const Operand& d, const char* m, bool limbs, const Acc& from, const F& finish) {
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
      __builtin_amdgcn_sched_barrier(0);
      const unsigned l = fresh_place();
      Sums v;
#pragma unroll
      for (int x = 0; x < kHalves; ++x) v.r[x] = from;
#pragma unroll
      for (int k = 0; k < kBlocks; ++k) {
        const Acc f = fragment(m, limbs ? limb_tile(i) : tile(i), k, l);
#pragma unroll
        for (int x = 0; x < kHalves; ++x) v.r[x] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f, d.q[x][k], v.r[x], 0, 0, 0);
      }
      finish(i, v);
    }
  }

  // The residue products of one base of a slot, u v or (SQ) u u: r0 = x0 y0 and r1 = x0 y1 + x1 y0 + e r0, in eight pieces.
  // FOLD: r0 has either one, by its lane.
  template <bool SQ>
  struct Product {
    u32 u0, u1, v0, v1, r0, r1;
    u32 m, f0, f1;
    s64 t, t1;
    __device__ __forceinline__ void step(int n, u32 second, u32 p, u32 pinv, u32 e) {
      if constexpr (FOLD) {
        if (n == 0) {
          f0 = of_first(u0);
          f1 = SQ ? 0u : of_first(v0);
        } else if (n == 1) {
          t = SQ ? smad(f0, u0, 0) : smad(u0 & second, f1, 0);
          if (SQ) asm("" : "+v"(t));  // x1's lanes twice, hidden from the compiler, which would multiply a wider sum of factors
        } else if (n == 2) {
          t = SQ ? smad(f0, u0 & second, t) : smad(f0, v0, t);
        } else if (n == 3) {
          m = (u32)t * pinv;
        } else if (n == 4) {
          f0 = from_first(upper(smad(m, p, t)));
        } else if (n == 5) {
          t = smad(f0, e, t);
        } else if (n == 6) {
          m = (u32)t * pinv;
        } else if (n == 7) {
          r0 = upper(smad(m, p, t));
          r1 = 0;
        }
      } else {
        if (n == 0) {
          t = smad(u0, SQ ? u0 : v0, 0);
        } else if (n == 1) {
          m = (u32)t * pinv;
          t1 = smad(u1, SQ ? u0 : v0, 0);
          if (SQ) asm("" : "+v"(t1));
        } else if (n == 2) {
          r0 = upper(smad(m, p, t));
        } else if (n == 3) {
          t1 = SQ ? smad(u1, u0, t1) : smad(u0, v1, t1);
        } else if (n == 4) {
          t1 = smad(r0, e, t1);
        } else if (n == 5) {
          m = (u32)t1 * pinv;
        } else if (n == 6) {
          r1 = upper(smad(m, p, t1));
        }
      }
    }
    __device__ __forceinline__ void all(u32 second, u32 p, u32 pinv, u32 e) {
#pragma unroll
      for (int n = 0; n < 8; ++n) step(n, second, p, pinv, e);
    }
    static __device__ __forceinline__ u32 upper(s64 v) {
      u32 r = (u32)((u64)v >> 32);
      asm("" : "+v"(r));  // see reduce()
      return r;
    }
  };
  // sigma of the product with y, whose words in base A these are, (SQ: of the square) to the other wavefronts
  template <bool SQ>
  __device__ __forceinline__ void sigma(const State& x, const Words& y) const {
    sigma<SQ>(x, y, [] {});
  }
  // `meanwhile` asks for y's words in base B, in place of those
  template <bool SQ, class F>
  __device__ __forceinline__ void sigma(const State& x, const Words& y_, const F& meanwhile) const {
    const Words y = y_;
    u32 s0[kOwn], s1[kOwn];
    meanwhile();
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
      const Quad k = cst(0, i);
      Product<SQ> r = {x.a0[i], kBoth ? x.a1[i] : 0u, y.w[i][0], y.w[i][1]};
      r.all(second, k[0], k[1], k[2]);
      s0[i] = r.r0;
      s1[i] = r.r1;
      put(0, 0, i, s0);
      if constexpr (kBoth) put(0, 1, i, s1);
    }
  }
  // quad j of this lane's own residues in base B, where the other wavefronts read them
  __device__ __forceinline__ Quad own_b(int x, int j) const { return sh.bytes[1][x][2 * wave + j][lane] ^ rns::kOmega; }
  // all of a value's residues in base B
  __device__ __forceinline__ void get_b(Words& y, const State& x) const {
#pragma unroll
    for (int j = 0; j < (HELD ? 0 : 2); ++j) {
      const Quad q0 = own_b(0, j), q1 = kBoth ? own_b(kHalves - 1, j) : Quad{0, 0, 0, 0};
#pragma unroll
      for (int k = 0; k < 4; ++k) y.w[4 * j + k] = Twin{q0[k], q1[k]};
    }
#pragma unroll
    for (int i = HELD ? 0 : 8; i < kOwn; ++i) y.w[i] = Twin{x.b0[i % kHeldB], kBoth ? x.b1[i % kHeldB] : 0u};
  }
  // what get_b() gives
  __device__ __forceinline__ void set_b(State& x, const Words& y) const {
    if constexpr (!HELD) {
      __syncthreads();  // those of the value before have been read
      put_b(y);
    }
#pragma unroll
    for (int i = HELD ? 0 : 8; i < kOwn; ++i) {
      x.b0[i % kHeldB] = y.w[i][0];
      x.b1[i % kHeldB] = y.w[i][1];
    }
  }
  __device__ __forceinline__ void put_b(const Words& y) const {
#pragma unroll
    for (int h = 0; h < kHalves; ++h) {
      u32 v[kOwn];
#pragma unroll
      for (int i = 0; i < kOwn; ++i) {
        v[i] = y.w[i][h];
        put(1, h, i, v);
      }
    }
  }
  // Base B of the reduced pair from sigma, and to the other wavefronts with alpha's sums. Its products z, w with y, whose words
  // in base B these are, (SQ: with itself) are made on the way.
  template <bool SQ>
  __device__ __forceinline__ void extend_to_b(State& x, const Words& y) {
    __syncthreads();
    Operand d;
    read<false>(d, 0);
    Product<SQ> r[2][kStep];
    Quad own[2][2] = {};  // of tiles 0 to 3 or 4 to 7, and the next ones'
    u32 sum[2] = {}, m, b0[kOwn], b1[kOwn];
    s64 t[2][kStep];
    sweep<0>(
        d,
        [&](int i) {
          if (HELD || i == 8 || i % 4 != 0) return;
          own[i / 4][0] = own_b(0, i / 4);
          if constexpr (kBoth) own[i / 4][1] = own_b(1, i / 4);
        },
        [&](int i, int n, const Quad& k) {
          Product<SQ>& q = r[i / kStep % 2][i % kStep];
          if (n == 0)
            q = Product<SQ>{HELD || i == 8 ? x.b0[i % kHeldB] : own[i / 4 % 2][0][i % 4],
                            !kBoth ? 0u : HELD || i == 8 ? x.b1[i % kHeldB] : own[i / 4 % 2][1][i % 4],
                            y.w[i][0], y.w[i][1]};
          q.step(n, second, k[0], k[1], 0u - k[3]);
        },
        [&](int i, int n, const Quad& k, const Sums& sums) {
          const Product<SQ>& q = r[i / kStep % 2][i % kStep];
          s64 &t0 = t[0][i % kStep], &t1 = t[1][i % kStep];
          const u32 mask = i < 8 ? ~0u : last;
          if (n == 0) {
            t0 = column(sums.r[0]);
          } else if (n == 1) {
            t0 = smad(q.r0, k[2], t0);
          } else if (n == 2) {
            m = (u32)t0 * k[1];
            if constexpr (kBoth) t1 = column(sums.r[kHalves - 1]);
            else t0 = smad(from_first(Product<SQ>::upper(smad(m, k[0], t0))), k[3], t0);
          } else if (n == 3) {
            if constexpr (kBoth) {
              b0[i] = Product<SQ>::upper(smad(m, k[0], t0));
              t1 = smad(q.r1, k[2], t1);
            } else {
              m = (u32)t0 * k[1];
              b0[i] = Product<SQ>::upper(smad(m, k[0], t0));
            }
          } else if (n == 4) {
            if constexpr (kBoth) t1 = smad(b0[i], k[3], t1);
          } else if (n == 5) {
            if constexpr (kBoth) m = (u32)t1 * k[1];
            sum[0] += (u32)((s32)b0[i] >> 16) & mask;
          } else if (n == 6) {
            if constexpr (kBoth) b1[i] = Product<SQ>::upper(smad(m, k[0], t1));
          } else if (n == 7) {
            if constexpr (kBoth) sum[1] += (u32)((s32)b1[i] >> 16) & mask;
            put(1, 0, i, b0);
          } else if (n == 8) {
            if constexpr (kBoth) put(1, 1, i, b1);
            if (HELD || i == 8) {
              x.b0[i % kHeldB] = b0[i];
              if constexpr (kBoth) x.b1[i % kHeldB] = b1[i];
            }
          }
        });
    publish_sums(sum[0], sum[1]);
  }
  __device__ __forceinline__ void publish_sums(u32 s0, u32 s1) {
    u32* s = (u32*)&sh.sum[turn][0][lane & 15] + g;
    atomicAdd(s, s0);
    if (kBoth) atomicAdd(s + 64, s1);
    __syncthreads();
    turn = turn == 2 ? 0 : turn + 1;
    // The sums of the publish_sums() before the last one, which were last read before its barrier, are next added to after the
    // barrier of the one that follows. Every wavefront clears them: a branch would part the loads that are on their way.
#pragma unroll
    for (int x = 0; x < kHalves; ++x) ((u32*)&sh.sum[turn == 2 ? 0 : turn + 1][x][0])[lane] = 0;
  }
  // base B's bytes and alpha's sums to the other wavefronts
  __device__ __forceinline__ void publish(const Words& y) {
    u32 sum[2] = {};
    put_b(y);
#pragma unroll
    for (int i = 0; i < kOwn; ++i)
#pragma unroll
      for (int h = 0; h < kHalves; ++h) sum[h] += (u32)((s32)y.w[i][h] >> 16) & (i < 8 ? ~0u : last);
    publish_sums(sum[0], sum[1]);
  }
  // Base A from what publish() left, NEXT: as sigma of the square, to the other wavefronts
  template <bool NEXT>
  __device__ __forceinline__ void extend_to_a(State& x) {
    Operand d;
    read<true>(d, 1);
    Product<true> r[kStep];
    u32 s0[kOwn], s1[kOwn], m, m1, u0[kStep], u1[kStep];
    s64 t[2][kStep];
    sweep<1>(
        d, [](int) {}, [](int, int, const Quad&) {},
        [&](int i, int n, const Quad& k, const Sums& sums) {
          s64 &t0 = t[0][i % kStep], &t1 = t[1][i % kStep];
          Product<true>& q = r[i % kStep];
          u32 &v0 = u0[i % kStep], &v1 = u1[i % kStep];
          if (n == 0) {
            t0 = column(sums.r[0]);
          } else if (n == 1) {
            m = (u32)t0 * k[1];
            if constexpr (kBoth) t1 = column(sums.r[kHalves - 1]);
            else v0 = Product<true>::upper(smad(m, k[0], t0));
          } else if (n == 2) {
            if constexpr (kBoth) {
              v0 = Product<true>::upper(smad(m, k[0], t0));
              m1 = (u32)t1 * k[1];
              v1 = Product<true>::upper(smad(m1, k[0], t1));
            }
          }
          if constexpr (NEXT) {
            if (n == 2) q = Product<true>{v0, kBoth ? v1 : 0u, 0u, 0u};
            const auto step = [&](int piece) { q.step(piece, second, k[0], k[1], k[2]); };
            if (n == 2) step(0);
            if (n == 3) step(1);
            if (n == 4) step(2);
            if (n == 5) {
              step(3);
              step(4);
            }
            if (n == 6) step(5);
            if (n == 7) {
              step(6);
              step(7);
              s0[i] = q.r0;
              s1[i] = q.r1;
            }
            if (n == 8) {
              put(0, 0, i, s0);
              if constexpr (kBoth) put(0, 1, i, s1);
            }
          } else if (n == 3) {
            x.a0[i] = v0;
            if constexpr (kBoth) x.a1[i] = v1;
          }
        });
  }
  // x times v. `meanwhile` asks for what the next product takes.
  template <bool SQ, class F>
  __device__ __forceinline__ void multiply(State& x, const Quad (&v)[kOwn], const F& meanwhile) {
    Words y;
#pragma unroll
    for (int i = 0; i < kOwn; ++i) y.w[i] = Twin{v[i][0], v[i][1]};
    sigma<SQ>(x, y);
#pragma unroll
    for (int i = 0; i < kOwn; ++i) y.w[i] = Twin{v[i][2], v[i][3]};
    extend_to_b<SQ>(x, y);
    meanwhile();
    extend_to_a<false>(x);
  }
  // the pairs whose limbs are at `src` (`left` of them, then zeros) into both bases
  __device__ __forceinline__ void load(State& x, const u32* src, unsigned left, int nl) {
    const int e = lane & (kElements - 1), half = FOLD ? lane >> 3 & 1 : 0;
    __syncthreads();  // the bytes of the elements before have been read
    for (int i = wave; i < kRegs; i += kWaves) {
      const int l = 4 * i + g;
      if (l == rns::bias_slot(kRegs)) continue;
      const bool ok = (unsigned)e < left && l < nl;
      const u32* p = src + (size_t)e * (2 * nl) + half * nl + l;
      word(0, 0, i, lane) = (ok ? p[0] : 0u) ^ rns::kOmega;
      if constexpr (kBoth) word(0, 1, i, lane) = (ok ? p[nl] : 0u) ^ rns::kOmega;
    }
    __syncthreads();
    Operand d;
    read<false>(d, 0);
    Words y;
    sweep_global(d, tables + rns::lds_bytes(kRegs), false, start, [&](int i, const Sums& v) {
      const Quad k = cst(1, i);
      y.w[i] = Twin{reduce(column(v.r[0]), k[0], k[1]), kBoth ? reduce(column(v.r[kHalves - 1]), k[0], k[1]) : 0u};
      if (HELD || i == 8) {
        x.b0[i % kHeldB] = y.w[i][0];
        x.b1[i % kHeldB] = y.w[i][1];
      }
    });
#pragma unroll
    for (int s = 0; s < RING; ++s) ask<1>(s);
    publish(y);
    extend_to_a<false>(x);
  }
  // the pairs as two integers each in columns of weight 2^(29 l)
  __device__ __forceinline__ void store(const State& x, long long* dst, unsigned left) {
    const unsigned e = (unsigned)(lane & (kElements - 1));
    store(x, dst, e, e < left);
  }
  // the same, this lane's to element `e` behind `dst`
  template <class I>
  __device__ __forceinline__ void store(const State& x, long long* dst, I e, bool active) {
    Words y;
    get_b(y, x);
    __syncthreads();  // the bytes of the last product have been read
    publish(y);
    Operand d;
    read<true>(d, 1);
    const unsigned half = FOLD ? (unsigned)lane >> 3 & 1 : 0;
    long long* to = dst + (size_t)e * (8 * kLimbTiles) + half * (4 * kLimbTiles) + g;
    sweep_global(d, tables + rns::lds_bytes(kRegs) + rns::in_matrix_bytes(kRegs), true, Acc{0, 0, 0, 0}, [&](int i, const Sums& v) {
      if (active) {
        to[4 * limb_tile(i)] = integer(v.r[0]);
        if constexpr (kBoth) to[4 * kLimbTiles + 4 * limb_tile(i)] = integer(v.r[kHalves - 1]);
      }
    });
  }
  // Window tables: [base][wavefront, tile][lane] words of x0 and x1
  static constexpr int kEntry = 2 * kLimbTiles * WAVE * kHalves;  // dwords
  __device__ __forceinline__ u32* entry_at(const u32* entry, int base, int i) const {
    return (u32*)entry + (base * kLimbTiles * WAVE + (kOwn * wave + i) * WAVE + lane) * kHalves;
  }
  static __device__ __forceinline__ Quad own(const State& x, int i) {
    return Quad{x.a0[i], kBoth ? x.a1[i] : 0u, x.b0[i % kHeldB], kBoth ? x.b1[i % kHeldB] : 0u};
  }
  __device__ __forceinline__ void load_entry(Words& y, const u32* entry, int base) const {
#pragma unroll
    for (int i = 0; i < kOwn; ++i)
      if constexpr (kBoth) y.w[i] = *(const Twin*)entry_at(entry, base, i);
      else y.w[i] = Twin{*entry_at(entry, base, i), 0};
  }
  // The same of an element in memory by itself (see item_words): quad j of this lane's half (kBoth: of half x) in a base
  __device__ __forceinline__ int item_quad(int base, int x, int j) const {
    const int half = kBoth ? x : lane >> 3 & 1;
    return base * (rns::item_words(kRegs) / 2) + ((2 * (j < 2 ? 2 * wave + j : 8) + half) * 4 + g) * 4;
  }
  __device__ __forceinline__ void load_item(Words& y, const u32* item, int base) const {
#pragma unroll
    for (int x = 0; x < kHalves; ++x) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const Quad q = *(const Quad*)(item + item_quad(base, x, j));
#pragma unroll
        for (int c = 0; c < 4; ++c) y.w[4 * j + c][x] = q[c];
      }
      y.w[8][x] = item[item_quad(base, x, 2) + tile(8) % 4];
    }
    if (!kBoth)
#pragma unroll
      for (int i = 0; i < kOwn; ++i) y.w[i][1] = 0;
  }
  __device__ __forceinline__ void load_item(Quad (&v)[kOwn], const u32* item) const {
    Words a, b;
    load_item(a, item, 0);
    load_item(b, item, 1);
#pragma unroll
    for (int i = 0; i < kOwn; ++i) v[i] = Quad{a.w[i][0], a.w[i][1], b.w[i][0], b.w[i][1]};
  }
  __device__ __forceinline__ void store_item(const State& x, u32* item) const {
    Words y[2];
#pragma unroll
    for (int i = 0; i < kOwn; ++i) y[0].w[i] = Twin{x.a0[i], kBoth ? x.a1[i] : 0u};
    get_b(y[1], x);
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int h = 0; h < kHalves; ++h) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
          *(Quad*)(item + item_quad(b, h, j)) = Quad{y[b].w[4 * j][h], y[b].w[4 * j + 1][h], y[b].w[4 * j + 2][h], y[b].w[4 * j + 3][h]};
        if (mine(8)) item[item_quad(b, h, 2) + wave] = y[b].w[8][h];
      }
  }
  __device__ __forceinline__ void set(State& x, const Quad (&v)[kOwn]) const {
    Words y[2];
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
      y[0].w[i] = Twin{v[i][0], v[i][1]};
      y[1].w[i] = Twin{v[i][2], v[i][3]};
    }
    set_a(x, y[0]);
    set_b(x, y[1]);
  }
  static __device__ __forceinline__ void set_a(State& x, const Words& y) {
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
      x.a0[i] = y.w[i][0];
      x.a1[i] = y.w[i][1];
    }
  }
  __device__ __forceinline__ void store_state(const State& x, u32* entry) const {
    Words y;
    get_b(y, x);
#pragma unroll
    for (int i = 0; i < kOwn; ++i)
      if constexpr (kBoth) {
        *(Twin*)entry_at(entry, 0, i) = Twin{x.a0[i], x.a1[i]};
        *(Twin*)entry_at(entry, 1, i) = y.w[i];
      } else {
        *entry_at(entry, 0, i) = x.a0[i];
        *entry_at(entry, 1, i) = y.w[i][0];
      }
  }
  __device__ __forceinline__ void load_state(State& x, const u32* entry) const {
    Words y;
    load_entry(y, entry, 0);
    set_a(x, y);
    load_entry(y, entry, 1);
    set_b(x, y);
  }
};

// Instruction pc of the program `prog` of `len`, asked for one after the other. A wavefront keeps 64 of them at a time in the
// lanes of `words`: read from memory between two products, one costs a wavefront that waits for little else 2 to 5 % of a
// product. PIN: they are waited for where they are read, not where the ways join, which would wait for all loads at each instruction;
// only k_rns_wide has loads on their way there (k_rns_group with it: 64 decryptions at a 4096-bit key 2.169 -> 2.184 ms).
// A macro: as a function's argument the program's place in the launch's arguments would cost a copy of them.
#define INSTRUCTION(ins, prog, len, pc, words, PIN)                           \
  do {                                                                        \
    if ((pc & (WAVE - 1)) == 0) {                                             \
      const int at = pc + (int)(threadIdx.x & (WAVE - 1));                    \
      words = prog[at < len ? at : len - 1];                                  \
      if constexpr (PIN) asm volatile("" : "+v"(words));                      \
    }                                                                         \
    ins = (u32)__builtin_amdgcn_readlane((int)words, pc & (WAVE - 1));        \
  } while (0)

// Every block runs the program on 16 (FOLD: 8) elements at a time. The first `split` blocks run j0, the others j1.
// W wavefronts with TW tiles each, then W1 with TW1: the tiles over the four SIMDs as evenly as they go. The single form of
// 1024-bit moduli is held to 80 registers, with which two blocks share a compute unit, up to six wavefronts to a SIMD: with 88,
// five, the second one waits (the key owner's first stage of 3000 encryptions at a 2048-bit key 1.25 instead of 0.8 ms).
template <int NR, int TW, int W, int TW1, int W1, bool PAIR, bool FOLD>
__global__ __launch_bounds__((W + W1) * 64, NR == 10 && !PAIR ? 6 : (W + W1 + 3) / 4) void k_rns_group(RnsJob j0, RnsJob j1, unsigned split, size_t count) {
  using Main = RnsGroup<NR, TW, W + W1, W * TW + W1 * TW1, PAIR, FOLD>;
  using Rest = RnsGroup<NR, TW1, W + W1, W * TW + W1 * TW1, PAIR, FOLD>;
  __shared__ __align__(16) typename Main::Shared shared;
  const bool second = blockIdx.x >= split;
  const RnsJob& j = second ? j1 : j0;
  const unsigned block = second ? blockIdx.x - split : blockIdx.x;
  const unsigned nblocks = second ? gridDim.x - split : split;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
  const u32* prog = j.prog ? j.prog : j.ins;
  const int len = __builtin_amdgcn_readfirstlane(j.len);
  u32* table = j.slots + (size_t)block * (size_t)j.entries * Main::kEntry;
// in the kernel itself: as a function's argument the program's place in the launch's arguments would cost a copy of them
#define RUN(G, FIRST_TILE)                                                                                          \
  do {                                                                                                              \
    G e(shared, j.tables, FIRST_TILE);                                                                              \
    for (size_t first = (size_t)block * G::kElements; first < count; first += (size_t)nblocks * G::kElements) {    \
      const unsigned left = (unsigned)std::min(count - first, (size_t)G::kElements);                               \
      typename G::State x;                                                                                          \
      e.load(x, j.in + first * (size_t)(2 * j.nl), left, j.nl);                                                     \
      u32 words = 0;                                                                                                \
      for (int pc = 0; pc < len;) {                                                                                 \
        u32 ins;                                                                                                    \
        INSTRUCTION(ins, prog, len, pc, words, false);                                                              \
        _Pragma("unroll 1") while (ins == ENG_SQ) {                                                                 \
          e.template multiply<true>(x, nullptr);                                                                    \
          ins = ~0u;                                                                                                \
          if (++pc < len) INSTRUCTION(ins, prog, len, pc, words, false);                                            \
        }                                                                                                           \
        if (pc++ >= len) break;                                                                                     \
        const u32 op = ins & 0xFFu, a = (ins >> 8) & 0xFFFu, b = ins >> 20;                                         \
        u32* entry = table + (size_t)a * G::kEntry;                                                                 \
        if (op == ENG_STORE_T) {                                                                                    \
          e.store_state(x, entry);                                                                                  \
        } else if (op == ENG_LOAD_T) {                                                                              \
          e.load_state(x, entry);                                                                                   \
        } else {                                                                                                    \
          e.template multiply<false>(x, entry);                                                                     \
          if (op == ENG_MUL_T_ST) e.store_state(x, table + (size_t)b * G::kEntry);                                  \
        }                                                                                                           \
      }                                                                                                             \
      e.store(x, j.out + first * (size_t)(8 * G::kLimbTiles), left);                                                \
    }                                                                                                               \
  } while (0)
  if (W1 == 0 || wave < W) {
    RUN(Main, wave * TW);
  } else if constexpr (W1 > 0) {
    // As many barriers as above, though elsewhere in the code: their number follows from the program and the count of
    // elements, which all wavefronts share, and a barrier counts wavefronts wherever they wait for it.
    RUN(Rest, W * TW + (wave - W) * TW1);
  }
#undef RUN
}

// The same for 4096-bit moduli. How many blocks stream, and how many of them are on their way, by what fits the registers: with one
// block less, or more on their way, the paths around the run of squarings spill (3001 encryptions 18.8 ms with three on their way, 19.9
// with six, 22.4 with nine; 64 of them 12.6 with six and 13.7 with nine). The ways through the lists' two values and an operand leave
// room for the residues of base B as registers.
template <bool FOLD>
struct Wide;
template <>
struct Wide<true> {
  using Power = RnsWide<true, 4, 4, 6, false>;
  using Chains = RnsWide<true, 4, 4, 6, false>;
  using Lists = RnsWide<true, 4, 4, 6, true>;
};
template <>
struct Wide<false> {
  using Power = RnsWide<false, 4, 4, 3, false>;
  using Chains = RnsWide<false, 4, 4, 6, false>;
};
template <bool FOLD>
__global__ __launch_bounds__(256, 1) void k_rns_wide(RnsJob j, size_t count) {
  using G = typename Wide<FOLD>::Power;
  __shared__ __align__(16) typename G::Shared shared;
  const u32* prog = j.prog ? j.prog : j.ins;
  const int len = __builtin_amdgcn_readfirstlane(j.len);
  u32* table = j.slots + (size_t)blockIdx.x * (size_t)j.entries * G::kEntry;
  G e(shared, j.tables);
  for (size_t first = (size_t)blockIdx.x * G::kElements; first < count; first += (size_t)gridDim.x * G::kElements) {
    const unsigned left = (unsigned)std::min(count - first, (size_t)G::kElements);
    typename G::State x;
    e.load(x, j.in + first * (size_t)(2 * j.nl), left, j.nl);
    u32 words = 0;
    for (int pc = 0; pc < len;) {
      u32 ins;
      INSTRUCTION(ins, prog, len, pc, words, true);
      ++pc;
      const u32 op = ins & 0xFFu, a = (ins >> 8) & 0xFFFu, b = ins >> 20;
      u32* entry = table + (size_t)a * G::kEntry;
      if (op == ENG_STORE_T) {
        e.store_state(x, entry);
        continue;
      }
      if (op == ENG_LOAD_T) {
        e.load_state(x, entry);
        continue;
      }
      typename G::Words y = {};
      if (op == ENG_SQ) {  // a run of them, each but the last with the next one's sigma
        e.template sigma<true>(x, y);
        for (;;) {
          e.template extend_to_b<true>(x, y);
          if (pc >= len) break;
          INSTRUCTION(ins, prog, len, pc, words, true);
          if (ins != ENG_SQ) break;
          ++pc;
          e.template extend_to_a<true>(x);
        }
      } else {
        e.load_entry(y, entry, 0);
        e.template sigma<false>(x, y);
        e.load_entry(y, entry, 1);
        e.template extend_to_b<false>(x, y);
      }
      e.template extend_to_a<false>(x);
      if (op == ENG_MUL_T_ST) e.store_state(x, table + (size_t)b * G::kEntry);
    }
    e.store(x, j.out + first * (size_t)(8 * G::kLimbTiles), left);
  }
}

// RnsLists' program on 8 elements at a time, for what is few and has long chains. All wavefronts take the same way through
// it: each knows every element's operands, whose places lie in LDS. An operand is on its way one product ahead. What bounds
// it is a product's chain from barrier to barrier, 1 to 1.5 us at 2048 bits; a wavefront to a pair on limbs takes 8.
struct ListShared {
  u32 place[kListRows][16];
};
template <class G>
__device__ __forceinline__ void run_lists(G& e, const RnsLists& j, ListShared& sh, u32 ops) {
  // scalars, all of them: the way through the program is the same for all lanes
  const unsigned count = j.live ? (unsigned)__builtin_amdgcn_readfirstlane((int)*j.live) : (unsigned)j.stride;
  const int limit = j.limit ? __builtin_amdgcn_readfirstlane((int)*j.limit) : kListOps;
  const int len = j.len < limit ? j.len : limit;
  e.begin();
  for (unsigned first = blockIdx.x * G::kElements; first < count; first += gridDim.x * G::kElements) {
    const unsigned left = std::min(count - first, (unsigned)G::kElements);
    const unsigned own = (unsigned)(e.lane & (G::kElements - 1));
    __syncthreads();  // the places before have been read
    for (int i = (int)threadIdx.x; i < j.rows * G::kElements; i += (int)blockDim.x) {
      const unsigned r = (unsigned)i / G::kElements, l = (unsigned)i % G::kElements;
      sh.place[r][l] = l < left ? j.operands[r * j.stride + first + l] : kNoOperand;
    }
    __syncthreads();
    int row = 0;
    const auto next_place = [&]() { return sh.place[row < j.rows ? row : j.rows - 1][own]; };
    // A program without operands, as those that make the element `one`, asks for constants in their place, and uses none.
    const u32* none = j.rows ? j.one : j.tables;
    const auto item = [&](u32 p) { return p == kNoOperand ? none : j.items + (size_t)p * rns::item_words(G::kRegs); };
    const u32* place = j.places + first;
    typename G::State run = {}, acc = {};
    bool run_one = true, acc_one = true;  // known to be one in all elements
    Quad next[G::kOwn];
    u32 p = j.rows ? next_place() : kNoOperand;
    e.load_item(next, item(p));
#pragma unroll 1
    for (int pc = 0; pc < len; ++pc) {
      const u32 op = (u32)__builtin_amdgcn_readlane((int)ops, pc / 8) >> pc % 8 * 4 & 15u;
      const bool on_run = op == LIST_RUN_ITEM || op == LIST_STORE_RUN;
      typename G::State x = on_run ? run : acc;
      const bool x_one = on_run ? run_one : acc_one;
      if (op <= LIST_ACC_SQ) {
        const bool from_item = op <= LIST_ACC_ITEM;
        Quad y[G::kOwn];
        bool y_one = op == LIST_ACC_RUN ? run_one : acc_one;
        if (from_item) {
          y_one = __builtin_amdgcn_ballot_w64(p != kNoOperand) == 0;
          ++row;
          p = next_place();
        }
#pragma unroll
        for (int i = 0; i < G::kOwn; ++i) {
          const Quad o = e.own(op == LIST_ACC_RUN ? run : acc, i);
          y[i] = from_item ? next[i] : o;
        }
        if (y_one || x_one) {
          e.load_item(next, item(p));
          if (y_one) continue;
          e.set(x, y);
        } else {
          e.template multiply<false>(x, y, [&] { e.load_item(next, item(p)); });
        }
        if (on_run) {
          run = x;
          run_one = false;
        } else {
          acc = x;
          acc_one = false;
        }
        continue;
      }
      if (op == LIST_ACC_LIMBS) {
        e.load(acc, j.limbs + (size_t)first * (2 * j.nl), left, j.nl);
        acc_one = false;
        continue;
      }
      if (x_one) {
        Quad one[G::kOwn];
        e.load_item(one, j.one);
        e.set(x, one);
      }
      if (op == LIST_COLUMNS) {
        e.store(x, j.columns + first * (size_t)(8 * G::kLimbTiles), left);
      } else {
        if (own < left) e.store_item(x, j.out + (size_t)(j.places ? place[own] : first + own) * rns::item_words(G::kRegs));
        place += j.stride;
      }
    }
  }
}
template <int NR, int TW, int W, int TW1, int W1>
__global__ __launch_bounds__((W + W1) * 64, (W + W1 + 3) / 4) void k_rns_lists(RnsLists j) {
  using Main = RnsGroup<NR, TW, W + W1, W * TW + W1 * TW1, true, true, true>;
  using Rest = RnsGroup<NR, TW1, W + W1, W * TW + W1 * TW1, true, true, true>;
  __shared__ __align__(16) typename Main::Shared shared;
  __shared__ ListShared lists;
  if (j.live && (size_t)blockIdx.x * Main::kElements >= *j.live) return;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
  u32 ops = 0;  // in the lanes of a register, as an index that varies would cost a copy of the arguments
#pragma unroll
  for (int i = 0; i < kListOps / 8; ++i) ops = (threadIdx.x & (WAVE - 1)) == i ? j.ops[i] : ops;
  if (W1 == 0 || wave < W) {
    Main e(shared, j.tables, wave * TW);
    run_lists(e, j, lists, ops);
  } else if constexpr (W1 > 0) {  // as many barriers, see k_rns_group
    Rest e(shared, j.tables, W * TW + (wave - W) * TW1);
    run_lists(e, j, lists, ops);
  }
}

__global__ __launch_bounds__(256, 1) void k_rns_wide_lists(RnsLists j) {
  using G = Wide<true>::Lists;
  __shared__ __align__(16) typename G::Shared shared;
  __shared__ ListShared lists;
  if (j.live && (size_t)blockIdx.x * G::kElements >= *j.live) return;
  u32 ops = 0;
#pragma unroll
  for (int i = 0; i < kListOps / 8; ++i) ops = (threadIdx.x & (WAVE - 1)) == i ? j.ops[i] : ops;
  G e(shared, j.tables);
  run_lists(e, j, lists, ops);
}

// k_rns_enter for 4096-bit moduli, on blocks of 16 elements. What bounds it are the matrices of the way in and of the way back, which
// stream from L2 for 16 elements at a time, those of the way in tile after tile: 20000 elements 86 us, 65536 233 to 243 (205 on blocks
// of twelve wavefronts, the form before).
__global__ __launch_bounds__(256, 1) void k_rns_wide_enter(const u32* __restrict__ tables, const u32* __restrict__ in,
                                                           size_t count, int nl, u32* __restrict__ items) {
  using G = Wide<false>::Chains;
  __shared__ __align__(16) typename G::Shared shared;
  G e(shared, tables);
  for (size_t first = (size_t)blockIdx.x * G::kElements; first < count; first += (size_t)gridDim.x * G::kElements) {
    const unsigned left = (unsigned)std::min(count - first, (size_t)G::kElements), own = (unsigned)(e.lane & (G::kElements - 1));
    typename G::State x;
    e.load(x, in + first * (size_t)(2 * nl), left, nl);
    if (own < left) e.store_item(x, items + (first + own) * (size_t)rns::item_words(G::kRegs));
  }
}

// RnsChains on blocks of 8 elements, as k_rns_chains does on wavefronts of 16
template <class G>
__device__ __forceinline__ void run_chains(G& e, const RnsChains& j, unsigned total) {
  const bool columns = __builtin_amdgcn_readfirstlane((int)j.control[kChainsColumns]) != 0;
  for (unsigned first = blockIdx.x * G::kElements; first < total; first += gridDim.x * G::kElements) {
    const unsigned own = first + (unsigned)(e.lane & (G::kElements - 1));
    const bool active = own < total;
    const Quad c = active ? ((const Quad*)j.chains)[own] : Quad{0, 0, 0, 0};
    const u32 start = c[1], len = c[2];
    const u32 longest = (u32)__builtin_amdgcn_readfirstlane((int)wave_max(len));  // each wavefront has all elements
    const auto place = [&](u32 i) -> u32 { return i < len ? j.index ? j.index[start + i] : start + i : kNoOperand; };
    const auto item = [&](u32 p) { return p == kNoOperand ? j.one : j.items + (size_t)p * rns::item_words(G::kRegs); };
    Quad next[G::kOwn];
    typename G::State x;
    e.load_item(next, item(place(0)));
    e.set(x, next);
    e.load_item(next, item(place(1)));
    u32 p = place(2);
#pragma unroll 1
    for (u32 i = 1; i < longest; ++i) {
      Quad y[G::kOwn];
#pragma unroll
      for (int t = 0; t < G::kOwn; ++t) y[t] = next[t];
      e.template multiply<false>(x, y, [&] {
        e.load_item(next, item(p));
        p = place(i + 2);
      });
    }
    if (columns) e.store(x, j.columns, (size_t)c[0], active);
    else if (active) e.store_item(x, j.out + (size_t)c[0] * rns::item_words(G::kRegs));
  }
}
template <int NR, int TW, int W, int TW1, int W1>
__global__ __launch_bounds__((W + W1) * 64, (W + W1 + 3) / 4) void k_rns_group_chains(RnsChains j) {
  using Main = RnsGroup<NR, TW, W + W1, W * TW + W1 * TW1, true, true, true>;
  using Rest = RnsGroup<NR, TW1, W + W1, W * TW + W1 * TW1, true, true, true>;
  __shared__ __align__(16) typename Main::Shared shared;
  const unsigned total = (unsigned)__builtin_amdgcn_readfirstlane((int)j.control[kChainsTotal]);
  if (blockIdx.x * Main::kElements >= total) return;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
  if (W1 == 0 || wave < W) {
    Main e(shared, j.tables, wave * TW);
    run_chains(e, j, total);
  } else if constexpr (W1 > 0) {  // as many barriers, see k_rns_group
    Rest e(shared, j.tables, W * TW + (wave - W) * TW1);
    run_chains(e, j, total);
  }
}

template <bool FOLD>
__global__ __launch_bounds__(256, 1) void k_rns_wide_chains(RnsChains j) {
  using G = typename Wide<FOLD>::Chains;
  __shared__ __align__(16) typename G::Shared shared;
  const unsigned total = (unsigned)__builtin_amdgcn_readfirstlane((int)j.control[kChainsTotal]);
  if (blockIdx.x * G::kElements >= total) return;
  G e(shared, j.tables);
  const bool columns = __builtin_amdgcn_readfirstlane((int)j.control[kChainsColumns]) != 0;
  e.begin();
  // as run_chains(), with a factor's words of one base after those of the other
  for (unsigned first = blockIdx.x * G::kElements; first < total; first += gridDim.x * G::kElements) {
    const unsigned own = first + (unsigned)(e.lane & (G::kElements - 1));
    const bool active = own < total;
    const Quad c = active ? ((const Quad*)j.chains)[own] : Quad{0, 0, 0, 0};
    const u32 start = c[1], len = c[2];
    const u32 longest = (u32)__builtin_amdgcn_readfirstlane((int)wave_max(len));  // each wavefront has all elements
    const auto place = [&](u32 i) -> u32 { return i < len ? j.index ? j.index[start + i] : start + i : kNoOperand; };
    const auto item = [&](u32 p) { return p == kNoOperand ? j.one : j.items + (size_t)p * rns::item_words(G::kRegs); };
    typename G::State x;
    typename G::Words y;
    const u32* from = item(place(0));
    e.load_item(y, from, 0);
    e.set_a(x, y);
    e.load_item(y, from, 1);
    e.set_b(x, y);
    from = item(place(1));
    e.load_item(y, from, 0);
    u32 p = place(2);
#pragma unroll 1
    for (u32 i = 1; i < longest; ++i) {
      e.template sigma<false>(x, y, [&] { e.load_item(y, from, 1); });
      e.template extend_to_b<false>(x, y);
      from = item(p);
      e.load_item(y, from, 0);
      p = place(i + 2);
      e.template extend_to_a<false>(x);
    }
    if (columns) e.store(x, j.columns, (size_t)c[0], active);
    else if (active) e.store_item(x, j.out + (size_t)c[0] * rns::item_words(G::kRegs));
  }
}

}  // namespace

namespace haflo {

constexpr int kRnsElementsPerCu = 256;  // in flight at once

namespace {
// The blocks of k_rns_group that are resident at once on a compute unit
int group_blocks_per_cu(int nr) { return nr <= 10 ? 2 : 1; }
// Blocks of 8 elements, while each has a compute unit to itself. ms with 16 / 8 to a block, up to the line: 2048 encryptions at
// a 1024-bit key 0.97 / 0.74, at 2048 bits 3.40 / 2.21, at 4096 bits 18.6 / 14.6 (100 of them 18.3 / 12.6); 1024 decryptions at
// 1024 bits 0.399 / 0.354, at 2048 bits 1.03 / 0.79, at 4096 bits 3.47 / 2.30. Beyond it, with two blocks of 8 and more to a
// compute unit: encryptions at 1024 bits 0.97 / 1.40 (2049), 0.99 / 1.43 (4096), 1.92 / 2.12 (6144), at 2048 bits 3.40 / 4.32
// (2049), 3.49 / 4.23 (4096), at 4096 bits 18.6 / 28.4 (2049); decryptions at 2048 bits 1.03 / 1.46 (1025), at 4096 bits 3.50 /
// 4.44. The short products of 256-bit primes are 2 to 3 % faster there with two blocks to a compute unit, but not with three:
// 0.400 / 0.388 (1025 decryptions at a 1024-bit key), 0.402 / 0.395 (2048), 0.473 / 0.723 (2500), 0.475 / 0.726 (3072).
bool group_folds(const haflo_ctx* ctx, size_t count, int jobs, bool pair) {
  return pair && (count + 7) / 8 * (size_t)jobs <= (size_t)ctx->num_cu;
}
size_t group_blocks(const haflo_ctx* ctx, int nr, size_t count, int jobs, bool fold) {
  const size_t all = fold ? (count + 7) / 8 : (count + 15) / 16;
  return std::min(all, std::max((size_t)ctx->num_cu * group_blocks_per_cu(nr) / (size_t)jobs, (size_t)1));
}
// Where the elements are few, or the matrices too large for the LDS, the slots of 16 elements are spread over a block.
// Measured on both sides (ms, spread / not): encryption at a 512-bit key 0.45 / 0.71 at 8192 elements, 0.73 / 0.72 at 9216; at
// 1024 bits 1.00 / 2.31 at 4096, 1.95 / 2.37 at 8192, 2.84 / 2.40 at 8193; at 2048 bits 7.4 / 17.1 at 8192, 21.5 / 24.0 at 24576,
// 24.6 / 23.9 at 24577, 24.8 / 25.4 at 28672 (seven full passes), 28.1 / 27.1 at 32768; decryption at a 1024-bit key 0.48 / 0.74 at
// 4096, 0.88 / 0.75 at 4097, at 2048 bits 2.00 / 2.42 and 2.91 / 2.44, at 4096 bits 21.4 / 24.2 at 12288, 24.9 / 24.3 at 12289, 28.3 /
// 27.5 at 16384. The key owner's encryption, whose first stage is of the single form: at a 1024-bit key 0.79 / 1.23 at 4096, 1.47 /
// 1.25 at 4097, at 2048 bits 2.80 / 4.00 and 4.45 / 4.06, at 4096 bits 32.6 / 35.7 at 12288, 38.0 / 35.5 at 12289.
bool use_group(const haflo_ctx* ctx, int nr, size_t count, int jobs) {
  return nr == 36 || (count + 15) / 16 * (size_t)jobs <= (size_t)ctx->num_cu * (nr == 18 ? 6 : 2);
}
// Sets of 16 elements per wavefront of k_rns. A SIMD's time follows from its wavefronts: with one set each 2.5, 4.0 and
// 6.1 ms for one, two and three of them (encryption at a 1024-bit key, 16384, 30000 and 40000 elements), with two sets 3.75
// and 7.5 - 8.4. So one set where its wavefronts are one or three to a SIMD (40000 elements 6.1 / 7.5 ms; 30000, two to a
// SIMD, 4.18 / 4.08; 65536, four, 9.3 / 8.4); the short products of 256-bit primes' pairs with two to a SIMD as well
// (12288 decryptions at a 1024-bit key 1.05 / 1.13). For pairs of 2048-bit halves one, which k_rns_one has; for single residues
// of 2048 bits two, one was not measured.
int rns_sets(const haflo_ctx* ctx, int nr, size_t count, int jobs, bool pair) {
  if (nr == 18) return pair ? 1 : 2;
  const size_t per_simd = ((count + 15) / 16 * (size_t)jobs + 4 * ctx->num_cu - 1) / (4 * (size_t)ctx->num_cu);
  return per_simd == 1 || per_simd == 3 || (nr == 6 && per_simd == 2) ? 1 : 2;
}
// Window tables of one modulus, each of 16 elements: one per block, or as many as the wavefronts that have elements hold
size_t table_slots(const haflo_ctx* ctx, int nr, size_t count, int jobs) {
  if (!use_group(ctx, nr, count, jobs)) return (count + 31) / 32 * 2;
  // Few enough for blocks of 8: one for two such blocks, and for a block of 16 of the single form, which none of the limits of
  // group_blocks cuts short at these counts. So the number does not depend on the form.
  if (group_folds(ctx, count, jobs, true)) return (count + 15) / 16;
  return group_blocks(ctx, nr, count, jobs, false);
}
}  // namespace

size_t rns_chunk(const haflo_ctx* ctx, int jobs) {
  return std::max((size_t)ctx->num_cu * kRnsElementsPerCu / 32 / (size_t)jobs, (size_t)1) * 32;
}
int rns_columns(const ModHost& m) { return 4 * rns::limb_tiles(rns::regs_for(m.nl)); }

RnsBuffers rns_buffers(const haflo_ctx* ctx, const ModHost& m, size_t count, int jobs, int entries) {
  const int nr = rns::regs_for(m.nl);
  const size_t n = std::min(count, rns_chunk(ctx, jobs));
  RnsBuffers b = {};
  size_t at = 0;
  for (int i = 0; i < jobs; ++i) {
    b.out[i] = at;  // 8-byte columns first
    at += n * 2 * 2 * (size_t)rns_columns(m);
  }
  for (int i = 0; i < jobs; ++i) {
    b.in[i] = at;
    at += (n * 2 * (size_t)m.nl + 3) & ~(size_t)3;
  }
  b.tables = at;  // 16 bytes aligned
  // the pair engine's slots before and after lie here too: as many as there are elements, 2 nl words each
  b.total = at + std::max((size_t)jobs * table_slots(ctx, nr, n, jobs) * (size_t)entries * 4 * (size_t)nr * 64,
                          (size_t)jobs * (n + 128) * 2 * (size_t)m.nl);
  return b;
}

size_t rns_item_words(const ModHost& m) { return (size_t)rns::item_words(rns::regs_for(m.nl)); }

namespace {
// One block per compute unit, with as many wavefronts, `most` of them, as spread `count` elements over all of them
LaunchShape rns_shape(const haflo_ctx* ctx, size_t count, size_t most) {
  const size_t tiles = std::max((count + 15) / 16, (size_t)1);
  const size_t waves = std::min((tiles + ctx->num_cu - 1) / ctx->num_cu, most);
  LaunchShape sh;
  sh.threads = (int)waves * WAVE;
  sh.gpb = (int)waves * 16;
  sh.blocks = (int)std::min((tiles + waves - 1) / waves, (size_t)ctx->num_cu);
  return sh;
}
}  // namespace

int rns_enter(const haflo_ctx* ctx, const ModHost& m, const uint32_t* in, size_t count, uint32_t* items, hipStream_t st) {
  if (rns::regs_for(m.nl) == 18) {
    HAFLO_LAUNCH((k_rns_enter<18>), rns_shape(ctx, count, 16), st, (const u32*)m.d_rns, in, count, m.nl, items);
    return hip_status(hipGetLastError());
  }
  if (rns::regs_for(m.nl) != 36) return HAFLO_EINVAL;
  const unsigned blocks = (unsigned)std::max(group_blocks(ctx, 36, count, 1, false), (size_t)1);
  hipLaunchKernelGGL(k_rns_wide_enter, dim3(blocks), dim3(256), 0, st, (const u32*)m.d_rns, in, count, m.nl, items);
  return hip_status(hipGetLastError());
}

int rns_lists(const haflo_ctx* ctx, const ModHost& m, RnsLists j, size_t bound, hipStream_t st) {
  const int nr = rns::regs_for(m.nl);
  // always 8 elements to a block: with 16 the matrices, two values and an operand on its way do not fit the registers (26
  // spilled; 12288 sub-products' shares of 8 factors 160 us, 120 so)
  const unsigned blocks = (unsigned)std::max(group_blocks(ctx, nr, bound, 1, true), (size_t)1);
  j.tables = m.d_rns;
  j.nl = m.nl;
  switch (nr) {
    case 18: hipLaunchKernelGGL((k_rns_lists<18, 2, 8, 1, 2>), dim3(blocks), dim3(640), 0, st, j); break;
    case 36: hipLaunchKernelGGL(k_rns_wide_lists, dim3(blocks), dim3(256), 0, st, j); break;
    default: return HAFLO_EINVAL;
  }
  return hip_status(hipGetLastError());
}

int rns_chains(const haflo_ctx* ctx, const ModHost& m, RnsChains j, size_t bound, size_t expected, hipStream_t st) {
  const int nr = rns::regs_for(m.nl);
  j.tables = m.d_rns;
  // Wavefronts of 16 elements once there are 32 to a compute unit, else blocks of 8 elements, whose products take less time on
  // their own. ms with wavefronts / blocks: forward 1000 by 64 (8000 chains) 0.57 / 0.53, 16384 by 8 (16384 of some five factors)
  // 0.57 / 0.53; gradient 4096 by 16 (8192) 0.795 / 0.798, 16384 by 8 (16384 of 16 factors) 0.82 / 0.87.
  if (nr == 18 && expected > (size_t)ctx->num_cu * 32) {
    HAFLO_LAUNCH((k_rns_chains<18>), rns_shape(ctx, bound, 12), st, j);
    return hip_status(hipGetLastError());
  }
  const bool fold = nr == 18 || expected <= (size_t)ctx->num_cu * 8 * group_blocks_per_cu(nr);
  const unsigned blocks = (unsigned)std::max(group_blocks(ctx, nr, bound, 1, fold), (size_t)1);
  switch (nr) {
    case 18: hipLaunchKernelGGL((k_rns_group_chains<18, 2, 8, 1, 2>), dim3(blocks), dim3(640), 0, st, j); break;
    case 36:
      if (fold) hipLaunchKernelGGL((k_rns_wide_chains<true>), dim3(blocks), dim3(256), 0, st, j);
      else hipLaunchKernelGGL((k_rns_wide_chains<false>), dim3(blocks), dim3(256), 0, st, j);
      break;
    default: return HAFLO_EINVAL;
  }
  return hip_status(hipGetLastError());
}

int rns_power(const ModHost* const* m, const DevProg* const* prog, int jobs, const haflo_ctx* ctx, uint32_t* ws,
              const RnsBuffers& b, size_t count, int entries, bool pair, hipStream_t st) {
  const int nr = rns::regs_for(m[0]->nl);
  const int sets = rns_sets(ctx, nr, count, jobs, pair);
  const size_t elements = 16 * (size_t)sets, tiles = (count + elements - 1) / elements;
  const bool group = use_group(ctx, nr, count, jobs);
  // wavefronts of 16 or 32 elements: one block per compute unit, with as many in each as it takes to spread the elements
  // over all of them
  size_t waves = (tiles * (size_t)jobs + ctx->num_cu - 1) / ctx->num_cu;
  waves = std::min(std::max(waves, (size_t)1), (size_t)(nr == 18 && pair ? 16 : 4 * rns_waves_per_simd(sets)));
  const size_t slots = table_slots(ctx, nr, count, jobs);
  const bool fold = group && group_folds(ctx, count, jobs, pair);
  const unsigned blocks = (unsigned)(group ? group_blocks(ctx, nr, count, jobs, fold) : (tiles + waves - 1) / waves);
  RnsJob job[2];
  for (int i = 0; i < jobs; ++i) {
    job[i].tables = m[i]->d_rns;
    job[i].prog = prog[i]->d_ins;
    job[i].len = (int)prog[i]->host.size();
    if (!prog[i]->d_ins) {
      if (prog[i]->host.size() > (size_t)kRnsInline) return HAFLO_EINVAL;
      std::copy(prog[i]->host.begin(), prog[i]->host.end(), job[i].ins);
    }
    job[i].in = ws + b.in[i];
    job[i].nl = m[i]->nl;
    job[i].out = (long long*)(ws + b.out[i]);
    job[i].slots = ws + b.tables + (size_t)i * slots * (size_t)entries * 4 * (size_t)nr * 64;
    job[i].entries = entries;
  }
  if (jobs == 1) job[1] = job[0];
#define LAUNCH(KERNEL, THREADS) \
  hipLaunchKernelGGL(KERNEL, dim3(blocks * jobs), dim3(THREADS), 0, st, job[0], job[1], blocks, count)
#define WAVES(NR)                                                                          \
  do {                                                                                     \
    if (pair && sets == 1) LAUNCH((k_rns<NR, true, 1>), (unsigned)waves * 64);             \
    else if (pair) LAUNCH((k_rns<NR, true, 2>), (unsigned)waves * 64);                     \
    else if (sets == 1) LAUNCH((k_rns<NR, false, 1>), (unsigned)waves * 64);               \
    else LAUNCH((k_rns<NR, false, 2>), (unsigned)waves * 64);                              \
  } while (0)
#define GROUP(NR, TW, W, TW1, W1)                                                      \
  do {                                                                                 \
    if (fold) LAUNCH((k_rns_group<NR, TW, W, TW1, W1, true, true>), (W + W1) * 64);       \
    else if (pair) LAUNCH((k_rns_group<NR, TW, W, TW1, W1, true, false>), (W + W1) * 64); \
    else LAUNCH((k_rns_group<NR, TW, W, TW1, W1, false, false>), (W + W1) * 64);          \
  } while (0)
  switch (nr) {
    case 6:
      if (group) GROUP(6, 1, 5, 1, 0);
      else WAVES(6);
      break;
    case 10:
      if (group) GROUP(10, 1, 9, 1, 0);
      else WAVES(10);
      break;
    case 18:
      if (group) GROUP(18, 2, 8, 1, 2);
      else if (pair) LAUNCH((k_rns_one<18>), (unsigned)waves * 64);
      else LAUNCH((k_rns<18, false, 2>), (unsigned)waves * 64);
      break;
    case 36:
      if (!pair || jobs != 1) return HAFLO_EINVAL;
      if (fold) hipLaunchKernelGGL((k_rns_wide<true>), dim3(blocks), dim3(256), 0, st, job[0], count);
      else hipLaunchKernelGGL((k_rns_wide<false>), dim3(blocks), dim3(256), 0, st, job[0], count);
      break;
    default: return HAFLO_EINVAL;
  }
#undef GROUP
#undef WAVES
#undef LAUNCH
  return hip_status(hipGetLastError());
}

}  // namespace haflo
