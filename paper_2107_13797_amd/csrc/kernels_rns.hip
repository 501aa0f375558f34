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
// multiple of s, which M_A's 22 to 28 spare bits absorb. The second extension is exact: t is far below M_B and the
// b_j are within 2^-17 of 2^30, so the sum lies within 2^-7 of an integer.)
// The word-serial pair product takes 3.6 (5 for a product of two elements) NL^2 multiply-adds per element; here the
// NL^2 part are four products with constant matrices over a whole batch, which the matrix cores do on the residues'
// bytes, and the vector unit is left with about 50 instructions per prime.
//
// Layout. A wavefront owns 16 elements; lane l holds a quarter (g = l / 16) of the residues of element l % 16: channel
// slot 4 i + g in register i. With the constant matrix as the first operand of v_mfma_i32_16x16x64_i8 and the residues'
// bytes as the second, four consecutive rows of a result belong to one lane: the four byte rows of one destination slot.
// So a lane gets whole residues from the product, works on them alone and feeds them to the next product as they are: no
// lane exchange, no LDS traffic but the matrices', no barrier. Both reductions of a product share every matrix fragment
// they read.
#include "kernels_common.hpp"
#include "rns.hpp"

using namespace haflo;
using namespace haflo::dev;

namespace {

typedef u32 Quad __attribute__((vector_size(16)));
typedef u32 Twin __attribute__((vector_size(8)));
typedef int Acc __attribute__((vector_size(16)));  // also a matrix operand of 16 bytes

struct RnsJob {
  const u32* tables;  // rns.hpp's device layout
  const u32* prog;    // ENG_SQ, ENG_MUL_T, ENG_MUL_T_ST, ENG_STORE_T, ENG_LOAD_T only
  int len;
  const u32* in;      // per element [x0: nl limbs][x1: nl limbs], limbs below 2^32
  int nl;
  long long* out;     // per element [x0: columns][x1: columns] of weight 2^(29 l), signed
  u32* slots;         // window tables: 4 NR dwords per lane and entry
  int entries;
};

// The residues of x0 and x1 of a lane in one base, in the registers that the matrix products take them from: full
// quads of each, and one quad with the last two of both.
template <int NR>
struct Residues {
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
    if (k < kFull) asm("" : "+v"(q[0][k]), "+v"(q[1][k]));
    else asm("" : "+v"(h));
  }
  // Hides where the values come from: the compiler would widen what is multiplied later to 64 bits where it is made
  // and carry the zero upper words along.
  __device__ __forceinline__ void forget() {
#pragma unroll
    for (int k = 0; k < kFull; ++k) asm("" : "+v"(q[0][k]), "+v"(q[1][k]));
    asm("" : "+v"(h));
  }
};
template <int NR>
struct RnsState {
  Residues<NR> a, b;
};

// T 2^-32 mod p, below (T + 2^32 p) / 2^32
__device__ __forceinline__ u32 reduce(u64 t, u32 p, u32 pinv) {
  const u32 m = (u32)t * pinv;
  u32 r = (u32)(mad64(m, p, t) >> 32);
  asm("" : "+v"(r));  // a register of its own: the compiler would carry the dead low word along with it
  return r;
}

struct RnsConsts {
  s32 k65536, one;  // hidden from the compiler, so that the column sums stay multiply-adds
  s64 base;
  __device__ __forceinline__ RnsConsts() : k65536(65536), one(1), base((s64)rns::kBase) {
    asm volatile("" : "+r"(k65536), "+r"(one), "+r"(base));
  }
};

// A residue as the bytes the matrix products take (each 128 less), and back. Hidden from the compiler, which would
// otherwise keep the residue beside its bytes instead of taking it back from them.
__device__ __forceinline__ u32 to_bytes(u32 v) {
  v ^= rns::kOmega;
  asm("" : "+v"(v));
  return v;
}

// the four byte rows of a slot as one number; BASE: 2^47 added
template <bool BASE>
__device__ __forceinline__ s64 column(const Acc& acc, const RnsConsts& kc) {
  const s32 lo = (s32)((u32)acc[1] << 8) + acc[0];
  const s32 hi = (s32)((u32)acc[3] << 8) + acc[2];
  const s64 t = (s64)hi * (s64)kc.k65536 + (BASE ? kc.base : (s64)0);
  return (s64)lo * (s64)kc.one + t;
}

// Where this lane's part of a fragment lies in a tile of 16 (kept) rows: of a full one, and of the half one
struct FragmentAt {
  int full, half;  // bytes
  __device__ __forceinline__ FragmentAt(int lane, int rows) {
    full = ((lane >> 4) * rows + (lane & (rows - 1))) * 16;
    half = full / 2;
  }
  // read again for each product: held in registers, the matrix would not fit them
  __device__ __forceinline__ void forget() { asm volatile("" : "+v"(full), "+v"(half)); }
};

// The operand of a matrix product: the half block's words of x0 and of x1 in a quad of their own, zeros behind them.
template <int NR>
struct Operand {
  Residues<NR>& d;
  Quad h0, h1;
  __device__ __forceinline__ explicit Operand(Residues<NR>& d_)
      : d(d_), h0(Quad{d_.h[0], d_.h[1], 0, 0}), h1(Quad{d_.h[2], d_.h[3], 0, 0}) {
    asm("" : "+v"(h0), "+v"(h1));  // made once, not for every tile
  }
  // back to the residues' own form
  __device__ __forceinline__ void release() { d.h = Quad{h0[0], h0[1], h1[0], h1[1]}; }
};

// One tile (4 destination slots, one per lane) of a matrix times both halves of a pair. Of the half block only 8 bytes
// of a row are stored: what lies in the other registers meets the operand's zeros. (A product of
// v_mfma_i32_16x16x32_i8 added to one of v_mfma_i32_16x16x64_i8 right after it comes out wrong on this chip, either
// way round: one shape only.)
template <int NR>
__device__ __forceinline__ void tile_products(Acc& r0, Acc& r1, const void* tile, int rows, const FragmentAt& at,
                                              const Operand<NR>& d) {
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
  r0 = Acc{0, 0, 0, 0};
  r1 = Acc{0, 0, 0, 0};
#pragma unroll
  for (int k = 0; k <= F; ++k) {
    r0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(m[k], (Acc)(k < F ? d.d.q[0][k < F ? k : 0] : d.h0), r0, 0, 0, 0);
    r1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(m[k], (Acc)(k < F ? d.d.q[1][k < F ? k : 0] : d.h1), r1, 0, 0, 0);
  }
}

template <int NR>
struct RnsEngine {
  static constexpr int kTiles = rns::tiles(NR);  // also the registers that hold primes
  static constexpr int kGroup = 3;               // tiles the compiler may mix
  static constexpr int kTileBytes = rns::tile_bytes(NR, 16);
  static constexpr int kLast = rns::last_rows(NR);
  const char* lds;
  int lane, g;
  RnsConsts kc;
  FragmentAt at, at_last;  // of a tile, and of the last one
  int cst_at;              // of this lane group's constants in a row of four slots
  u32 keep, mine, one;     // masks of set_extra

  __device__ __forceinline__ RnsEngine(const void* lds_)
      : lds((const char*)lds_), lane((int)(threadIdx.x & (WAVE - 1))), g(lane >> 4), at(lane, 16), at_last(lane, kLast),
        cst_at(16 * g), keep(g < 2 ? ~0u : 0u), mine(g == 2 ? ~0u : 0u), one(g == 3 ? 1u : 0u) {
    asm volatile("" : "+v"(keep), "+v"(mine), "+v"(one));  // no branches
  }
  // Everything a wavefront reads from LDS is constant over the launch: without these the compiler would read it once
  // and not have the registers for it. They also bound what it may mix.
  __device__ __forceinline__ void forget() {
    __builtin_amdgcn_sched_barrier(0);
    at.forget();
    if (kLast != 16) at_last.forget();
    asm volatile("" : "+v"(cst_at));
  }
  __device__ __forceinline__ Quad cst(int base, int i) const {
    return *(const Quad*)(lds + 2 * rns::lds_matrix_bytes(NR) + (base * rns::slots(NR) + 4 * i) * 16 + cst_at);
  }
  template <int MATRIX>
  __device__ __forceinline__ void lds_products(Acc& r0, Acc& r1, int t, const Operand<NR>& d) const {
    const char* p = lds + MATRIX * rns::lds_matrix_bytes(NR) + t * kTileBytes;
    if (t == kTiles - 1) tile_products<NR>(r0, r1, p, kLast, kLast != 16 ? at_last : at, d);
    else tile_products<NR>(r0, r1, p, 16, at, d);
  }

  // The residue products of one base of a square (y null) or of a product with the table entry y: bytes of sigma in
  // base A (BASE 0), z and w in base B. The entry's quads are on their way one step ahead.
  template <int BASE, bool SQ>
  __device__ __forceinline__ void base_products(Residues<NR>& x, const u32* y) {
    constexpr int kQuads = NR / 4 + 1;
    const Quad* p = (const Quad*)(y + BASE * kArray) + lane;
    x.forget();
    Quad n0 = {}, n1 = {};
    if (!SQ) {
      n0 = p[0];
      n1 = p[WAVE];
    }
#pragma unroll
    for (int q = 0; q < kQuads; ++q) {
      const Quad y0 = n0, y1 = n1;
      forget();
      if (!SQ && q + 1 < kQuads) {
        n0 = p[2 * (q + 1) * WAVE];
        if (q + 2 < kQuads) n1 = p[(2 * (q + 1) + 1) * WAVE];
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int i = 4 * q + c;
        if (i >= kTiles || i >= NR) continue;
        const Quad k = cst(BASE, i);
        const u32 u0 = x.template get<0>(i), u1 = x.template get<1>(i);
        const u32 v0 = SQ ? u0 : y0[c], v1 = SQ ? u1 : (q + 1 < kQuads ? y1[c] : y0[(2 + c) % 4]);
        const u32 s0 = reduce(mad64(u0, v0, 0), k[0], k[1]);
        const u64 cross = SQ ? mad64(u0 << 1, u1, 0) : mad64(u0, v1, mad64(u1, v0, 0));
        const u32 s1 = reduce(mad64(s0, BASE ? k[3] : k[2], cross), k[0], k[1]);
        x.template set<0>(i, BASE ? s0 : to_bytes(s0));
        x.template set<1>(i, BASE ? s1 : to_bytes(s1));
      }
      x.gather(q);
    }
  }
  template <bool SQ>
  __device__ __forceinline__ void products(RnsState<NR>& x, const u32* y) {
    base_products<0, SQ>(x.a, y);
    base_products<1, SQ>(x.b, y);
  }

  // the constant 1 of the bias in its slot, and alpha's bytes in theirs (lane groups 3 and 2 of the last register)
  __device__ __forceinline__ void set_extra(Residues<NR>& d, u32 alpha0, u32 alpha1) const {
    d.h[1] = (d.h[1] & keep) | (alpha0 & mine) | one;
    d.h[3] = (d.h[3] & keep) | (alpha1 & mine) | one;
  }
  // alpha of a value from the sum of its residues' upper halves over this lane's slots
  __device__ __forceinline__ u32 alpha_bytes(u32 sum) const {
    sum += (u32)__builtin_amdgcn_ds_bpermute((lane ^ 16) << 2, (int)sum);
    sum += (u32)__builtin_amdgcn_ds_bpermute((lane ^ 32) << 2, (int)sum);
    const u32 a = (sum + (1u << 13)) >> 14;
    return (a & 127u) | ((a >> 7) << 8);
  }

  // Base B of the reduced pair from sigma (bytes, in base A) and the products z, w (in base B); leaves base B as bytes,
  // alpha among them, for the way back.
  __device__ __forceinline__ void extend_to_b(RnsState<NR>& x) {
    x.b.forget();
    set_extra(x.a, 0, 0);
    Operand<NR> d(x.a);
    u32 sum0 = 0, sum1 = 0;
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      if (t % kGroup == 0) {
        asm volatile("" : "+v"(sum0), "+v"(sum1));  // running sums: summed up at the end they would keep every term alive
        forget();
      }
      Acc r0, r1;
      lds_products<0>(r0, r1, t, d);
      const Quad k = cst(1, t);
      const u32 t0 = reduce(mad64(x.b.template get<0>(t), k[2], (u64)column<true>(r0, kc)), k[0], k[1]);
      const u64 col = mad64(x.b.template get<1>(t), k[2], (u64)column<true>(r1, kc));
      const u32 t1 = reduce(mad64(t0, k[0] - k[3], col), k[0], k[1]);
      sum0 += t0 >> 16;
      sum1 += t1 >> 16;
      x.b.template set<0>(t, to_bytes(t0));
      x.b.template set<1>(t, to_bytes(t1));
      if (t % 4 == 3) x.b.gather(t / 4);
    }
    set_extra(x.b, alpha_bytes(sum0), alpha_bytes(sum1));
  }
  // base A from base B's bytes; turns base B back to residues
  __device__ __forceinline__ void extend_to_a(RnsState<NR>& x) {
    Operand<NR> d(x.b);
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      if (t % kGroup == 0) forget();
      Acc r0, r1;
      lds_products<1>(r0, r1, t, d);
      const Quad k = cst(0, t);
      x.a.template set<0>(t, reduce((u64)column<true>(r0, kc), k[0], k[1]));
      x.a.template set<1>(t, reduce((u64)column<true>(r1, kc), k[0], k[1]));
      if (t % 4 == 3) x.a.gather(t / 4);
    }
    d.release();
    flip(x.b);
  }
  // residues <-> bytes
  static __device__ __forceinline__ void flip(Residues<NR>& d) {
#pragma unroll
    for (int k = 0; k < NR / 4; ++k) {
      d.q[0][k] ^= rns::kOmega;
      d.q[1][k] ^= rns::kOmega;
    }
    d.h ^= rns::kOmega;
  }

  // the pairs whose limbs are at `src` (`left` of them, then zeros) into both bases
  __device__ __forceinline__ void load(RnsState<NR>& x, const u32* src, unsigned left, int nl, const char* matrix) {
    const bool active = (unsigned)(lane & 15) < left;
    src += (lane & 15) * 2 * nl;
    x = RnsState<NR>();
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int l = 4 * i + g;
      const bool ok = active && l < nl;
      x.a.template set<0>(i, (ok ? src[l] : 0u) ^ rns::kOmega);
      x.a.template set<1>(i, (ok ? src[nl + l] : 0u) ^ rns::kOmega);
    }
    if (g == 3) {  // in place of a limb that is zero
      x.a.template set<0>(NR - 1, 1);
      x.a.template set<1>(NR - 1, 1);
    }
    Operand<NR> d(x.a);
    u32 sum0 = 0, sum1 = 0;
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      forget();
      Acc r0, r1;
      tile_products<NR>(r0, r1, matrix + t * kTileBytes, 16, at, d);
      const Quad k = cst(1, t);
      const u32 t0 = reduce((u64)column<true>(r0, kc), k[0], k[1]);
      const u32 t1 = reduce((u64)column<true>(r1, kc), k[0], k[1]);
      sum0 += t0 >> 16;
      sum1 += t1 >> 16;
      asm volatile("" : "+v"(sum0), "+v"(sum1));
      x.b.template set<0>(t, to_bytes(t0));
      x.b.template set<1>(t, to_bytes(t1));
    }
    set_extra(x.b, alpha_bytes(sum0), alpha_bytes(sum1));
    extend_to_a(x);
  }
  // The pair as two integers in columns of weight 2^(29 l). Base B still holds what the way back left there, alpha and
  // the bias among it.
  __device__ __forceinline__ void store(RnsState<NR>& x, long long* dst, unsigned left, const char* matrix) {
    const bool active = (unsigned)(lane & 15) < left;
    dst += (lane & 15) * 8 * kTiles;
    flip(x.b);
    Operand<NR> d(x.b);
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      forget();
      Acc r0, r1;
      tile_products<NR>(r0, r1, matrix + t * kTileBytes, 16, at, d);
      if (active) {
        dst[4 * t + g] = column<false>(r0, kc);
        dst[4 * kTiles + 4 * t + g] = column<false>(r1, kc);
      }
    }
  }

  // Window tables: an entry holds the registers of base A and of base B one after the other, each as [quad][lane].
  static constexpr int kArray = (2 * (NR / 4) + 1) * 4 * WAVE;  // dwords
  __device__ __forceinline__ void load_entry(Residues<NR>& d, const u32* entry, int array) const {
    const Quad* p = (const Quad*)(entry + array * kArray) + lane;
#pragma unroll
    for (int k = 0; k < NR / 4; ++k) {
      d.q[0][k] = p[2 * k * WAVE];
      d.q[1][k] = p[(2 * k + 1) * WAVE];
    }
    d.h = p[2 * (NR / 4) * WAVE];
  }
  __device__ __forceinline__ void store_entry(const Residues<NR>& d, u32* entry, int array) const {
    Quad* p = (Quad*)(entry + array * kArray) + lane;
#pragma unroll
    for (int k = 0; k < NR / 4; ++k) {
      p[2 * k * WAVE] = d.q[0][k];
      p[(2 * k + 1) * WAVE] = d.q[1][k];
    }
    p[2 * (NR / 4) * WAVE] = d.h;
  }
  __device__ __forceinline__ void load_state(RnsState<NR>& x, const u32* entry) const {
    load_entry(x.a, entry, 0);
    load_entry(x.b, entry, 1);
  }
  __device__ __forceinline__ void store_state(const RnsState<NR>& x, u32* entry) const {
    store_entry(x.a, entry, 0);
    store_entry(x.b, entry, 1);
  }
};

// Four wavefronts per SIMD, 128 registers: 72 of state, 20 for a tile's fragments, 8 for its sums. Measured at 65536
// elements and a 2048-bit modulus: 49 ms per 2363 products where the word-serial pair products took 128 (1024 bits: 10
// against 25 ms); the matrix cores are busy 61 % of the cycles, the vector units issue in 64 % of them (1119 vector and
// 360 matrix instructions per squaring and wavefront), LDS reads take 41 %, at 1.9 GHz. 32 elements per wavefront (half
// the matrix reads) need 256 registers and more, and spilled.
// Every wavefront runs the program on 16 elements at a time. The first `split` blocks run j0, the others j1.
template <int NR>
__global__ __launch_bounds__(1024, 4) void k_rns(RnsJob j0, RnsJob j1, unsigned split, size_t count) {
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
  RnsEngine<NR> e(lds);
  const unsigned waves = blockDim.x / 64;
  // the same for the whole wavefront, so that what follows from it stays in scalar registers
  const size_t wave = (size_t)block * waves + (unsigned)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64));
  constexpr size_t kEntry = 4 * NR * WAVE;
  const u32* prog = j.prog;
  const int len = __builtin_amdgcn_readfirstlane(j.len);
  u32* table = j.slots + wave * (size_t)j.entries * kEntry;
  for (size_t tile = wave; tile * 16 < count; tile += (size_t)nblocks * waves) {
    const unsigned left = (unsigned)std::min(count - tile * 16, (size_t)16);
    RnsState<NR> x;
    e.load(x, j.in + tile * (size_t)(16 * 2 * j.nl), left, j.nl, in_matrix);
    for (int pc = 0; pc < len;) {
      u32 ins = (u32)__builtin_amdgcn_readfirstlane((int)prog[pc]);
      // a run of squarings (nine tenths of a program) in a loop of its own, where the state stays in registers
#pragma unroll 1
      while (ins == ENG_SQ) {
        e.template products<true>(x, nullptr);
        e.extend_to_b(x);
        e.extend_to_a(x);
        ins = ++pc < len ? (u32)__builtin_amdgcn_readfirstlane((int)prog[pc]) : ~0u;
      }
      if (pc++ >= len) break;
      const u32 op = ins & 0xFFu, a = (ins >> 8) & 0xFFFu, b = ins >> 20;
      u32* entry = table + (size_t)a * kEntry;
      if (op == ENG_STORE_T) {
        e.store_state(x, entry);
      } else if (op == ENG_LOAD_T) {
        e.load_state(x, entry);
      } else {
        e.template products<false>(x, entry);
        e.extend_to_b(x);
        e.extend_to_a(x);
        if (op == ENG_MUL_T_ST) e.store_state(x, table + (size_t)b * kEntry);
      }
    }
    e.store(x, j.out + tile * (size_t)(16 * 8 * rns::tiles(NR)), left, out_matrix);
  }
}

}  // namespace

namespace haflo {

// Wavefronts of 16 elements that are resident at once: four per SIMD
constexpr int kRnsWavesPerCu = 16;

// From how many chains (elements times moduli) on. One wavefront's chain takes the same time however few elements it
// holds: 3.2 ms for an encryption at a 1024-bit key (2.7 ms with an integer per wavefront up to 1024 chains, 3.7 ms at
// 2048), 17.1 ms at 2048 bits (8.5 ms up to 1024, 14.7 ms at 2048, 17.5 ms at 3000), 3.2 ms for a decryption at 2048
// bits (2.7 ms at 512 chains, 3.7 ms at 2048), 17.1 ms at 4096 bits (14.9 ms at 2048 chains, 29 ms at 6000).
bool rns_pays(const haflo_ctx* ctx, const ModHost& m, size_t count, int jobs) {
  return m.d_rns && count * (size_t)jobs >= (size_t)ctx->num_cu * (m.nl == 72 ? 10 : 7);
}
size_t rns_chunk(const haflo_ctx* ctx, int jobs) {
  return std::max((size_t)ctx->num_cu * kRnsWavesPerCu / (size_t)jobs, (size_t)1) * 16;
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
  const size_t tiles = ((n + 15) / 16 + kRnsWavesPerCu - 1) / kRnsWavesPerCu * kRnsWavesPerCu;  // whole blocks
  b.total = at + std::max((size_t)jobs * tiles * (size_t)entries * 4 * (size_t)nr * 64,
                          (size_t)jobs * (n + 128) * 2 * (size_t)m.nl);
  return b;
}

int rns_power(const ModHost* const* m, const DevProg* const* prog, int jobs, const haflo_ctx* ctx, uint32_t* ws,
              const RnsBuffers& b, size_t count, int entries, hipStream_t st) {
  const int nr = rns::regs_for(m[0]->nl);
  const size_t tiles = (count + 15) / 16;
  // wavefronts of 16 elements: one block per compute unit, with as many in each as it takes to spread the elements
  // over all of them
  size_t waves = (tiles * (size_t)jobs + ctx->num_cu - 1) / ctx->num_cu;
  waves = std::min(std::max(waves, (size_t)1), (size_t)kRnsWavesPerCu);
  const unsigned blocks = (unsigned)((tiles + waves - 1) / waves);
  const size_t slots = (size_t)blocks * waves;
  RnsJob job[2];
  for (int i = 0; i < jobs; ++i) {
    job[i].tables = m[i]->d_rns;
    job[i].prog = prog[i]->d_ins;
    job[i].len = (int)prog[i]->host.size();
    job[i].in = ws + b.in[i];
    job[i].nl = m[i]->nl;
    job[i].out = (long long*)(ws + b.out[i]);
    job[i].slots = ws + b.tables + (size_t)i * slots * (size_t)entries * 4 * (size_t)nr * 64;
    job[i].entries = entries;
  }
  if (jobs == 1) job[1] = job[0];
#define WAVES(NR) \
  hipLaunchKernelGGL((k_rns<NR>), dim3(blocks * jobs), dim3((unsigned)waves * 64), 0, st, job[0], job[1], blocks, count)
  switch (nr) {
    case 6: WAVES(6); break;
    case 10: WAVES(10); break;
    case 18: WAVES(18); break;
    default: return HAFLO_EINVAL;
  }
#undef WAVES
  return hip_status(hipGetLastError());
}

}  // namespace haflo
