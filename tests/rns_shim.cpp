// C wrapper around the table geometry of the residue number system engine, for tests/test_rns_tables.py.
#include "../paper_2107_13797_amd/csrc/rns.hpp"

using namespace haflo;

extern "C" {
int rns_primes(int k, unsigned residue, uint32_t* out) {
  const std::vector<uint32_t> p = rns::primes(k, residue);
  for (int i = 0; i < k; ++i) out[i] = p[i];
  return (int)p.size();
}
// the four row bytes of a constant modulo p, from the matrix they are written to (source slot 0, byte 0)
void rns_rows(int nr, int dst, uint32_t value, uint32_t p, int8_t* out) {
  rns::Matrix m(nr, rns::tiles(nr), 16);
  m.set(0, 0, dst, value, rns::Matrix::Weight(p));
  const int tile = dst / 4, g = dst % 4;
  for (int v = 0; v < 4; ++v) out[v] = (int8_t)m.bytes()[(size_t)tile * rns::tile_bytes(nr, 16) + (size_t)(4 * g + v) * (rns::full_blocks(nr) ? 16 : 8)];
}
uint32_t rns_times256(uint32_t v, uint32_t p) { return rns::times256(v, p); }
// the limbs that go into the bases, of the modulus size that has `nr` registers
int rns_limb_sources(int nr) {
  for (int nl : {18, 36, 72, 144})
    if (rns::regs_for(nl) == nr) return nl < rns::bias_slot(nr) ? nl : rns::bias_slot(nr);
  return 0;
}
uint32_t rns_primes_for(int nr) { return (uint32_t)rns::primes_for(nr); }
}
