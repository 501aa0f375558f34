// Calls the residue engine's power by itself with a program of the test's own, for tests/test_emu_rns.py (linked with the CPU
// build).
#include <vector>

#include "haflo_internal.hpp"

using namespace haflo;

extern "C" {
// where the columns of a result, and how many of them per half
int power_columns(const haflo_ctx* ctx) { return rns_columns(ctx->Nh); }
size_t power_workspace_words(const haflo_ctx* ctx, size_t count, int entries) {
  return rns_buffers(ctx, ctx->Nh, count, 1, entries).total;
}
// `count` pairs of limbs, at `limbs`, raised by `ins`; the columns of the results to `out`
int power_program(const haflo_ctx* ctx, uint32_t* ws, const uint32_t* limbs, size_t count, int entries, const uint32_t* ins, int len,
                  long long* out) {
  const ModHost& m = ctx->Nh;
  DevProg prog;
  prog.host.assign(ins, ins + len);
  const RnsBuffers b = rns_buffers(ctx, m, count, 1, entries);
  for (size_t i = 0; i < count * 2 * (size_t)m.nl; ++i) ws[b.in[0] + i] = limbs[i];
  const ModHost* mods[1] = {&m};
  const DevProg* progs[1] = {&prog};
  const int rc = rns_power(mods, progs, 1, ctx, ws, b, count, entries, true, nullptr);
  for (size_t i = 0; i < count * 2 * (size_t)rns_columns(m); ++i) out[i] = ((const long long*)(ws + b.out[0]))[i];
  return rc;
}
}
