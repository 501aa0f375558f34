// Calls the residue engine's list programs by themselves, for tests/test_emu_rns.py (linked with the CPU build).
#include "haflo_internal.hpp"

using namespace haflo;

extern "C" {
size_t lists_item_words(const haflo_ctx* ctx) { return rns_item_words(ctx->Nh); }
// `count` pairs of limbs into the form, by a program that has no operands: there is nothing at the places of those, or of one
int lists_without_operands(const haflo_ctx* ctx, const uint32_t* limbs, size_t count, uint32_t* out) {
  RnsLists j = {};
  j.limbs = limbs;
  j.out = out;
  j.stride = count;
  j.add(LIST_ACC_LIMBS);
  j.add(LIST_ACC_SQ);
  j.add(LIST_STORE_ACC);
  return rns_lists(ctx, ctx->Nh, j, count, nullptr);
}
}
