// k_pow_pair with one lane per integer, bases of 32 limbs (2048-bit keys; n of 1024-bit keys)
#include "pow_pair.hpp"

namespace he {

const void *pow_lane32(int SN, int L, PairPow which) {
  if (SN == 32 && L == 0) return pow_pair_fn<32, 0>(which);
  if (SN == 32 && L == 1) return pow_pair_fn<32, 1>(which);
  return nullptr;
}

}  // namespace he
