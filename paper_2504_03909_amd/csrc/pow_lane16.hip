// k_pow_pair with one or two lanes per integer, bases of 16 limbs (1024-bit keys)
#include "pow_pair.hpp"

namespace he {

const void *pow_lane16(int SN, int L, PairPow which) {
  if (SN == 16 && L == 0) return pow_pair_fn<16, 0>(which);
  if (SN == 16 && L == 1) return pow_pair_fn<16, 1>(which);
  if (SN == 16 && L == 2) return pow_pair_fn<16, 2>(which);
  return nullptr;
}

}  // namespace he
