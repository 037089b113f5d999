// k_pow_pair with two lanes per integer, bases of 32 limbs
#include "pow_pair.hpp"

namespace he {

const void *pow_twin32(int SN, int L, PairPow which) {
  if (SN == 32 && L == 2) return pow_pair_fn<32, 2>(which);
  return nullptr;
}

}  // namespace he
