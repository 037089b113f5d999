// k_pow_pair with 2, 4 or 8 lanes per digit
#include "pow_pair.hpp"

namespace he {

const void *pow_group(int SN, int L, PairPow which) {
  if (SN == 16 && L == 4) return pow_pair_fn<16, 4>(which);
  if (SN == 16 && L == 8) return pow_pair_fn<16, 8>(which);
  if (SN == 16 && L == 16) return pow_pair_fn<16, 16>(which);
  if (SN == 32 && L == 4) return pow_pair_fn<32, 4>(which);
  if (SN == 32 && L == 8) return pow_pair_fn<32, 8>(which);
  if (SN == 32 && L == 16) return pow_pair_fn<32, 16>(which);
  if (SN == 64 && L == 8) return pow_pair_fn<64, 8>(which);
  if (SN == 64 && L == 16) return pow_pair_fn<64, 16>(which);
  return nullptr;
}

}  // namespace he
