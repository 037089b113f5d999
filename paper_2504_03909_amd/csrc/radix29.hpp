// Size of the radix-2^29 Montgomery representation used by the modular
// exponentiation loops (shared by the host key set-up and the kernels).
//
// A modulus N below 2^(32 S) is written in S29 limbs of 29 bits with
// R = 2^(29 S29).  S29 is the fewest limbs with R > 4N, so that Montgomery
// products of operands below 2N stay below 2N without a final subtraction,
// rounded up so that every lane of a G-lane group holds the same number of
// limbs.  Three roundings cover the group widths: variant 0 (multiple of 4:
// groups of 2 or 4 lanes), 1 (multiple of 8: 8 lanes), 2 (multiple of 16:
// 16 lanes); the key stores constants for each.
#pragma once

namespace he29 {

constexpr int kBits = 29;
constexpr int kVariants = 3;

constexpr int variant(int G) { return G <= 4 ? 0 : (G == 8 ? 1 : 2); }
constexpr int multiple(int v) { return v == 0 ? 4 : (v == 1 ? 8 : 16); }
constexpr int limbs(int S, int v) {
  const int m = (32 * S + 2 + kBits - 1) / kBits;
  const int u = multiple(v);
  return (m + u - 1) / u * u;
}
constexpr int limbs_for_group(int S, int G) { return limbs(S, variant(G)); }

// Residues mod N^2 as two digits base N (pair29.hpp): each digit is an
// integer below 2N in S29 limbs held by g lanes.  Three roundings of the limb
// count: 0 (multiple of 2: 1 or 2 lanes per digit), 1 (4 lanes), 2 (8 lanes).
constexpr int kPairVariants = 3;
constexpr int pair_variant(int g) { return g <= 2 ? 0 : (g == 4 ? 1 : 2); }
constexpr int pair_limbs(int S, int v) {
  const int m = (32 * S + 2 + kBits - 1) / kBits;
  const int u = 2 << v;
  return (m + u - 1) / u * u;
}
// Constants of the two-digit form, in pairs of 2 S29 words (first digit, then
// second), one after the other; then N in S29 limbs.
constexpr int kPairPieces = 4;                // input pieces of 32 S bits
constexpr int kPairOne = kPairPieces;         // (1, 0): leaves the Montgomery domain
constexpr int kPairUnscale = kPairOne + 1;    // (2^(29 (S29 - 1)) mod N, 0): drops the second digit's 2^29
constexpr int kPairR = kPairUnscale + 1;      // R mod N^2: Montgomery form of 1
constexpr int kPairE = kPairR + 1;            // e R mod N^2, and (1 - e) R mod N^2: with e the other prime mod
constexpr int kPairE1 = kPairE + 1;           // (N - 1), they raise 1 + f N to the power e (0 where there is no e)
constexpr int kPairN = kPairE1 + 1;           // N
constexpr int pair_words(int S, int v) { return (2 * kPairN + 1) * pair_limbs(S, v); }

// Schedule of two powers that share their squarings (keysetup.hpp,
// joint_schedule): what an op does with its slot.
constexpr int kJointBits = 5, kJointBuckets = 16;
enum JointOp : unsigned {
  kJointPut,   // slot = state
  kJointLoad,  // state = slot
  kJointTake,  // state *= slot
  kJointAcc,   // slot *= state
};

}  // namespace he29
