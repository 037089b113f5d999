// The exponentiation kernel on the engines of pair29.hpp, and its launchers'
// interface.
#pragma once
#include "he_internal.hpp"
#include "pair29.hpp"

namespace he {

template <int SN, int L>
struct PairEngine;
template <int SN>
struct PairEngine<SN, 0> { using T = LaneMod<SN>; };
template <int SN>
struct PairEngine<SN, 1> { using T = LanePair<SN>; };
template <int SN>
struct PairEngine<SN, 2> { using T = TwinPair<SN>; };
template <int SN>
struct PairEngine<SN, 4> { using T = GroupPair<SN, 2>; };
template <int SN>
struct PairEngine<SN, 8> { using T = GroupPair<SN, 4>; };
template <int SN>
struct PairEngine<SN, 16> { using T = GroupPair<SN, 8>; };

// Work unit = (prime, 64 / lanes consecutive ciphertexts), claimed from
// `next` or taken by index, as in k_pow.
template <int SN, int L, bool CT>
__global__ __launch_bounds__(kBlockThreads, 2) void k_pow_pair(PairPowArgs p) {
  using E = typename PairEngine<SN, L>::T;
  constexpr int NG = 64 / E::kLanes, ROWS = E::kLds ? kBlockThreads / E::kLanes : 0;
  constexpr int ZERO = E::kLds ? E::S : 0;
  __shared__ __align__(16) uint32_t lds_all[ROWS * E::kLds + ZERO + 4];
  uint32_t *const zeros = lds_all + ROWS * E::kLds;
  if constexpr (ZERO > 0) zero_lds(zeros, ZERO);
  uint32_t *const row = lds_all + (threadIdx.x / E::kLanes) * E::kLds;
  const uint64_t gw = (uint64_t)blockIdx.x * 4 + wave_in_block();
  const uint64_t nw = (uint64_t)gridDim.x * 4;
  uint32_t *const tab = p.tabs + gw * (uint64_t)(kTable + 1) * E::kSlot;
  const uint64_t nunits = 2 * ((p.count + NG - 1) / NG);
  for (uint64_t qd = p.next ? claim_unit(p.next) : gw; qd < nunits; qd = p.next ? claim_unit(p.next) : qd + nw) {
    const int which = (int)(qd & 1);
    uint64_t i = (qd >> 1) * NG + E::member();
    const bool valid = i < p.count;
    if (!valid) i = p.count - 1;
    E eng(UnitArgs{p.consts[which], p.ninv[which], tab}, row, zeros);
    power_unit<E, SN, CT>(eng, p.exp[which], p.in + i * p.in_i + which * p.in_w, p.pieces,
                          p.out + i * p.out_i + which * p.out_w, valid);
  }
}

// Work units as k_pow_pair's; joint_unit on r mod P, one piece in, two digits out.
template <int SN, int L>
__global__ __launch_bounds__(kBlockThreads, 2) void k_pow_joint(PairPowArgs p) {
  using E = typename PairEngine<SN, L>::T;
  constexpr int NG = 64 / E::kLanes, ROWS = E::kLds ? kBlockThreads / E::kLanes : 0;
  constexpr int ZERO = E::kLds ? E::S : 0;
  __shared__ __align__(16) uint32_t lds_all[ROWS * E::kLds + ZERO + 4];
  uint32_t *const zeros = lds_all + ROWS * E::kLds;
  if constexpr (ZERO > 0) zero_lds(zeros, ZERO);
  uint32_t *const row = lds_all + (threadIdx.x / E::kLanes) * E::kLds;
  const uint64_t gw = (uint64_t)blockIdx.x * 4 + wave_in_block();
  const uint64_t nw = (uint64_t)gridDim.x * 4;
  uint32_t *const tab = p.tabs + gw * (uint64_t)(kTable + 1) * E::kSlot;
  const uint64_t nunits = 2 * ((p.count + NG - 1) / NG);
  for (uint64_t qd = p.next ? claim_unit(p.next) : gw; qd < nunits; qd = p.next ? claim_unit(p.next) : qd + nw) {
    const int which = (int)(qd & 1);
    uint64_t i = (qd >> 1) * NG + E::member();
    const bool valid = i < p.count;
    if (!valid) i = p.count - 1;
    E eng(UnitArgs{p.consts[which], p.ninv[which], tab}, row, zeros);
    joint_unit<E, SN>(eng, p.exp[which], p.in + i * p.in_i + which * p.in_w, p.out + i * p.out_i + which * p.out_w,
                      valid);
  }
}

// Per source file: its kernels, null for the others'.
const void *pow_lane16(int SN, int L, PairPow which);
const void *pow_lane32(int SN, int L, PairPow which);
const void *pow_twin32(int SN, int L, PairPow which);
const void *pow_group(int SN, int L, PairPow which);

template <int SN, int L>
const void *pow_pair_fn(PairPow which) {
  if constexpr (L > 0 && SN <= 32)
    if (which == PairPow::kJoint) return (const void *)k_pow_joint<SN, L>;
  if constexpr (L > 0)
    if (which == PairPow::kSliding) return (const void *)k_pow_pair<SN, L, false>;
  if constexpr (SN <= 32)  // the public exponent n is never masked
    if (which == PairPow::kMasked) return (const void *)k_pow_pair<SN, L, true>;
  return nullptr;
}

}  // namespace he
