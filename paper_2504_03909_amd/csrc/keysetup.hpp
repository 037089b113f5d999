// Host-side derivation of every per-key constant the kernels read, laid out
// in one blob of 32-bit limbs (uploaded once per key).  Host only; no HIP.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "hostbn.hpp"
#include "radix29.hpp"

namespace hekey {

using hebn::Limbs;
constexpr int kWindowBits = 5;

struct Blob {
  std::vector<uint32_t> words;
  // Appends x as exactly `limbs` limbs (plus `pad` zero limbs), 16-byte
  // aligned; returns the offset in limbs.
  size_t put(const Limbs &x, size_t limbs, size_t pad = 0) {
    const size_t off = words.size();
    words.resize(off + limbs + pad, 0u);
    hebn::to_words(x, words.data() + off, limbs);
    words.resize((words.size() + 3) & ~size_t(3), 0u);
    return off;
  }
  // Appends x as exactly `limbs` limbs of 29 bits (one per 32-bit word),
  // 16-byte aligned; throws if it does not fit.
  size_t put29(const Limbs &x, size_t limbs) {
    if (hebn::bit_length(x) > he29::kBits * limbs) throw std::runtime_error("value exceeds 29-bit limbs");
    const size_t off = words.size();
    words.resize(off + limbs, 0u);
    for (size_t i = 0; i < limbs; ++i) {
      uint32_t v = 0;
      for (int k = 0; k < he29::kBits; ++k) v |= (uint32_t)hebn::bit(x, he29::kBits * i + k) << k;
      words[off + i] = v;
    }
    words.resize((words.size() + 3) & ~size_t(3), 0u);
    return off;
  }
};

struct ModOff {  // Montgomery modulus N of S limbs, R = 2^(32 S)
  size_t N, R1, R2, R3, R4;
  uint32_t ninv;
  // radix-2^29 form per variant asked for: N, R mod N and R^2 mod N with R = 2^(29
  // S29); 0 where it was not
  size_t N29[he29::kVariants] = {}, R1_29[he29::kVariants] = {}, R2_29[he29::kVariants] = {};
};
// Constants of the two-digit form of residues mod N^2, per limb-count variant.
struct PairOff {
  size_t c[he29::kPairVariants];
  uint32_t ninv;
};
struct ExpOff {
  size_t e;
  int nwin;
  size_t ops;  // sliding-window schedule (see sliding_schedule)
  int nops;
};

// Sliding-window schedule of e >= 1 with windows of up to kSlideBits bits
// whose lowest bit is 1 (Koc 1995, left to right): the first op loads the
// odd power x^(2 k + 1) of its window (k in bits 0..7); every later op is
// `nsq` squarings (bits 8..31) and then a multiplication by the odd power
// of its window, or no multiplication when k = kSlideNoMul (the trailing
// zero bits).  Evaluating e' = 2 k0 + 1, then e' = e' 2^nsq + (2 k + 1) per
// op rebuilds e.  Empty for e = 0.
constexpr int kSlideBits = 6;
constexpr uint32_t kSlideNoMul = 0xFF;
inline std::vector<uint32_t> sliding_schedule(const Limbs &e) {
  std::vector<uint32_t> ops;
  int i = (int)hebn::bit_length(e) - 1;
  uint32_t pend = 0;
  bool first = true;
  while (i >= 0) {
    if (!hebn::bit(e, (size_t)i)) {
      ++pend;
      --i;
      continue;
    }
    int j = std::max(i - kSlideBits + 1, 0);
    while (!hebn::bit(e, (size_t)j)) ++j;
    uint32_t val = 0;
    for (int b = i; b >= j; --b) val = (val << 1) | (uint32_t)hebn::bit(e, (size_t)b);
    const uint32_t k = (val - 1) >> 1;
    ops.push_back(first ? k : (((pend + (uint32_t)(i - j + 1)) << 8) | k));
    first = false;
    pend = 0;
    i = j - 1;
  }
  if (pend) ops.push_back((pend << 8) | kSlideNoMul);
  return ops;
}

// Two powers x^f and x^e of one base, f, e >= 1, sharing the squarings (Yao
// 1976, right to left): x runs through x^(2^i); where a window of he29::kJointBits
// bits with lowest bit 1 and value 2 k + 1 starts at bit i of an exponent, x^(2^i)
// is multiplied into that exponent's bucket k, and at the end an exponent's
// power is prod_k B_k^(2 k + 1) = (prod_k B_k^k)^2 prod_k B_k, the inner product
// by suffix products.  f's buckets are slots 0..15, e's 16..31.  An op is its
// slot (bits 0..7), what to do with it (bits 8..9) and the squarings of the
// state before (bits 10..31).  At the end slot 0 holds x^f, the state x^e.
inline std::vector<uint32_t> joint_schedule(const Limbs &f, const Limbs &e) {
  std::vector<uint32_t> ops;
  auto op = [&](size_t nsq, he29::JointOp what, uint32_t slot) { ops.push_back((uint32_t)(nsq << 10) | (what << 8) | slot); };
  bool used[2 * he29::kJointBuckets] = {};
  size_t next[2] = {0, 0}, at = 0;  // bit of the next window, bit the state is at
  const Limbs *x[2] = {&f, &e};
  const size_t bits = std::max(hebn::bit_length(f), hebn::bit_length(e));
  for (size_t i = 0; i < bits; ++i)
    for (uint32_t w = 0; w < 2; ++w) {
      if (i < next[w] || !hebn::bit(*x[w], i)) continue;
      uint32_t val = 0;
      for (int b = he29::kJointBits - 1; b >= 0; --b) val = (val << 1) | (uint32_t)hebn::bit(*x[w], i + (size_t)b);
      const uint32_t slot = w * he29::kJointBuckets + (val >> 1);
      op(i - at, used[slot] ? he29::kJointAcc : he29::kJointPut, slot);
      used[slot] = true;
      at = i;
      next[w] = i + he29::kJointBits;
    }
  for (uint32_t w = 0; w < 2; ++w) {
    const uint32_t base = w * he29::kJointBuckets;
    uint32_t top = he29::kJointBuckets - 1;
    while (top > 0 && !used[base + top]) --top;
    op(0, he29::kJointLoad, base + top);
    if (top > 0) {
      // the state: prod of the buckets from j up; slot top: the product of those
      for (uint32_t j = top - 1; j >= 1; --j) {
        if (used[base + j]) op(0, he29::kJointTake, base + j);
        op(0, he29::kJointAcc, base + top);
      }
      if (used[base]) op(0, he29::kJointTake, base);
      op(0, he29::kJointPut, base);
      op(0, he29::kJointLoad, base + top);
      op(1, he29::kJointTake, base);
    }
    if (w == 0) op(0, he29::kJointPut, 0);
  }
  return ops;
}
struct PrimeOff {
  ModOff P, P2;
  PairOff pair;
  ExpOff e_enc, e_lift, e_dec, joint;
  size_t QR_P, QR2_P, PR_P2, Pinv, hR_P;
};
struct KeyConsts {
  Blob blob;
  ModOff n, n2;
  PairOff pair_n;
  ExpOff e_n;
  size_t nR_n2 = 0, half = 0;
  PrimeOff pr[2]{};
  size_t Cq = 0, q2R_n2 = 0, qinv_p = 0, qR_n = 0;
};

inline Limbs pow2(size_t e) { return hebn::shl(hebn::from_u64(1), e); }

// v29: the radix-2^29 variants a kernel reads of N (bit v), none of n and P^2.
inline ModOff put_mod(Blob &b, const Limbs &N, size_t S, uint32_t v29) {
  ModOff m;
  const Limbs R1 = hebn::mod(pow2(32 * S), N);
  const Limbs R2 = hebn::mulmod(R1, R1, N);
  const Limbs R3 = hebn::mulmod(R2, R1, N);
  const Limbs R4 = hebn::mulmod(R3, R1, N);
  m.N = b.put(N, S);
  m.R1 = b.put(R1, S);
  m.R2 = b.put(R2, S);
  m.R3 = b.put(R3, S);
  m.R4 = b.put(R4, S);
  m.ninv = hebn::neg_inv32(N[0]);
  for (int v = 0; v < he29::kVariants; ++v) {
    if (!(v29 >> v & 1u)) continue;
    const size_t S29 = (size_t)he29::limbs((int)S, v);
    const Limbs Q1 = hebn::mod(pow2(he29::kBits * S29), N);
    m.N29[v] = b.put29(N, S29);
    m.R1_29[v] = b.put29(Q1, S29);
    m.R2_29[v] = b.put29(hebn::mulmod(Q1, Q1, N), S29);
  }
  return m;
}

// The two-digit constants of N (S 32-bit limbs), see radix29.hpp.  X mod N^2
// is the pair (c, d 2^29 mod N) with X = c - d N.  Piece h of an input
// sum_h x_h 2^(32 S h) enters by the product with 2^(32 S h) R^2 mod N^2.
// e: see kPairE.
inline PairOff put_pair(Blob &b, const Limbs &N, size_t S, const Limbs &e) {
  PairOff o;
  o.ninv = hebn::neg_inv32(N[0]);
  const Limbs N2 = hebn::mul(N, N), shift = hebn::mod(pow2(he29::kBits), N);
  for (int v = 0; v < he29::kPairVariants; ++v) {
    const size_t S29 = (size_t)he29::pair_limbs((int)S, v);
    const Limbs R = hebn::mod(pow2(he29::kBits * S29), N2);
    auto put = [&](const Limbs &X) {
      Limbs e, c;
      hebn::divmod(X, N, &e, &c);  // X = c + e N
      const Limbs d = hebn::is_zero(e) ? e : hebn::sub(N, e);
      const size_t at = b.put29(c, S29);
      b.words.resize(at + S29);  // the digits are adjacent
      b.put29(hebn::mulmod(d, shift, N), S29);
      b.words.resize(at + 2 * S29);
    };
    o.c[v] = b.words.size();
    Limbs piece = hebn::mulmod(R, R, N2);
    const Limbs step = hebn::mod(pow2(32 * S), N2);
    for (int h = 0; h < he29::kPairPieces; ++h) {
      put(piece);
      piece = hebn::mulmod(piece, step, N2);
    }
    put(hebn::from_u64(1));
    put(hebn::mod(pow2(he29::kBits * (S29 - 1)), N));
    put(R);
    const Limbs eR = hebn::mulmod(hebn::mod(e, N2), R, N2);
    put(eR);
    put(hebn::mod(hebn::sub(hebn::add(R, N2), eR), N2));
    b.put29(N, S29);
  }
  return o;
}

inline ExpOff put_exp(Blob &b, const Limbs &e, size_t limbs) {
  ExpOff x;
  x.e = b.put(e, limbs, 1);
  const size_t bits = std::max<size_t>(hebn::bit_length(e), 1);
  x.nwin = (int)((bits + kWindowBits - 1) / kWindowBits);
  const std::vector<uint32_t> ops = sliding_schedule(e);
  x.nops = (int)ops.size();
  x.ops = b.words.size();
  b.words.insert(b.words.end(), ops.begin(), ops.end());
  b.words.resize((b.words.size() + 3) & ~size_t(3), 0u);
  return x;
}

inline ExpOff put_joint(Blob &b, const Limbs &f, const Limbs &e) {
  ExpOff x{};
  const std::vector<uint32_t> ops = joint_schedule(f, e);
  x.nops = (int)ops.size();
  x.ops = b.words.size();
  b.words.insert(b.words.end(), ops.begin(), ops.end());
  b.words.resize((b.words.size() + 3) & ~size_t(3), 0u);
  return x;
}

// Constants of prime P (other prime Q) for the CRT paths; S_P limbs per prime.
inline PrimeOff put_prime(Blob &b, const Limbs &P, const Limbs &Q, const Limbs &n, size_t SP) {
  PrimeOff o;
  const Limbs one = hebn::from_u64(1);
  const Limbs P2 = hebn::mul(P, P);
  o.P = put_mod(b, P, SP, 7);
  o.P2 = put_mod(b, P2, 2 * SP, 0);
  const Limbs Pm1 = hebn::sub(P, one), e = hebn::mod(Q, Pm1);
  const Limbs ej = hebn::is_zero(e) ? Pm1 : e;  // x^(P-1) = x^0 mod P
  o.pair = put_pair(b, P, SP, ej);
  o.joint = put_joint(b, Pm1, ej);
  o.e_enc = put_exp(b, e, SP);
  o.e_lift = put_exp(b, P, SP);
  o.e_dec = put_exp(b, Pm1, SP);
  const Limbs RP = hebn::mod(pow2(32 * SP), P);
  const Limbs RP2 = hebn::mod(pow2(64 * SP), P2);
  o.QR_P = b.put(hebn::mulmod(Q, RP, P), SP);
  o.QR2_P = b.put(hebn::mulmod(hebn::mulmod(Q, RP, P), RP, P), SP);
  o.PR_P2 = b.put(hebn::mulmod(P, RP2, P2), 2 * SP);
  o.Pinv = b.put(hebn::inv_pow2(P, 32 * SP), SP);
  // h_P = L_P(g^(P-1) mod P^2)^-1 mod P with g = n + 1, L_P(x) = (x - 1) / P
  const Limbs gp = hebn::powmod(hebn::add(n, one), Pm1, P2);
  Limbs Lp;
  hebn::divmod(hebn::sub(gp, one), P, &Lp, nullptr);
  o.hR_P = b.put(hebn::mulmod(hebn::invmod(Lp, P), RP, P), SP);
  return o;
}

// All constants of a key of n_bits bits (L = n_bits / 32 limbs of n).
inline KeyConsts derive(uint32_t n_bits, const Limbs &n, const Limbs &p, const Limbs &q, bool priv) {
  KeyConsts k;
  const size_t L = n_bits / 32, SP = L / 2;
  const Limbs one = hebn::from_u64(1);
  const Limbs n2 = hebn::mul(n, n);
  Blob &b = k.blob;
  k.n = put_mod(b, n, L, 0);
  k.n2 = put_mod(b, n2, 2 * L, 1u << he29::variant(16));  // the form the histograms take
  k.pair_n = put_pair(b, n, L, Limbs());
  k.e_n = put_exp(b, n, L);
  const Limbs Rn2 = hebn::mod(pow2(64 * L), n2);
  const Limbs Rn = hebn::mod(pow2(32 * L), n);
  k.nR_n2 = b.put(hebn::mulmod(n, Rn2, n2), 2 * L);
  Limbs h = hebn::add(n, one);  // (n + 1) / 2
  for (size_t i = 0; i < h.size(); ++i) h[i] = (h[i] >> 1) | (i + 1 < h.size() ? h[i + 1] << 31 : 0u);
  hebn::norm(h);
  k.half = b.put(h, L);
  if (priv) {
    k.pr[0] = put_prime(b, p, q, n, SP);
    k.pr[1] = put_prime(b, q, p, n, SP);
    const Limbs p2 = hebn::mul(p, p), q2 = hebn::mul(q, q);
    const Limbs Rp2 = hebn::mod(pow2(32 * L), p2);
    k.Cq = b.put(hebn::mulmod(hebn::invmod(q2, p2), Rp2, p2), L);
    k.q2R_n2 = b.put(hebn::mulmod(q2, Rn2, n2), 2 * L);
    k.qinv_p = b.put(hebn::invmod(q, p), SP);
    k.qR_n = b.put(hebn::mulmod(q, Rn, n), L);
  }
  return k;
}

}  // namespace hekey
