// Powers mod N^2 in two digits base N, radix 2^29, for gfx950.
//
// A residue X mod N^2 is held as the pair (a, b) with X = a - b N, both
// digits integers below 2N.  With R = 2^(29 S) the Montgomery product of a
// and c leaves an exact quotient m: a c + m N = R a', so
//   (a - b N)(c - d N) R^-1 = a' - N [(a d + b c + m) R^-1 mod N]   (mod N^2):
// one product and two more, two Montgomery reductions, all of S limbs.  In
// units of S^2 limb products a square costs 1/2 + 1 + 1 + 1 = 3.5 and a product
// 5, where the same residue as one integer of 2S limbs costs 6 and 8.
// The second digit is kept times 2^29 (written be = 2^29 b mod N): then m
// enters its reduction one column late, be' = (a de + be c + 2^29 m) R^-1
// mod N, so both digits' reductions can run side by side, digit i of m being
// handed over after the step that makes it.
//
// Three engines share one exponentiation (power_unit):
//  * LanePair: one integer per lane, both digits in it;
//  * TwinPair: two lanes per integer, one digit each;
//  * GroupPair<G>: G lanes per digit, 2G lanes per integer.
// LanePair and TwinPair sum a product column by column with every limb in
// registers and the modulus, which is the same for the whole wave, in scalar
// registers: no cross-lane step, no LDS and no shift of accumulators, so 84%
// of the instructions are the multiply-adds (GroupPair 75-80% at K = 18).
// LaneMod is the same for plain residues mod N.
// A multiply-add issues every 4.2-4.5 cycles from one wave per SIMD already,
// so what counts is instructions per lane and a wave on every SIMD: the wide
// engines are for batches too small for 64 integers per wave.
//
// Measured (2048-bit key, against the same powers as one integer mod P^2 at 4
// to 16 lanes): 200,000 lifts 131 -> 84 ms, 16,384 decryptions 12.2 -> 8.0 ms,
// 2,006 lifts 4.4 -> 2.6 ms, 2,501 pairs of powers mod n^2 28.5 -> 17.0 ms.
// What bounds it: VALU issue (a LanePair square is 4,630 multiply-adds of 4.2
// cycles, 4,554 of them limb products, the rest hand over quotient digits and
// join wide columns); below a wave per SIMD, the latency of a step.
#pragma once
#include "mont29.hpp"

namespace he {

__device__ __forceinline__ uint64_t mad(uint32_t x, uint32_t y, uint64_t acc) { return (uint64_t)x * y + acc; }
// acc + x P: one instruction where an addition needs x extended to 64
// bits first
template <int P>
__device__ __forceinline__ uint64_t add_mul(uint32_t x, uint64_t acc) {
  uint64_t k;
  asm("v_mad_u64_u32 %0, %1, %2, %3, %0" : "+v"(acc), "=s"(k) : "v"(x), "n"(P));
  return acc;
}
// a 2^s + b: s per lane, or SH
__device__ __forceinline__ uint64_t shl_add(uint64_t a, uint32_t s, uint64_t b) {
  uint64_t r;
  asm("v_lshl_add_u64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(s), "v"(b));
  return r;
}
template <int SH>
__device__ __forceinline__ uint64_t shl_add(uint64_t a, uint64_t b) {
  uint64_t r;
  asm("v_lshl_add_u64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "n"(SH), "v"(b));
  return r;
}
// One column's sum total = P 2^SH + Q, below 2^64 unless `WIDE`: then the part of
// P above its low 29 bits joins the carry instead (carry_wide).  A column of cnt
// limb products each below 2^58 sums to less than cnt 2^58, so the caller sets
// WIDE where the products weighted by 2^SH count 64 or more.
template <bool WIDE, int SH>
__device__ __forceinline__ uint64_t join(uint64_t P, uint64_t Q) {
  if constexpr (WIDE) return add_mul<1 << SH>((uint32_t)P & kMask29, Q);
  else return shl_add<SH>(P, Q);
}
template <bool WIDE, int SH>
__device__ __forceinline__ void carry_wide(uint64_t P, uint64_t &carry) {
  if constexpr (WIDE) carry = shl_add<SH>(P >> he29::kBits, carry);
}

template <int S, int k>
struct Col {
  static constexpr int lo = k < S ? 0 : k - S + 1, hi = k < S ? k : S - 1, cnt = hi - lo + 1;
};

// Ends column k of a reduction: below S its quotient digit q[k], which clears
// the column's low 29 bits; from S on the result's limb k - S.
template <int S, int k>
__device__ __forceinline__ uint32_t end_col(uint64_t low, uint32_t (&q)[S], const uint32_t (&n)[S], uint32_t ninv,
                                            uint64_t &carry) {
  uint32_t r = 0;
  if constexpr (k < S) {
    q[k] = ((uint32_t)low * ninv) & kMask29;
    low = mad(q[k], n[0], low);
  } else {
    r = (uint32_t)low & kMask29;
  }
  carry = low >> he29::kBits;
  return r;
}

// Vectors of 4 (2) words: word w of an operand at p + (w / V) vs + w % V.
template <int S>
constexpr int kVec = S % 4 == 0 ? 4 : 2;
template <int S>
__device__ __forceinline__ void ldv(uint32_t (&x)[S], const uint32_t *p, uint32_t vs) {
#pragma unroll
  for (int w = 0; w < S; w += kVec<S>) {
    if constexpr (kVec<S> == 4) {
      const uint4 v = *reinterpret_cast<const uint4 *>(p);
      x[w] = v.x; x[w + 1] = v.y; x[w + 2] = v.z; x[w + 3] = v.w;
    } else {
      const uint2 v = *reinterpret_cast<const uint2 *>(p);
      x[w] = v.x; x[w + 1] = v.y;
    }
    p += vs;
  }
}
template <int S>
__device__ __forceinline__ void stv(uint32_t *p, const uint32_t (&x)[S], uint32_t vs) {
#pragma unroll
  for (int w = 0; w < S; w += kVec<S>) {
    if constexpr (kVec<S> == 4)
      *reinterpret_cast<uint4 *>(p) = make_uint4(x[w], x[w + 1], x[w + 2], x[w + 3]);
    else
      *reinterpret_cast<uint2 *>(p) = make_uint2(x[w], x[w + 1]);
    p += vs;
  }
}

// SN 32-bit limbs at p (16-byte aligned) <-> S limbs of 29 bits in this lane.
template <int SN, int S>
__device__ __forceinline__ void lane_to29(uint32_t (&t)[S], const uint32_t *p) {
  uint32_t w[SN];
  ldv<SN>(w, p, 4);
#pragma unroll
  for (int j = 0; j < S; ++j) {
    const int bit = he29::kBits * j, i = bit >> 5, o = bit & 31;
    const uint32_t lo = i < SN ? w[i < SN ? i : 0] : 0u, hi = i + 1 < SN ? w[i + 1 < SN ? i + 1 : 0] : 0u;
    t[j] = (o ? (lo >> o) | (hi << (32 - o)) : lo) & kMask29;
  }
}
template <int SN, int S>
__device__ __forceinline__ void lane_to32(uint32_t *p, const uint32_t (&t)[S]) {
  uint32_t w[SN];
#pragma unroll
  for (int j = 0; j < SN; ++j) {
    const int bit = 32 * j, i = bit / he29::kBits, o = bit % he29::kBits;
    w[j] = (t[i] >> o) | (i + 1 < S ? t[i + 1 < S ? i + 1 : 0] << (he29::kBits - o) : 0u);
    if (2 * he29::kBits - o < 32 && i + 2 < S) w[j] |= t[i + 2 < S ? i + 2 : 0] << (2 * he29::kBits - o);
  }
  stv<SN>(p, w, 4);
}
// t mod N for t <= 2N - 1 with limbs below 2^29; true if N was subtracted.
template <int S>
__device__ __forceinline__ bool lane_canon(uint32_t (&t)[S], const uint32_t (&n)[S]) {
  uint32_t d[S], b = 0;
#pragma unroll
  for (int j = 0; j < S; ++j) {
    const uint32_t s = t[j] - n[j] - b;
    d[j] = s & kMask29;
    b = s >> 31;
  }
#pragma unroll
  for (int j = 0; j < S; ++j) t[j] = b ? t[j] : d[j];
  return b == 0;
}
// t = (f - t) mod N for t in [0, N), f in {0, 1}.
template <int S>
__device__ __forceinline__ void lane_neg(uint32_t (&t)[S], const uint32_t (&n)[S], uint32_t f) {
  uint32_t c = f;  // N - t + f, carries in {0, 1, -1} as the sign of an int
#pragma unroll
  for (int j = 0; j < S; ++j) {
    const uint32_t s = n[j] - t[j] + c;
    t[j] = s & kMask29;
    c = (uint32_t)((int32_t)s >> he29::kBits);
  }
  lane_canon<S>(t, n);
}

// What an engine is made from: the key's constants of N (radix29.hpp) and
// this wave's table, kTable + 1 slots.
struct UnitArgs {
  const uint32_t *consts;
  uint32_t ninv;  // -N^-1 mod 2^32
  uint32_t *tab;
};

// ------------------------------------------------- one integer per lane
template <int SN>
struct LanePair {
  static constexpr int kLanes = 1, S = he29::pair_limbs(SN, 0), V = kVec<S>;
  static constexpr uint32_t kSlot = 2 * S * 64;  // words of a table slot of the wave
  static constexpr int kLds = 0, kDigits = 2;
  uint32_t n[S], ninv, a[S], b[S], c[S], d[S];
  const uint32_t *k;
  uint32_t *tab;

  __device__ __forceinline__ LanePair(const UnitArgs &u, uint32_t *, uint32_t *) : ninv(u.ninv), k(u.consts), tab(u.tab) {
#pragma unroll
    for (int j = 0; j < S; ++j) n[j] = __builtin_amdgcn_readfirstlane(k[2 * he29::kPairN * S + j]);
  }
  static __device__ __forceinline__ uint32_t member() { return lane_id(); }
  __device__ __forceinline__ uint32_t *slot(uint32_t e) const { return tab + e * kSlot + lane_id() * V; }
  __device__ __forceinline__ void load_piece(const uint32_t *p) {
    lane_to29<SN, S>(a, p);
#pragma unroll
    for (int j = 0; j < S; ++j) b[j] = 0;
  }
  __device__ __forceinline__ void store(uint32_t e) const {
    stv<S>(slot(e), a, 64 * V);
    stv<S>(slot(e) + S * 64, b, 64 * V);
  }
  __device__ __forceinline__ void load(uint32_t e) {
    ldv<S>(a, slot(e), 64 * V);
    ldv<S>(b, slot(e) + S * 64, 64 * V);
  }
  __device__ __forceinline__ void load_const(int e) {
    ldv<S>(a, k + 2 * e * S, V);
    ldv<S>(b, k + (2 * e + 1) * S, V);
  }
  // the state in one set of registers at this point, whichever way it came here
  // (left to the compiler, a product held copies and spilled: 40 to 700 words)
  __device__ __forceinline__ void pin() {
#pragma unroll
    for (int j = 0; j < S; ++j) asm volatile("" : "+v"(a[j]), "+v"(b[j]));
  }
  // the state becomes the operand and slot e the state; back() undoes the first
  __device__ __forceinline__ void turn(uint32_t e) {
#pragma unroll
    for (int j = 0; j < S; ++j) {
      c[j] = a[j];
      d[j] = b[j];
    }
    load(e);
  }
  __device__ __forceinline__ void back() {
#pragma unroll
    for (int j = 0; j < S; ++j) {
      a[j] = c[j];
      b[j] = d[j];
    }
  }
  // the operand of the next product: a table slot or a constant pair
  __device__ __forceinline__ void fetch(uint32_t e, bool constant = false) {
    const uint32_t *p = constant ? k + 2 * e * S : slot(e);
    const uint32_t vs = constant ? V : 64 * V;
    ldv<S>(c, p, vs);
    ldv<S>(d, p + (constant ? S : S * 64), vs);
  }
  // every slot below kTable is read, the wanted one kept by a mask
  __device__ __forceinline__ void fetch_masked(uint32_t digit) {
    uint32_t dv = digit;
    asm volatile("" : "+v"(dv));
#pragma unroll
    for (int j = 0; j < S; ++j) c[j] = d[j] = 0u;
#pragma unroll 1
    for (uint32_t e = 0; e < (uint32_t)kTable; ++e) {
      const uint32_t m = dv == e ? 0xFFFFFFFFu : 0u;
      uint32_t t[S];
      ldv<S>(t, slot(e), 64 * V);
#pragma unroll
      for (int j = 0; j < S; ++j) c[j] |= t[j] & m;
      ldv<S>(t, slot(e) + S * 64, 64 * V);
#pragma unroll
      for (int j = 0; j < S; ++j) d[j] |= t[j] & m;
    }
  }
  // digits += those of slot e (sums below 4N; a carry pass keeps 29-bit limbs)
  __device__ __forceinline__ void add(uint32_t e) {
    fetch(e);
    uint32_t ca = 0, cb = 0;
#pragma unroll
    for (int j = 0; j < S; ++j) {
      ca += a[j] + c[j];
      cb += b[j] + d[j];
      a[j] = ca & kMask29;
      b[j] = cb & kMask29;
      ca >>= he29::kBits;
      cb >>= he29::kBits;
    }
  }
  __device__ __forceinline__ void sq() {
    uint32_t q[S], p[S];
    uint64_t ca = 0, cb = 0;
    static_for<0, 2 * S - 1>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      using C = Col<S, k>;
      constexpr bool wide1 = 2 * C::cnt >= 64, wide2 = 3 * C::cnt >= 63;
      uint64_t Q = ca, P = 0, Q2 = cb, P2 = 0;
      static_for<C::lo, C::hi + 1>([&](auto ic) {
        constexpr int i = decltype(ic)::value, j = k - i;
        if constexpr (i < j) P = mad(a[i], a[j], P);
        if constexpr (k >= S || i < k) Q = mad(q[i], n[j], Q);
        if constexpr (i == j) Q = mad(a[i], a[i], Q);
      });
      const uint32_t ra = end_col<S, k>(join<wide1, 1>(P, Q), q, n, ninv, ca);
      carry_wide<wide1, 1>(P, ca);
      if constexpr (k >= 1 && k <= S) Q2 = add_mul<1>(q[k >= 1 && k <= S ? k - 1 : 0], Q2);
      static_for<C::lo, C::hi + 1>([&](auto ic) {
        constexpr int i = decltype(ic)::value, j = k - i;
        P2 = mad(a[i], b[j], P2);
        if constexpr (k >= S || i < k) Q2 = mad(p[i], n[j], Q2);
      });
      const uint32_t rb = end_col<S, k>(join<wide2, 1>(P2, Q2), p, n, ninv, cb);
      carry_wide<wide2, 1>(P2, cb);
      if constexpr (k >= S) {
        a[k - S] = ra;
        b[k - S] = rb;
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    a[S - 1] = (uint32_t)ca;
    b[S - 1] = (uint32_t)cb;
  }
  __device__ __forceinline__ void mul() {
    uint32_t q[S], p[S];
    uint64_t ca = 0, cb = 0;
    static_for<0, 2 * S - 1>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      using C = Col<S, k>;
      constexpr bool wide = 3 * C::cnt >= 63;
      constexpr bool wide1 = 2 * C::cnt >= 64;
      uint64_t Q = ca, P = 0, Q2 = cb, P2 = 0, P3 = 0;
      static_for<C::lo, C::hi + 1>([&](auto ic) {
        constexpr int i = decltype(ic)::value, j = k - i;
        P = mad(a[i], c[j], P);
        if constexpr (k >= S || i < k) Q = mad(q[i], n[j], Q);
      });
      const uint32_t ra = end_col<S, k>(join<wide1, 0>(P, Q), q, n, ninv, ca);
      carry_wide<wide1, 0>(P, ca);
      if constexpr (k >= 1 && k <= S) Q2 = add_mul<1>(q[k >= 1 && k <= S ? k - 1 : 0], Q2);
      static_for<C::lo, C::hi + 1>([&](auto ic) {
        constexpr int i = decltype(ic)::value, j = k - i;
        P2 = mad(a[i], d[j], P2);
        P3 = mad(b[i], c[j], P3);
        if constexpr (k >= S || i < k) Q2 = mad(p[i], n[j], Q2);
      });
      const uint32_t rb = end_col<S, k>(join<wide, 0>(P3, join<wide, 0>(P2, Q2)), p, n, ninv, cb);
      carry_wide<wide, 0>(P2, cb);
      carry_wide<wide, 0>(P3, cb);
      if constexpr (k >= S) {
        a[k - S] = ra;
        b[k - S] = rb;
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    a[S - 1] = (uint32_t)ca;
    b[S - 1] = (uint32_t)cb;
  }
  // a kept in slot 0, then (b, 0) in its place
  __device__ __forceinline__ void second() {
#pragma unroll
    for (int j = 0; j < S; ++j) {
      a[j] = b[j];
      b[j] = 0;
    }
  }
  // X = a - b N in [0, N^2) as a + e N: a from slot 0, b in a
  __device__ __forceinline__ void out(uint32_t *o, bool valid) {
    ldv<S>(c, slot(0), 64 * V);
    const bool sub = lane_canon<S>(c, n);
    lane_canon<S>(a, n);
    lane_neg<S>(a, n, sub ? 1u : 0u);
    if (valid) {
      lane_to32<SN, S>(o, c);
      lane_to32<SN, S>(o + SN, a);
    }
  }
};

// ------------------------------------------------- one residue mod N per lane
template <int SN>
struct LaneMod {
  static constexpr int kLanes = 1, S = he29::pair_limbs(SN, 0), V = kVec<S>;
  static constexpr uint32_t kSlot = S * 64;
  static constexpr int kLds = 0, kDigits = 1;
  uint32_t n[S], ninv, a[S], c[S];
  const uint32_t *k;
  uint32_t *tab;

  __device__ __forceinline__ LaneMod(const UnitArgs &u, uint32_t *, uint32_t *) : ninv(u.ninv), k(u.consts), tab(u.tab) {
#pragma unroll
    for (int j = 0; j < S; ++j) n[j] = __builtin_amdgcn_readfirstlane(k[2 * he29::kPairN * S + j]);
  }
  static __device__ __forceinline__ uint32_t member() { return lane_id(); }
  __device__ __forceinline__ uint32_t *slot(uint32_t e) const { return tab + e * kSlot + lane_id() * V; }
  __device__ __forceinline__ void load_piece(const uint32_t *p) { lane_to29<SN, S>(a, p); }
  __device__ __forceinline__ void store(uint32_t e) const { stv<S>(slot(e), a, 64 * V); }
  __device__ __forceinline__ void load(uint32_t e) { ldv<S>(a, slot(e), 64 * V); }
  __device__ __forceinline__ void load_const(int e) { ldv<S>(a, k + 2 * e * S, V); }
  __device__ __forceinline__ void fetch(uint32_t e, bool constant = false) {
    ldv<S>(c, constant ? k + 2 * e * S : slot(e), constant ? V : 64 * V);
  }
  __device__ __forceinline__ void fetch_masked(uint32_t digit) {
    uint32_t dv = digit;
    asm volatile("" : "+v"(dv));
#pragma unroll
    for (int j = 0; j < S; ++j) c[j] = 0u;
#pragma unroll 1
    for (uint32_t e = 0; e < (uint32_t)kTable; ++e) {
      uint32_t t[S];
      ldv<S>(t, slot(e), 64 * V);
      const uint32_t m = dv == e ? 0xFFFFFFFFu : 0u;
#pragma unroll
      for (int j = 0; j < S; ++j) c[j] |= t[j] & m;
    }
  }
  __device__ __forceinline__ void add(uint32_t) {}
  __device__ __forceinline__ void second() {}
  template <bool SQ>
  __device__ __forceinline__ void product() {
    uint32_t q[S];
    uint64_t ca = 0;
    static_for<0, 2 * S - 1>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      using C = Col<S, k>;
      constexpr bool wide = 2 * C::cnt >= 64;
      constexpr int sh = SQ ? 1 : 0;
      uint64_t Q = ca, P = 0;
      static_for<C::lo, C::hi + 1>([&](auto ic) {
        constexpr int i = decltype(ic)::value, j = k - i;
        if constexpr (!SQ) P = mad(a[i], c[j], P);
        if constexpr (SQ && i < j) P = mad(a[i], a[j], P);
        if constexpr (k >= S || i < k) Q = mad(q[i], n[j], Q);
        if constexpr (SQ && i == j) Q = mad(a[i], a[i], Q);
      });
      const uint32_t r = end_col<S, k>(join<wide, sh>(P, Q), q, n, ninv, ca);
      carry_wide<wide, sh>(P, ca);
      if constexpr (k >= S) a[k - S] = r;
      __builtin_amdgcn_sched_barrier(0);
    });
    a[S - 1] = (uint32_t)ca;
  }
  __device__ __forceinline__ void sq() { product<true>(); }
  __device__ __forceinline__ void mul() { product<false>(); }
  __device__ __forceinline__ void out(uint32_t *o, bool valid) {
    lane_canon<S>(a, n);
    if (valid) lane_to32<SN, S>(o, a);
  }
};

// ------------------------------------------------- one digit per lane
// Even lanes hold a, odd lanes be; x is a in both.
template <int SN>
struct TwinPair {
  static constexpr int kLanes = 2, S = he29::pair_limbs(SN, 0), V = kVec<S>;
  static constexpr uint32_t kSlot = S * 64;
  static constexpr int kLds = 0, kDigits = 2;
  uint32_t n[S], ninv, x[S], r[S], y[S], z[S];  // y: own digit of the operand, z: its first digit
  const uint32_t *k;
  uint32_t *tab;
  uint32_t odd, hand;  // 1 and 2^29 - 1 in odd lanes

  __device__ __forceinline__ TwinPair(const UnitArgs &u, uint32_t *, uint32_t *) : ninv(u.ninv), k(u.consts), tab(u.tab) {
#pragma unroll
    for (int j = 0; j < S; ++j) n[j] = __builtin_amdgcn_readfirstlane(k[2 * he29::kPairN * S + j]);
    odd = lane_id() & 1u;
    hand = odd ? kMask29 : 0u;
    asm volatile("" : "+v"(odd), "+v"(hand));
  }
  static __device__ __forceinline__ uint32_t member() { return lane_id() >> 1; }
  __device__ __forceinline__ uint32_t *slot(uint32_t e) const { return tab + e * kSlot + lane_id() * V; }
  __device__ __forceinline__ uint32_t *slot_first(uint32_t e) const { return tab + e * kSlot + (lane_id() & ~1u) * V; }
  // x from the even lane's r
  __device__ __forceinline__ void share() {
#pragma unroll
    for (int j = 0; j < S; ++j) x[j] = bcast_first<2>(r[j]);
  }
  __device__ __forceinline__ void load_piece(const uint32_t *p) {
    lane_to29<SN, S>(x, p);
#pragma unroll
    for (int j = 0; j < S; ++j) r[j] = odd ? 0u : x[j];
  }
  __device__ __forceinline__ void store(uint32_t e) const {
    stv<S>(slot(e), r, 64 * V);
    __threadfence_block();
  }
  __device__ __forceinline__ void load(uint32_t e) {
    ldv<S>(r, slot(e), 64 * V);
    share();
  }
  __device__ __forceinline__ void load_const(int e) {
    ldv<S>(r, k + (2 * e + odd) * S, V);
    share();
  }
  __device__ __forceinline__ void turn(uint32_t e) {
#pragma unroll
    for (int j = 0; j < S; ++j) {
      y[j] = r[j];
      z[j] = x[j];
    }
    load(e);
  }
  __device__ __forceinline__ void back() {
#pragma unroll
    for (int j = 0; j < S; ++j) {
      r[j] = y[j];
      x[j] = z[j];
    }
  }
  __device__ __forceinline__ void pin() {
#pragma unroll
    for (int j = 0; j < S; ++j) asm volatile("" : "+v"(x[j]), "+v"(r[j]));
  }
  __device__ __forceinline__ void fetch(uint32_t e, bool constant = false) {
    const uint32_t vs = constant ? V : 64 * V;
    ldv<S>(y, constant ? k + (2 * e + odd) * S : slot(e), vs);
    ldv<S>(z, constant ? k + 2 * e * S : slot_first(e), vs);
  }
  __device__ __forceinline__ void fetch_masked(uint32_t digit) {
    uint32_t dv = digit;
    asm volatile("" : "+v"(dv));
#pragma unroll
    for (int j = 0; j < S; ++j) y[j] = 0u;
#pragma unroll 1
    for (uint32_t e = 0; e < (uint32_t)kTable; ++e) {
      uint32_t t[S];
      ldv<S>(t, slot(e), 64 * V);
      const uint32_t m = dv == e ? 0xFFFFFFFFu : 0u;
#pragma unroll
      for (int j = 0; j < S; ++j) y[j] |= t[j] & m;
    }
#pragma unroll
    for (int j = 0; j < S; ++j) z[j] = bcast_first<2>(y[j]);
  }
  __device__ __forceinline__ void add(uint32_t e) {
    ldv<S>(y, slot(e), 64 * V);
    uint32_t c = 0;
#pragma unroll
    for (int j = 0; j < S; ++j) {
      c += r[j] + y[j];
      r[j] = c & kMask29;
      c >>= he29::kBits;
    }
    share();
  }
  // the even lane's quotient digit, in the odd lane (0 in the even one)
  __device__ __forceinline__ uint32_t handed(uint32_t q) const { return bcast_first<2>(q) & hand; }
  __device__ __forceinline__ void sq() {
    uint32_t q[S];
    uint64_t c = 0;
    static_for<0, 2 * S - 1>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      using C = Col<S, k>;
      constexpr bool wide = 3 * C::cnt >= 63;
      uint64_t Q = c, P = 0;
      if constexpr (k >= 1 && k <= S) Q += handed(q[k >= 1 && k <= S ? k - 1 : 0]);
      static_for<C::lo, C::hi + 1>([&](auto ic) {
        constexpr int i = decltype(ic)::value, j = k - i;
        P = mad(x[i], r[j], P);
        if constexpr (k >= S || i < k) Q = mad(q[i], n[j], Q);
      });
      const uint64_t low = shl_add(wide ? (uint64_t)((uint32_t)P & kMask29) : P, odd, Q);
      const uint64_t high = wide ? shl_add(P >> he29::kBits, odd, 0) : 0;
      const uint32_t t = end_col<S, k>(low, q, n, ninv, c);
      if constexpr (wide) c += high;
      asm("" : "+v"(c));  // the columns stay apart (one wave per SIMD: 3% over letting the compiler merge them)
      if constexpr (k >= S) r[k - S] = t;
      __builtin_amdgcn_sched_barrier(0);
    });
    r[S - 1] = (uint32_t)c;
    share();
  }
  __device__ __forceinline__ void mul() {
    uint32_t q[S];
    uint64_t c = 0;
#pragma unroll
    for (int j = 0; j < S; ++j) r[j] = odd ? r[j] : 0u;
    static_for<0, 2 * S - 1>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      using C = Col<S, k>;
      constexpr bool wide = 3 * C::cnt >= 63;
      uint64_t Q = c, P = 0, P2 = 0;
      if constexpr (k >= 1 && k <= S) Q += handed(q[k >= 1 && k <= S ? k - 1 : 0]);
      static_for<C::lo, C::hi + 1>([&](auto ic) {
        constexpr int i = decltype(ic)::value, j = k - i;
        P = mad(x[i], y[j], P);
        P2 = mad(r[i], z[j], P2);
        if constexpr (k >= S || i < k) Q = mad(q[i], n[j], Q);
      });
      uint64_t low = Q, high = 0;
      if constexpr (wide) {
        low = shl_add<0>((uint32_t)P2 & kMask29, shl_add<0>((uint32_t)P & kMask29, Q));
        high = shl_add<0>(P2 >> he29::kBits, P >> he29::kBits);
      } else {
        low = shl_add<0>(P2, shl_add<0>(P, Q));
      }
      const uint32_t t = end_col<S, k>(low, q, n, ninv, c);
      if constexpr (wide) c += high;
      asm("" : "+v"(c));  // the columns stay apart (one wave per SIMD: 3% over letting the compiler merge them)
      if constexpr (k >= S) r[k - S] = t;
      __builtin_amdgcn_sched_barrier(0);
    });
    r[S - 1] = (uint32_t)c;
    share();
  }
  __device__ __forceinline__ void second() {
#pragma unroll
    for (int j = 0; j < S; ++j) {
      x[j] = (uint32_t)__builtin_amdgcn_mov_dpp((int)r[j], 0xF5, 0xF, 0xF, false);  // quad_perm [1,1,3,3]
      r[j] = odd ? 0u : x[j];
    }
  }
  __device__ __forceinline__ void out(uint32_t *o, bool valid) {
    ldv<S>(z, slot_first(0), 64 * V);
    const bool sub = lane_canon<S>(z, n);
    lane_canon<S>(x, n);
    lane_neg<S>(x, n, sub ? 1u : 0u);
#pragma unroll
    for (int j = 0; j < S; ++j) x[j] = odd ? x[j] : z[j];
    if (valid) lane_to32<SN, S>(o + odd * SN, x);
  }
};

// ------------------------------------------------- G lanes per digit
// Lanes 0..G-1 of an integer's 2G hold a, the others be, K limbs each.  The
// steps are mont29.hpp's (one multiplier limb and one quotient digit per
// step, accumulators shifted down one limb); limbs are settled, not exact.
template <int SN, int G>
struct GroupPair {
  static constexpr int kLanes = 2 * G, S = he29::pair_limbs(SN, he29::pair_variant(G)), K = S / G, K32 = SN / G;
  static constexpr uint32_t kSlot = 2 * S * (64 / kLanes);
  static constexpr int SR = (S + 3) / 4 * 4;  // 16-byte aligned second row for the limb conversions
  static constexpr int kLds = 2 * SR, kDigits = 2;  // LDS words per integer: both digits
  static constexpr int U = K % 2 == 0 ? K : 2 * K;  // steps per loop iteration (even)
  static_assert(K >= 2 && K <= 21 && S % U == 0, "column bound: 3 K products of 2^58");
  Mod29<K> M;
  uint32_t r[K], y[K], z[K];
  const uint32_t *k;
  uint32_t *tab, *lds, *zeros;
  uint32_t second_digit, hand;

  __device__ __forceinline__ GroupPair(const UnitArgs &u, uint32_t *row, uint32_t *zero_row)
      : k(u.consts), lds(row), zeros(zero_row) {
    ld29<K, G>(M.n, k + 2 * he29::kPairN * S);
    M.ninv = u.ninv & kMask29;
    M.mask = mask_vgpr();
    tab = u.tab + (lane_id() / kLanes) * 2 * S;
    second_digit = lane_id() & (uint32_t)G;
    hand = (lane_id() & (uint32_t)(kLanes - 1)) == (uint32_t)G ? kMask29 : 0u;
    asm volatile("" : "+v"(second_digit), "+v"(hand));
  }
  static __device__ __forceinline__ uint32_t member() { return lane_id() / kLanes; }
  __device__ __forceinline__ uint32_t *slot(uint32_t e) const { return tab + e * kSlot; }
  __device__ __forceinline__ uint32_t *digit_row() const { return lds + (second_digit ? SR : 0); }
  __device__ __forceinline__ void load_piece(const uint32_t *p) {
    uint32_t w[K32];
    ld<K32, G>(w, p);
    to29<K32, K, G>(r, w, digit_row());
#pragma unroll
    for (int j = 0; j < K; ++j) r[j] = second_digit ? 0u : r[j];
  }
  __device__ __forceinline__ void store(uint32_t e) const {
    st29<K, 2 * G>(slot(e), r);
    __threadfence_block();
  }
  __device__ __forceinline__ void load(uint32_t e) { ld29<K, 2 * G>(r, slot(e)); }
  __device__ __forceinline__ void load_const(int e) { ld29<K, 2 * G>(r, k + 2 * e * S); }
  // (the first digit's lanes take no part of z: their multiplier row is zeros)
  __device__ __forceinline__ void turn(uint32_t e) {
#pragma unroll
    for (int j = 0; j < K; ++j) {
      y[j] = r[j];
      z[j] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)r[j], 0x110 + G, 0xF, 0xF, true);  // row_shr:G
    }
    load(e);
  }
  __device__ __forceinline__ void back() {
#pragma unroll
    for (int j = 0; j < K; ++j) r[j] = y[j];
  }
  __device__ __forceinline__ void pin() {}
  __device__ __forceinline__ void fetch(uint32_t e, bool constant = false) {
    const uint32_t *p = constant ? k + 2 * e * S : slot(e);
    ld29<K, 2 * G>(y, p);
    ld29<K, G>(z, p);
  }
  __device__ __forceinline__ void fetch_masked(uint32_t digit) {
    uint32_t dv = digit;
    asm volatile("" : "+v"(dv));
#pragma unroll
    for (int j = 0; j < K; ++j) y[j] = z[j] = 0u;
#pragma unroll 1
    for (uint32_t e = 0; e < (uint32_t)kTable; ++e) {
      const uint32_t m = dv == e ? 0xFFFFFFFFu : 0u;
      uint32_t t[K];
      ld29<K, 2 * G>(t, slot(e));
#pragma unroll
      for (int j = 0; j < K; ++j) y[j] |= t[j] & m;
      ld29<K, G>(t, slot(e));
#pragma unroll
      for (int j = 0; j < K; ++j) z[j] |= t[j] & m;
    }
  }
  __device__ __forceinline__ void add(uint32_t e) {
    uint32_t t[K];
    uint64_t C[K];
    ld29<K, 2 * G>(t, slot(e));
#pragma unroll
    for (int j = 0; j < K; ++j) C[j] = (uint64_t)r[j] + t[j];
    settle29<K, G>(r, C);
  }
  // The reduction's part of a step: the quotient digit of the lowest column,
  // the shift by one limb and (HAND) the first digit's q into the second's
  // next column.
  template <bool HAND>
  __device__ __forceinline__ void reduce_step(uint64_t (&C)[K], uint32_t &top) const {
    const uint32_t q = bcast_first_m29<G>(mul_lo32((uint32_t)C[0], M.ninv), M.mask);
#pragma unroll
    for (int j = 0; j < K; ++j) C[j] += (uint64_t)q * M.n[j];
    top = rotate_next_m29<G>((uint32_t)C[0], M.mask);
    C[1] += C[0] >> he29::kBits;
    if constexpr (HAND) {
      // the first digit's q, in the second digit's first lane
      const uint32_t h = (uint32_t)__builtin_amdgcn_mov_dpp((int)q, 0x111, 0xF, 0xF, true) & hand;
      uint64_t kk;
      asm("v_mad_u64_u32 %0, %1, %2, 1, %0" : "+v"(C[1]), "=s"(kk) : "v"(h));
    }
#pragma unroll
    for (int j = 0; j + 1 < K; ++j) C[j] = C[j + 1];
#pragma unroll
    for (int j = 0; j + 1 < K; ++j) asm("" : "+v"(C[j]));
    asm("" : "+v"(top));
  }
  // r = (u Y + v Z + q n, ...) over all steps: u the first digit's limbs, v
  // (TWO) this lane's second multiplier row (zeros in the first digit's lanes)
  template <bool TWO>
  __device__ __forceinline__ void steps(const uint32_t (&Y)[K]) {
    st29<K, 2 * G>(lds, r);
    __builtin_amdgcn_wave_barrier();
    const uint32_t *row = lds;
    const int voff = second_digit ? S : (int)(zeros - lds);
    uint64_t C[K];
    uint32_t top = 0;
#pragma unroll
    for (int j = 0; j < K; ++j) C[j] = 0;
#pragma unroll 1
    for (int i0 = 0; i0 < S; i0 += U) {
      // multiplier limbs two at a time, read one pair ahead of their steps
      uint2 u2, v2, un = *reinterpret_cast<const uint2 *>(row + i0), vn;
      if constexpr (TWO) vn = *reinterpret_cast<const uint2 *>(row + voff + i0);
      static_for<0, U>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        if constexpr (s % 2 == 0) {
          if constexpr (s > 0) __builtin_amdgcn_sched_barrier(0);
          u2 = un;
          if constexpr (TWO) v2 = vn;
          if constexpr (s + 2 < U) {
            un = *reinterpret_cast<const uint2 *>(row + i0 + s + 2);
            if constexpr (TWO) vn = *reinterpret_cast<const uint2 *>(row + voff + i0 + s + 2);
          }
        }
        const uint32_t u = s % 2 == 0 ? u2.x : u2.y;
#pragma unroll
        for (int j = 0; j + 1 < K; ++j) C[j] += (uint64_t)u * Y[j];
        C[K - 1] = (uint64_t)top + (uint64_t)u * Y[K - 1];
        if constexpr (TWO) {
          const uint32_t v = s % 2 == 0 ? v2.x : v2.y;
          // opaque between the two products, or they are summed apart first
#pragma unroll
          for (int j = 0; j < K; ++j) asm("" : "+v"(C[j]));
#pragma unroll
          for (int j = 0; j < K; ++j) C[j] += (uint64_t)v * z[j];
        }
        reduce_step<true>(C, top);
      });
    }
    C[K - 1] = top;
    settle29<K, G>(r, C);
    __builtin_amdgcn_wave_barrier();
  }
  __device__ __forceinline__ void sq() {
    uint32_t t[K];
    const uint32_t sh = second_digit ? 1u : 0u;
#pragma unroll
    for (int j = 0; j < K; ++j) t[j] = r[j] << sh;
    steps<false>(t);
  }
  __device__ __forceinline__ void mul() { steps<true>(y); }
  __device__ __forceinline__ void second() {
    st29<K, 2 * G>(lds, r);
    __builtin_amdgcn_wave_barrier();
    ld29<K, G>(r, lds + S);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < K; ++j) r[j] = second_digit ? 0u : r[j];
  }
  // d = (f - t) mod N for t in [0, N): N - t + f, a borrow pass in the lane and
  // one across the group
  __device__ __forceinline__ void negate(uint32_t (&d)[K], const uint32_t (&t)[K], bool f) const {
    uint32_t b = 0;
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const uint32_t s = M.n[j] - t[j] - b;
      d[j] = s & kMask29;
      b = s >> 31;
    }
    bool zp = true;
#pragma unroll
    for (int j = 0; j < K; ++j) zp = zp && d[j] == 0u;
    uint32_t bi = carry_in<G>(b != 0u, zp) ? 1u : 0u;
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const uint32_t s = d[j] - bi;
      d[j] = s & kMask29;
      bi = s >> 31;
    }
    if (glane<G>() == 0 && f) d[0] += 1u;
    canon29<K, G>(d, M);
  }
  // X of the pair of X R, canonical mod N^2, as 2 SN 32-bit limbs at o.  Two
  // reductions side by side leave the Montgomery form (no product), one more
  // step divides the second digit by 2^29, and a + e N is one plain product.
  __device__ __forceinline__ void finish(uint32_t *o, bool valid) {
    uint64_t C[K];
    uint32_t top = r[K - 1], t[K], e[K];
#pragma unroll
    for (int j = 0; j < K; ++j) C[j] = r[j];
#pragma unroll 1
    for (int i = 0; i < S; ++i) {
      C[K - 1] = top;
      reduce_step<true>(C, top);
    }
    C[K - 1] = top;
    settle29<K, G>(r, C);
#pragma unroll
    for (int j = 0; j < K; ++j) C[j] = r[j];
    top = r[K - 1];
    reduce_step<false>(C, top);
    C[K - 1] = top;
    settle29<K, G>(t, C);
#pragma unroll
    for (int j = 0; j < K; ++j) r[j] = second_digit ? t[j] : r[j];
    const bool sub = canon29<K, G>(r, M);
    // the first digit's subtraction, in the second digit's lanes
    const uint32_t f = (uint32_t)__builtin_amdgcn_update_dpp(0, sub ? 1 : 0, 0x110 + G, 0xF, 0xF, true);
    negate(e, r, f != 0u);
#pragma unroll
    for (int j = 0; j < K; ++j) t[j] = second_digit ? e[j] : r[j];
    st29<K, 2 * G>(lds, t);
    __builtin_amdgcn_wave_barrier();
    const bool first_lane = (lane_id() & (uint32_t)(kLanes - 1)) == 0;
#pragma unroll
    for (int j = 0; j < K; ++j) C[j] = r[j];
    top = r[K - 1];
#pragma unroll 1
    for (int i = 0; i < S; ++i) {
      const uint32_t u = lds[S + i];
      C[K - 1] = top;
#pragma unroll
      for (int j = 0; j < K; ++j) C[j] += (uint64_t)u * M.n[j];
      const uint32_t low = (uint32_t)C[0] & kMask29;
      if (first_lane) lds[i] = low;  // limb i of the result
      top = from_next<G>(low);
      C[1] += C[0] >> he29::kBits;
#pragma unroll
      for (int j = 0; j + 1 < K; ++j) C[j] = C[j + 1];
    }
    C[K - 1] = top;
    settle29<K, G>(t, C);
    carry29<K, G>(t);
    __builtin_amdgcn_wave_barrier();
    if (!second_digit) {
#pragma unroll
      for (int j = 0; j < K; ++j) lds[S + glane<G>() * K + j] = t[j];
    }
    __builtin_amdgcn_wave_barrier();
    constexpr int W = 2 * SN / kLanes;
    uint32_t w[W];
#pragma unroll
    for (int j = 0; j < W; ++j) {
      const uint32_t bit = 32u * (glane<2 * G>() * W + j);
      const uint32_t k0 = bit / he29::kBits, sh = bit % he29::kBits;
      const uint64_t l0 = lds[k0], l1 = k0 + 1 < 2 * S ? lds[k0 + 1] : 0u, l2 = k0 + 2 < 2 * S ? lds[k0 + 2] : 0u;
      w[j] = (uint32_t)((l0 | (l1 << he29::kBits) | (l2 << (2 * he29::kBits))) >> sh);
    }
    __builtin_amdgcn_wave_barrier();
    if (valid) st<W, 2 * G>(o, w);
  }
  __device__ __forceinline__ void out(uint32_t *o, bool valid) {
    // valid in the first digit's lanes; the others compute along
    ld29<K, G>(z, slot(0));
    const bool sub = canon29<K, G>(z, M);
    canon29<K, G>(r, M);
    uint32_t d[K];
    negate(d, r, sub);
    uint32_t w[K32];
    to32<K, K32, G>(w, z, digit_row());
    if (valid && !second_digit) st<K32, G>(o, w);
    to32<K, K32, G>(w, d, digit_row());
    if (valid && !second_digit) st<K32, G>(o + SN, w);
  }
};

// X <- X^e mod N^2 (mod N for LaneMod) for one unit of 64 / kLanes integers:
// in, `pieces` pieces of SN 32-bit limbs (X = sum_h x_h 2^(32 SN h)); out, the
// digits (a, e) of X^e = a + e N, canonical, SN limbs each (LaneMod: X^e).
// Schedules: sliding windows over odd powers (keysetup.hpp), or (CT) fixed
// windows and masked reads of every table entry, as in pow29.  One loop holds the only copy
// of the squaring and of the product, since each fills a good part of the
// instruction cache; what surrounds them is chosen by wave-uniform state.
template <class E, int SN, bool CT>
__device__ __forceinline__ void power_unit(E &eng, const DExp &X, const uint32_t *in, int pieces, uint32_t *out,
                                           bool valid) {
  enum { IN, SQUARE, TABLE, RUN, LEAVE, UNSCALE };
  int state = IN, t = 0;
#pragma unroll 1
  for (;;) {
    // the squarings, then the product with this operand
    uint32_t nsq = 0, entry = CT ? 1u : (uint32_t)kTable;
    bool product = true, constant = false;
    if (state == IN) {
      eng.load_piece(in + t * SN);
      entry = t;
      constant = true;
    } else if (state == SQUARE) {
      nsq = 1;
      product = false;
    } else if (state == RUN) {
      if constexpr (CT) {
        nsq = kWindow;
        entry = __builtin_amdgcn_readfirstlane(exp_digit(X.e, t));
      } else {
        const uint32_t op = __builtin_amdgcn_readfirstlane(X.ops[t]);
        nsq = op >> 8;
        entry = op & 0xFFu;
        product = entry < (uint32_t)kTable;
      }
    } else if (state != TABLE) {
      entry = state == LEAVE ? he29::kPairOne : he29::kPairUnscale;
      constant = true;
    }
#pragma unroll 1
    for (; nsq > 0; --nsq) eng.sq();
    if (product) {
      if (CT && state == RUN)
        eng.fetch_masked(entry);
      else
        eng.fetch(entry, constant);
      eng.mul();
    }
    // what the product was for
    if (state == IN) {
      if (t) eng.add(CT ? 1 : 0);
      eng.store(CT ? 1 : 0);
      if (++t < pieces) continue;
      state = CT ? TABLE : SQUARE;
      t = CT ? 2 : 1;
    } else if (state == SQUARE) {
      eng.store(kTable);
      eng.load(0);
      state = TABLE;
    } else if (state == TABLE) {
      eng.store(t);
      if (++t < kTable) continue;
      if constexpr (CT) {
        eng.load_const(he29::kPairR);
        eng.store(0);
        // the top window's entry: 1 times it
        t = X.nwin - 1;
        state = RUN;
      } else {
        if (X.nops) eng.load(__builtin_amdgcn_readfirstlane(X.ops[0]) & 0xFFu);
        else eng.load_const(he29::kPairR);
        t = 1;
        state = X.nops > 1 ? RUN : LEAVE;
      }
    } else if (state == RUN) {
      if constexpr (CT) state = --t >= 0 ? RUN : LEAVE;
      else state = ++t < X.nops ? RUN : LEAVE;
    } else if (state == LEAVE && E::kDigits == 2) {
      eng.store(0);
      eng.second();
      state = UNSCALE;
    } else {
      break;
    }
  }
  eng.out(out, valid);
}

// x -> x^(N e) mod N^2 for a prime N and x below 2^(32 SN), e the key's other
// prime mod N - 1: what encryption needs of r, since r^n = (r^q)^p mod p^2
// depends on r^q mod p only.  As x^(N e) = (x^(N - 1))^e x^e and x^(N - 1) is
// R (1 + f N) in Montgomery form, its power e is R (1 + e f N), which is
// linear: e times it plus (1 - e) R.  So one chain of squarings mod N^2 serves
// both exponents (keysetup.hpp, joint_schedule) instead of one chain mod N for
// r^q and one mod N^2 for the power p.  (x = 0 mod N: x^e is 0 and so is the
// product.)  Multiplications per bit, in S^2: 3.5 for the square and 2 / 6 of
// a bucket product of 5, against 1.5 + 3.5 for the squares of two chains and
// 7 / 7 for their products; 31 products join the buckets of an exponent.
// The state stays in registers as the operand while a bucket takes its place
// (turn, back).  Bound by VALU issue at a wave or more per SIMD, by the latency
// of a step below.  Measured against the two chains, 2048-bit key: 500
// encryptions' powers 4.75 -> 3.16 ms, 16,384 11.8 -> 10.4, 200,000 117 -> 98;
// 1024-bit key: 500 1.26 -> 0.89.
// The schedule's addresses follow the exponents: keys that ask for secret
// digits run the two chains with masked tables (power_unit, CT).
template <class E, int SN>
__device__ __forceinline__ void joint_unit(E &eng, const DExp &X, const uint32_t *in, uint32_t *out, bool valid) {
  enum { IN, RUN, POWER, JOIN, LEAVE, UNSCALE };
  constexpr uint32_t kOther = he29::kJointBuckets;  // slots the schedule is done with: x^e, and (1 - e) R
  // a slot number the compiler does not know: the addresses of fixed ones would
  // be kept in registers through the loop
  auto at = [](uint32_t e) {
    asm volatile("" : "+s"(e));
    return e;
  };
  int state = IN, t = 0;
  eng.load_piece(in);
#pragma unroll 1
  for (;;) {
    uint32_t nsq = 0, entry = 0, what = he29::kJointTake;
    bool constant = true;
    if (state == RUN) {
      const uint32_t op = __builtin_amdgcn_readfirstlane(X.ops[t]);
      nsq = op >> 10;
      what = (op >> 8) & 3u;
      entry = op & 0xFFu;
      constant = false;
    } else if (state == POWER) {
      eng.store(at(kOther));
      eng.load_const(at(he29::kPairE1));
      eng.store(at(kOther + 1));
      eng.load(at(0));
      entry = he29::kPairE;
    } else if (state == JOIN) {
      entry = kOther;
      constant = false;
    } else if (state != IN) {
      entry = state == LEAVE ? he29::kPairOne : he29::kPairUnscale;
    }
#pragma unroll 1
    for (; nsq > 0; --nsq) eng.sq();
    if (what & he29::kJointTake) {
      if (what == he29::kJointAcc) eng.turn(entry);
      else eng.fetch(entry, constant);
      eng.pin();
      eng.mul();
    }
    eng.pin();
    if (what == he29::kJointPut || what == he29::kJointAcc) eng.store(entry);
    if (what == he29::kJointLoad) eng.load(entry);
    if (what == he29::kJointAcc) eng.back();
    eng.pin();
    if (state == RUN) {
      if (++t == X.nops) state = POWER;
    } else if (state == POWER) {
      eng.add(at(kOther + 1));
      state = JOIN;
    } else if (state == LEAVE) {
      eng.store(at(0));
      eng.second();
      state = UNSCALE;
    } else if (state == UNSCALE) {
      break;
    } else {
      state = state == IN ? RUN : LEAVE;
    }
  }
  eng.out(out, valid);
}

}  // namespace he
