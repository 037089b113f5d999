// Histogram products in two digits base n (pair29.hpp): the conversion of the
// ciphertexts, the products of the work items and the join of their partials.
#pragma once
#include "he_internal.hpp"
#include "hist_bucket.hpp"
#include "pair29.hpp"

namespace he {

constexpr int kHistVariant = 2;  // limb-count variant: R = 2^(29 S), R^2 the factor of HE_FORM_MONT

// Both digits of an integer in the same G lanes, K limbs of each per lane.
// A product by a row in LDS takes two passes: the first digit's (its quotient
// digits go to LDS), then the second digit's, which starts from them.  Per step
// of 18 limbs per lane that is 54 multiply-adds and 6 other instructions (36
// and 6 in the first pass) on 4 lanes; side by side (GroupPair) the same
// product costs 54 and 9 on 8.
template <int SN, int G>
struct SeqPair {
  static constexpr int S = he29::pair_limbs(SN, kHistVariant), K = S / G;
  static constexpr int U = K % 2 == 0 ? K : 2 * K;
  // LDS words per group: c, d, then a zero and the quotient digits (which so
  // start on an even word); a stride of 4 mod 32 keeps the rows 16-byte aligned
  // and the groups' reads of one limb pair on different banks
  static constexpr int kM = 2 * S + 1, kLds = ((3 * S + 2 - 4 + 31) / 32) * 32 + 4;
  static_assert(2 * S == he29::limbs_for_group(2 * SN, 16), "HE_FORM_MONT holds x R^2");
  static_assert(S % U == 0 && K >= 2 && K <= 21 && S % 2 == 0, "column bound: 3 K products of 2^58");
  Mod29<K> M;
  uint32_t *lds;

  __device__ __forceinline__ SeqPair(const DPair &c, uint32_t *row) : lds(row) {
    ld29<K, G>(M.n, c.c[kHistVariant] + 2 * he29::kPairN * S);
    M.ninv = c.ninv & kMask29;
    M.mask = mask_vgpr();
    if (glane<G>() == 0) lds[kM] = 0;
  }
  // C <- (C + sum_i (u_i Y + v_i Z) 2^(29 i) + q N) 2^(-29 S): u, v (PRODS of
  // them) limbs in LDS; KEEP: the quotient digits to LDS.
  template <int PRODS, bool KEEP>
  __device__ __forceinline__ void pass(uint64_t (&C)[K], const uint32_t *u, const uint32_t (&Y)[K], const uint32_t *v,
                                       const uint32_t (&Z)[K]) {
    uint32_t top = (uint32_t)C[K - 1];
#pragma unroll 1
    for (int i0 = 0; i0 < S; i0 += U) {
      uint2 u2, v2, un{}, vn{}, qs{};
      if constexpr (PRODS >= 1) un = *reinterpret_cast<const uint2 *>(u + i0);
      if constexpr (PRODS >= 2) vn = *reinterpret_cast<const uint2 *>(v + i0);
      static_for<0, U>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        if constexpr (s % 2 == 0) {
          if constexpr (s > 0) __builtin_amdgcn_sched_barrier(0);
          u2 = un;
          v2 = vn;
          if constexpr (s + 2 < U) {
            if constexpr (PRODS >= 1) un = *reinterpret_cast<const uint2 *>(u + i0 + s + 2);
            if constexpr (PRODS >= 2) vn = *reinterpret_cast<const uint2 *>(v + i0 + s + 2);
          }
        }
        C[K - 1] = top;
        if constexpr (PRODS >= 1) {
          const uint32_t ui = s % 2 == 0 ? u2.x : u2.y;
#pragma unroll
          for (int j = 0; j < K; ++j) C[j] += (uint64_t)ui * Y[j];
        }
        if constexpr (PRODS >= 2) {
          const uint32_t vi = s % 2 == 0 ? v2.x : v2.y;
#pragma unroll
          for (int j = 0; j < K; ++j) asm("" : "+v"(C[j]));
#pragma unroll
          for (int j = 0; j < K; ++j) C[j] += (uint64_t)vi * Z[j];
        }
        const uint32_t q = bcast_first_m29<G>(mul_lo32((uint32_t)C[0], M.ninv), M.mask);
        if constexpr (KEEP) {
          if constexpr (s % 2 == 0) {
            qs.x = q;
          } else {
            qs.y = q;
            *reinterpret_cast<uint2 *>(lds + kM + 1 + i0 + s - 1) = qs;
          }
        }
#pragma unroll
        for (int j = 0; j < K; ++j) C[j] += (uint64_t)q * M.n[j];
        top = rotate_next_m29<G>((uint32_t)C[0], M.mask);
        C[1] += C[0] >> he29::kBits;
#pragma unroll
        for (int j = 0; j + 1 < K; ++j) C[j] = C[j + 1];
#pragma unroll
        for (int j = 0; j + 1 < K; ++j) asm("" : "+v"(C[j]));
        asm("" : "+v"(top));
      });
    }
    C[K - 1] = top;
  }
  // C <- 2^29 m (the quotient digits one limb up, the last of them kept back)
  __device__ __forceinline__ void start_second(uint64_t (&C)[K]) {
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < K; ++j) C[j] = lds[kM + glane<G>() * K + j];
  }
  __device__ __forceinline__ void end_second(uint64_t (&C)[K]) {
    if (glane<G>() == 0) C[0] += lds[kM + S];
    __builtin_amdgcn_wave_barrier();
  }
  // (a, b) <- (a, b) (c, d) R^-1, c and d in LDS rows.
  __device__ __forceinline__ void mul(uint32_t (&a)[K], uint32_t (&b)[K], const uint32_t *c, const uint32_t *d) {
    uint64_t C[K];
    uint32_t a1[K];
#pragma unroll
    for (int j = 0; j < K; ++j) C[j] = 0;
    pass<1, true>(C, c, a, c, a);
    settle29<K, G>(a1, C);
    start_second(C);
    pass<2, false>(C, c, b, d, a);
    end_second(C);
    settle29<K, G>(b, C);
#pragma unroll
    for (int j = 0; j < K; ++j) a[j] = a1[j];
  }
  // The pair (a, b) of x R from the ciphertext x (2 SN words): from the Montgomery
  // form X = x R^2 by two reductions alone: X + m n = R a', so X R^-1 = a' - (m
  // R^-1) n.  From x itself by the products of its two halves with the constants'
  // (c0) first two pieces.
  __device__ __forceinline__ void enter(uint32_t (&a)[K], uint32_t (&b)[K], const uint32_t *x, bool mont,
                                        const uint32_t *c0) {
    constexpr int K32 = SN / G;
    uint32_t lo[K], hi[K];
    uint64_t C[K];
    if (mont) {
      // X's 2 S limbs: the low half is the reduction's input, the high half its addend
      uint32_t w[2 * K32];
      ld<2 * K32, G>(w, x);
      st<2 * K32, G>(lds, w);
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int j = 0; j < K; ++j) {
          const uint32_t bit = he29::kBits * (h * S + glane<G>() * K + j), i = bit >> 5;
          const uint32_t l = i < 2 * SN ? lds[i] : 0u, u = i + 1 < 2 * SN ? lds[i + 1] : 0u;
          const uint32_t t = __builtin_amdgcn_alignbit(u, l, bit & 31u) & kMask29;
          if (h) hi[j] = t;
          else lo[j] = t;
        }
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int j = 0; j < K; ++j) C[j] = lo[j];
      pass<0, true>(C, nullptr, lo, nullptr, lo);
#pragma unroll
      for (int j = 0; j < K; ++j) C[j] += hi[j];
      settle29<K, G>(a, C);
      start_second(C);
      pass<0, false>(C, nullptr, lo, nullptr, lo);
      end_second(C);
      settle29<K, G>(b, C);
    } else {
      const uint32_t *c1 = c0 + 2 * S;
      uint32_t w[K32];
      ld<K32, G>(w, x);
      to29<K32, K, G>(lo, w, lds);
      ld<K32, G>(w, x + SN);
      to29<K32, K, G>(hi, w, lds);
      st29<K, G>(lds, lo);
      st29<K, G>(lds + S, hi);
      __builtin_amdgcn_wave_barrier();
      ld29<K, G>(lo, c0);
      ld29<K, G>(hi, c1);
#pragma unroll
      for (int j = 0; j < K; ++j) C[j] = 0;
      pass<2, true>(C, lds, lo, lds + S, hi);
      settle29<K, G>(a, C);
      ld29<K, G>(lo, c0 + S);
      ld29<K, G>(hi, c1 + S);
      start_second(C);
      pass<2, false>(C, lds, lo, lds + S, hi);
      end_second(C);
      settle29<K, G>(b, C);
    }
  }
};

// ---- ciphertexts -> pairs ------------------------------------------------------
// Pair of x R per ciphertext x: 2 S words (first digit, then the second times
// 2^29).  `rows` ciphertext pairs: all resident rows in order, or (gather) the
// samples of every job one after the other; a job's sample whose row is not
// resident is left out.  4 lanes per ciphertext; two reductions are 0.4 of one
// histogram product, six limb products 1.2 of one.
template <int KP, int G>
__global__ __launch_bounds__(kBlockThreads, 2) void k_hist_pairs(DPair pc, const uint32_t *__restrict__ in, int mont,
                                                                 HistWs ws, uint64_t count) {
  constexpr int SN = 32 * KP, GB = kBlockThreads / G;
  using E = SeqPair<SN, G>;
  constexpr int S = E::S, K = E::K;
  __shared__ __align__(16) uint32_t lds_all[GB * E::kLds];
  uint64_t r = (uint64_t)blockIdx.x * (GB / 2) + threadIdx.x / (2 * G);
  const uint32_t slot = (threadIdx.x / G) & 1u;
  bool valid = r < count;
  if (!valid) r = count - 1;
  uint64_t row = r;
  if (ws.gather) {
    const DJob J = ws.jobs[find_job(ws.jobs, ws.n_jobs, &DJob::s_off, r)];
    const uint32_t at = J.idx[r - J.s_off];
    valid = valid && at < ws.rows;
    row = at < ws.rows ? at : 0;
  }
  E eng(pc, lds_all + (threadIdx.x / G) * E::kLds);
  uint32_t a[K], b[K];
  eng.enter(a, b, in + (row * 2 + slot) * (uint64_t)(2 * SN), mont != 0, pc.c[kHistVariant]);
  if (valid) {
    uint32_t *o = ws.pairs + (r * 2 + slot) * (uint64_t)(2 * S);
    st29<K, G>(o, a);
    st29<K, G>(o + S, b);
  }
}

// ---- products of the work items ---------------------------------------------------
// Product of the ciphertexts of one item (chunk) per (item, slot g/h), 4 lanes
// per ciphertext: a wave's 16 groups are 8 / P items x P runs x 2 slots (bit 0
// of the group's index the slot, then the run); an item is cut into P runs of
// equal length (to one), joined in log2 P levels.  Items are claimed from a
// counter, longest first over the whole batch (k_hist_items), so a wave's items
// are of one length (to one) and the waves end together to within a short
// item.  A group past the end of its run multiplies by the Montgomery one.
// Each row is staged through registers into LDS one product ahead of its use.
// VALU-bound: 7,400 instructions a product per lane of 4, 6,480 of them
// multiply-adds, where the product as one 144-limb integer took 6,200 on 8
// lanes; two waves per SIMD (LDS and VGPRs allow no third) issue every cycle.
// Root node of 100,000 samples x 32 features x 256 bins: 9.6 -> 6.0 ms for 6.4 M
// products, 27.6 T multiply-adds/s.
// DIRECT: the ciphertexts are read as they are resident and converted one by one,
// 1.4 to 2.2 times the work, for callers whose memory holds no second copy.
template <int KP, int G, bool DIRECT>
__global__ __launch_bounds__(kBlockThreads, 2) void k_hist_chunk(DPair pc, HistWs ws) {
  constexpr int SN = 32 * KP, GW = 64 / G;
  using E = SeqPair<SN, G>;
  constexpr int S = E::S, K = E::K, ROW = 2 * S, V = ROW / (4 * G);  // 16-byte pieces per lane and row
  static_assert(ROW % (4 * G) == 0, "rows are whole 16-byte pieces per lane");
  __shared__ __align__(16) uint32_t lds_all[(kBlockThreads / G) * E::kLds];
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t g = (threadIdx.x & 63u) / G;
  uint32_t *lds = lds_all + (wave * GW + g) * E::kLds;
  const uint32_t P = ws.runs, slot = g & 1u, run = (g >> 1) & (P - 1u), which = (g >> 1) / P;
  const uint32_t per_wave = GW / 2 / P;
  E eng(pc, lds);
  const uint32_t *one = pc.c[kHistVariant] + 2 * he29::kPairR * S;
  const uint64_t n_items = *ws.n_items;
  // The grid is sized for the most items there could be.  Where there are fewer
  // units than its waves, whichever waves claim first would take them, two on one
  // SIMD and none on another: the blocks past the units leave (784 units on 512
  // blocks 0.66 ms, on the 196 they need 0.52).
  if ((uint64_t)blockIdx.x * (kBlockThreads / 64) * per_wave >= n_items) return;
  auto stage = [&](const uint32_t (&p)[4 * V]) __attribute__((always_inline)) {  // a row to LDS words [0, 2 S)
    stv<4 * V>(lds + glane<G>() * 4, p, 4 * G);
    __builtin_amdgcn_wave_barrier();
  };
  auto load = [&](uint32_t (&p)[4 * V], const uint32_t *row) __attribute__((always_inline)) {
    ldv<4 * V>(p, row + glane<G>() * 4, 4 * G);
  };
  for (;;) {
    uint32_t v = 0;
    if (lane_id() == 0) v = atomicAdd(ws.next, 1u);
    const uint64_t w0 = (uint64_t)__builtin_amdgcn_readfirstlane(v) * per_wave;
    if (w0 >= n_items) break;
    const uint64_t it = w0 + which;
    const bool valid = it < n_items;
    const HistItem item = ws.items[valid ? it : n_items - 1];
    const uint32_t lo = valid ? (uint32_t)((uint64_t)run * item.len / P) : 0u;
    const uint32_t len = valid ? (uint32_t)((uint64_t)(run + 1) * item.len / P) - lo : 0u;
    uint32_t trip = 0;  // the longest run in the wave
    for (uint64_t w = w0; w < w0 + per_wave && w < n_items; ++w) trip = max(trip, (ws.items[w].len + P - 1) / P);
    trip = __builtin_amdgcn_readfirstlane(trip);
    const uint32_t *pp = ws.perm + item.start + lo;
    auto row_at = [&](uint32_t k) __attribute__((always_inline)) {
      return k < len ? ws.pairs + ((uint64_t)pp[k] * 2 + slot) * ROW : one;
    };
    uint32_t a[K], b[K];
    if constexpr (DIRECT) {
      // sample k's pair; past the run a resident row is read and the one kept
      auto take = [&](uint32_t (&u)[K], uint32_t (&v)[K], uint32_t k) __attribute__((always_inline)) {
        uint32_t o[K];
        eng.enter(u, v, ws.ct + ((uint64_t)(k < len ? pp[k] : 0u) * 2 + slot) * (2 * SN), ws.mont != 0, pc.c[kHistVariant]);
        ld29<K, G>(o, one);
        select(u, k < len, u, o);
        ld29<K, G>(o, one + S);
        select(v, k < len, v, o);
      };
      take(a, b, 0);
#pragma unroll 1
      for (uint32_t k = 1; k < trip; ++k) {
        uint32_t u[K], v[K];
        take(u, v, k);
        st29<K, G>(lds, u);
        st29<K, G>(lds + S, v);
        __builtin_amdgcn_wave_barrier();
        eng.mul(a, b, lds, lds + S);
        __builtin_amdgcn_wave_barrier();
      }
    } else {
      const uint32_t *first = row_at(0);
      ld29<K, G>(a, first);
      ld29<K, G>(b, first + S);
      uint32_t next[4 * V];
      load(next, row_at(1));
#pragma unroll 1
      for (uint32_t k = 1; k < trip; ++k) {
        stage(next);
        load(next, row_at(k + 1));  // (past the run: the one)
        eng.mul(a, b, lds, lds + S);
        __builtin_amdgcn_wave_barrier();
      }
    }
    uint64_t done = trip ? trip - 1 : 0, real = len ? len - 1 : 0;
    for (uint32_t d = 1; d < P; d <<= 1) {
      // run p joins run p + d for p a multiple of 2 d; the others' products are not kept
      st29<K, G>(lds, a);
      st29<K, G>(lds + S, b);
      __builtin_amdgcn_wave_barrier();
      const uint32_t *other = lds_all + (wave * GW + ((g + 2 * d) & (GW - 1))) * E::kLds;
      const bool join = (run & (2 * d - 1)) == 0;
      uint32_t a1[K], b1[K];
#pragma unroll
      for (int j = 0; j < K; ++j) {
        a1[j] = a[j];
        b1[j] = b[j];
      }
      eng.mul(a1, b1, other, other + S);
      select(a, join, a1, a);
      select(b, join, b1, b);
      __builtin_amdgcn_wave_barrier();
      ++done;
      if (join && valid) {
        // real where both sides hold samples: run + d's share is not empty
        const uint32_t lo2 = (uint32_t)((uint64_t)(run + d) * item.len / P);
        const uint32_t hi2 = (uint32_t)((uint64_t)min(run + 2 * d, P) * item.len / P);
        const uint32_t mid = (uint32_t)((uint64_t)run * item.len / P);
        if (hi2 > lo2 && lo2 > mid) ++real;
      }
    }
    if (run == 0 && valid) {
      uint32_t *o = ws.partials + (it * 2 + slot) * (uint64_t)ROW;
      st29<K, G>(o, a);
      st29<K, G>(o + S, b);
    }
    if (ws.mm_count && glane<G>() == 0) {
      atomicAdd(&ws.mm_count[0], (unsigned long long)real);
      atomicAdd(&ws.mm_count[1], (unsigned long long)done);
    }
  }
}

}  // namespace he
