// CKKS for the secure horizontal path (clients encrypt local G/H histogram
// vectors, the server adds ciphertexts, clients decrypt the global
// histogram): public-key encryption, addition and decryption over
// R_Q = Z_Q[X]/(X^N + 1) in RNS form (three primes q_i < 2^30, q_i = 1 mod
// 2N), with the canonical-embedding encoding.  Everything runs in the
// kernels below; the host part builds the per-prime tables and the keys.
//
// Layouts: a polynomial is uint32 [L][N] residues (prime-major); a
// ciphertext is [2][L][N] (c0 then c1), coefficient domain.  Keys stay on
// the device in the NTT domain and in Montgomery form (times 2^32 mod q).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/he.h"
#include "../../include/he_ckks.h"
#include "he_internal.hpp"
#include "mont.hpp"

namespace {

constexpr int kL = 3;            // RNS primes
constexpr int kPrimeBits = 30;
constexpr int kEta = 21;         // centered binomial parameter
constexpr uint64_t kKeyEBase = 1ull << 40;
constexpr uint64_t kKeyABase = 1ull << 41;

struct Prime {
  uint32_t q, qinv;       // qinv = -q^-1 mod 2^32
  uint32_t r1, r2;        // 2^32 and 2^64 mod q (into Montgomery form)
  uint32_t ninv, ninv_s;  // N^-1 mod q and its Shoup companion
};

struct Tables {
  Prime p[kL];
  const uint2 *psi;   // [L][N] psi^bitrev(i) and its Shoup companion floor(w 2^32 / q)
  const uint2 *ipsi;  // [L][N] psi^-bitrev(i), the same way
};

// ---- modular helpers (q < 2^30) -------------------------------------------
__device__ __forceinline__ uint32_t add_q(uint32_t a, uint32_t b, uint32_t q) {
  const uint32_t s = a + b;
  return s >= q ? s - q : s;
}
__device__ __forceinline__ uint32_t sub_q(uint32_t a, uint32_t b, uint32_t q) {
  return a >= b ? a - b : a + q - b;
}
// a b 2^-32 mod q (Montgomery), a, b < q.
__device__ __forceinline__ uint32_t mont_q(uint32_t a, uint32_t b, uint32_t q, uint32_t qinv) {
  const uint64_t t = (uint64_t)a * b;
  const uint32_t m = (uint32_t)t * qinv;
  const uint32_t r = (uint32_t)((t + (uint64_t)m * q) >> 32);
  return r >= q ? r - q : r;
}
// a mod q for a < 2q.
__device__ __forceinline__ uint32_t once(uint32_t a, uint32_t q) { return a >= q ? a - q : a; }
// x w mod q in [0, 2q) for any x.
__device__ __forceinline__ uint32_t mul_lazy(uint32_t x, uint2 w, uint32_t q) { return x * w.x - __umulhi(x, w.y) * q; }
// v mod q by two Montgomery products (|v| = hi 2^32 + lo; a product by 2^32
// resp. 2^64 mod q stays below q 2^32, so one subtraction reduces it).
__device__ __forceinline__ uint32_t to_residue(int64_t v, const Prime &P) {
  const uint64_t m = v < 0 ? (uint64_t)0 - (uint64_t)v : (uint64_t)v;
  const uint32_t r =
      add_q(mont_q((uint32_t)(m >> 32), P.r2, P.q, P.qinv), mont_q((uint32_t)m, P.r1, P.q, P.qinv), P.q);
  return v < 0 && r ? P.q - r : r;
}

// ---- sampling ---------------------------------------------------------------
// Ternary (word mod 3 - 1) and centered binomial (popcount of bits 0..20 minus
// popcount of bits 21..41) values of one stream word.
__device__ __forceinline__ uint32_t ternary(uint64_t w, uint32_t q) {
  const uint32_t t = (uint32_t)(w % 3);
  return t ? t - 1u : q - 1u;
}
__device__ __forceinline__ uint32_t binomial(uint64_t w, uint32_t shift) {  // value + shift
  const uint32_t mask = (1u << kEta) - 1u;
  return shift + __popc((uint32_t)w & mask) - __popc((uint32_t)(w >> kEta) & mask);
}
// kind 0: ternary; 1: centered binomial; 2: uniform mod q_i, with the counter
// base advanced by i N for prime i.  out: [L][N].
__global__ void k_sample(int kind, uint64_t seed, uint64_t base, uint32_t n, Tables T, uint32_t *out) {
  const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  for (int i = 0; i < kL; ++i) {
    const uint64_t w = he::splitmix64(seed, base + (kind == 2 ? (uint64_t)i * n : 0ull) + j);
    const uint32_t q = T.p[i].q;
    out[(uint64_t)i * n + j] = kind == 0 ? ternary(w, q) : (kind == 1 ? once(binomial(w, q), q) : (uint32_t)(w % q));
  }
}

// ---- negacyclic NTT ------------------------------------------------------------
// One block of N / 16 threads per (polynomial, prime).  Forward: Cooley-Tukey
// with psi powers in bit-reversed order (natural order in, bit-reversed out);
// inverse: Gentleman-Sande with inverse powers, then N^-1 (Longa & Naehrig, CANS
// 2016, Algorithms 1 and 2).  A thread holds 16 values and runs up to four
// stages on them in registers, so the polynomial crosses LDS three times
// instead of once per stage (14 at N = 2^14); values stay below 4q between
// stages (Harvey's lazy butterflies, q < 2^30).  Few polynomials are in flight
// at a time, so what one block issues bounds it: a transform of 2^14 took 37-44 us
// stage by stage and takes about 11 inside the kernels below.
//
// Register c of thread t holds, before the forward and after the inverse
// transform, coefficient t + c T (T threads); in between it holds position
// ntt_pos(c) of the bit-reversed order.
template <int LOGN>
struct Ntt {
  static constexpr uint32_t N = 1u << LOGN, T = N / 16;
  static constexpr int R = LOGN - 12;  // stages of the short pass
  static constexpr uint32_t kLds = N + N / 16;  // words, 4 of padding after every 64
};
__device__ __forceinline__ uint32_t pad(uint32_t i) { return i + ((i >> 6) << 2); }
template <int LOGN>
__device__ __forceinline__ uint32_t ntt_pos(int c) {
  constexpr int R = Ntt<LOGN>::R;
  if constexpr (R == 0) return 16 * threadIdx.x + c;
  return ((threadIdx.x + Ntt<LOGN>::T * (c >> R)) << R) + (c & ((1 << R) - 1));
}
// Stages s .. s + RR - 1 of the forward transform on the 2^RR values of group
// `grp` (of 2^s) in v[at ..].
template <int RR>
__device__ __forceinline__ void fwd_stages(uint32_t (&v)[16], int at, int s, uint32_t grp, const uint2 *w, uint32_t q) {
#pragma unroll
  for (int i = 0; i < RR; ++i) {
    __builtin_amdgcn_sched_barrier(0);  // not all stages' twiddles at once
    const uint2 *ws = w + ((1u + grp) << i) + ((((1u << s) - 1u)) << i);
#pragma unroll
    for (int c = 0; c < (1 << RR); ++c) {
      const int h = 1 << (RR - 1 - i);
      if (c & h) continue;
      const uint2 t = ws[c >> (RR - i)];
      uint32_t u = v[at + c];
      u = u >= 2 * q ? u - 2 * q : u;
      const uint32_t x = mul_lazy(v[at + c + h], t, q);
      v[at + c] = u + x;
      v[at + c + h] = u - x + 2 * q;
    }
  }
}
// Stages with half-lengths 2^e .. 2^(e + RR - 1) of the inverse transform.
template <int LOGN, int RR>
__device__ __forceinline__ void inv_stages(uint32_t (&v)[16], int at, int e, uint32_t grp, const uint2 *w, uint32_t q) {
#pragma unroll
  for (int i = 0; i < RR; ++i) {
    __builtin_amdgcn_sched_barrier(0);
    const uint2 *ws = w + (Ntt<LOGN>::N >> (e + i + 1)) + (grp << (RR - 1 - i));
#pragma unroll
    for (int c = 0; c < (1 << RR); ++c) {
      if (c & (1 << i)) continue;
      const uint2 t = ws[c >> (i + 1)];
      const uint32_t u = v[at + c], x = v[at + c + (1 << i)];
      const uint32_t y = u + x;
      v[at + c] = y >= 2 * q ? y - 2 * q : y;
      v[at + c + (1 << i)] = mul_lazy(u - x + 2 * q, t, q);
    }
  }
}
// Set of 16 values `stride` apart: thread t's set starts at set_base.
__device__ __forceinline__ uint32_t set_base(uint32_t stride) {
  return (threadIdx.x / stride) * (16 * stride) + threadIdx.x % stride;
}
__device__ __forceinline__ void to_lds(uint32_t *a, const uint32_t (&v)[16], uint32_t base, uint32_t stride) {
#pragma unroll
  for (int c = 0; c < 16; ++c) a[pad(base + c * stride)] = v[c];
}
__device__ __forceinline__ void from_lds(uint32_t (&v)[16], const uint32_t *a, uint32_t base, uint32_t stride) {
#pragma unroll
  for (int c = 0; c < 16; ++c) v[c] = a[pad(base + c * stride)];
}
template <int LOGN>
__device__ __forceinline__ void ntt_forward(uint32_t (&v)[16], uint32_t *a, const uint2 *w, uint32_t q) {
  using C = Ntt<LOGN>;
  constexpr uint32_t S1 = C::T, S2 = C::N >> 8, S3 = C::N >> 12;
  fwd_stages<4>(v, 0, 0, 0, w, q);
  to_lds(a, v, threadIdx.x, S1);
  __syncthreads();
  from_lds(v, a, set_base(S2), S2);
  fwd_stages<4>(v, 0, 4, threadIdx.x / S2, w, q);
  to_lds(a, v, set_base(S2), S2);
  __syncthreads();
  from_lds(v, a, set_base(S3), S3);
  fwd_stages<4>(v, 0, 8, threadIdx.x / S3, w, q);
  if constexpr (C::R > 0) {
    to_lds(a, v, set_base(S3), S3);
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 16; ++c) v[c] = a[pad(ntt_pos<LOGN>(c))];
#pragma unroll
    for (int k = 0; k < (16 >> C::R); ++k) fwd_stages<C::R>(v, k << C::R, 12, threadIdx.x + C::T * k, w, q);
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    const uint32_t x = v[c] >= 2 * q ? v[c] - 2 * q : v[c];
    v[c] = x >= q ? x - q : x;
  }
}
template <int LOGN>
__device__ __forceinline__ void ntt_inverse(uint32_t (&v)[16], uint32_t *a, const uint2 *w, const Prime &P) {
  using C = Ntt<LOGN>;
  constexpr uint32_t S1 = C::T, S2 = C::N >> 8, S3 = C::N >> 12;
  const uint32_t q = P.q;
  if constexpr (C::R > 0) {
#pragma unroll
    for (int k = 0; k < (16 >> C::R); ++k) inv_stages<LOGN, C::R>(v, k << C::R, 0, threadIdx.x + C::T * k, w, q);
#pragma unroll
    for (int c = 0; c < 16; ++c) a[pad(ntt_pos<LOGN>(c))] = v[c];
    __syncthreads();
    from_lds(v, a, set_base(S3), S3);
  }
  inv_stages<LOGN, 4>(v, 0, C::R, threadIdx.x / S3, w, q);
  to_lds(a, v, set_base(S3), S3);
  __syncthreads();
  from_lds(v, a, set_base(S2), S2);
  inv_stages<LOGN, 4>(v, 0, C::R + 4, threadIdx.x / S2, w, q);
  to_lds(a, v, set_base(S2), S2);
  __syncthreads();
  from_lds(v, a, threadIdx.x, S1);
  inv_stages<LOGN, 4>(v, 0, C::R + 8, 0, w, q);
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    const uint32_t x = mul_lazy(v[c], make_uint2(P.ninv, P.ninv_s), q);
    v[c] = x >= q ? x - q : x;
  }
}

// Forward transform in place of the L polynomials at x (key generation).
template <int LOGN>
__global__ __launch_bounds__(Ntt<LOGN>::T) void k_ntt(uint32_t *x, Tables T) {
  extern __shared__ uint32_t a[];
  x += (uint64_t)blockIdx.x * Ntt<LOGN>::N;
  uint32_t v[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) v[c] = x[threadIdx.x + c * Ntt<LOGN>::T];
  ntt_forward<LOGN>(v, a, T.psi + (uint64_t)blockIdx.x * Ntt<LOGN>::N, T.p[blockIdx.x].q);
#pragma unroll
  for (int c = 0; c < 16; ++c) x[ntt_pos<LOGN>(c)] = v[c];
}

// Samples of ciphertext t from counters (offset + t) 3N + {0, N, 2N} (u, e0, e1),
// one byte each, four coefficients per thread.  They go into the ciphertext's
// own buffer: the region of (part k, prime i), N words, first holds the N bytes
// of u and then those of e_k, which only the block that later writes the region
// reads.  Sampled once here and not in each of the six blocks of a ciphertext:
// ten ciphertexts at N = 2^14 took 52 us with the sampling in those blocks and
// take 29 (4 of them here).
__global__ __launch_bounds__(256) void k_sample_enc(uint64_t seed, uint64_t offset, uint32_t log_n, uint64_t quads,
                                                    uint32_t *ct) {
  const uint64_t id = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (id >= quads) return;
  const uint64_t t = id >> (log_n - 2), N = 1ull << log_n, j = id & (N / 4 - 1);
  const uint64_t base = (offset + t) * 3 * N + 4 * j;
  uint32_t u = 0, e[2] = {0, 0};
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    u |= (uint32_t)(he::splitmix64(seed, base + b) % 3) << (8 * b);  // value + 1
#pragma unroll
    for (int k = 0; k < 2; ++k) e[k] |= binomial(he::splitmix64(seed, base + (k + 1) * N + b), kEta) << (8 * b);
  }
#pragma unroll
  for (int r = 0; r < 2 * kL; ++r) {
    uint32_t *o = ct + (t * 2 * kL + r) * N + j;
    o[0] = u;
    o[N / 4] = r < kL ? e[0] : e[1];
  }
}

// Part k of ciphertext t for one prime: INTT(b u) + e0 + m or INTT(a u) + e1, from
// the samples k_sample_enc left in its region of ct.  With it two launches
// instead of nine: transforms, product and sums stay in registers.  Each part
// transforms u again: a block that made both from one transform had to hold it
// beside the inverse's values and spilled, and took 1.14 ms for 1,000
// ciphertexts at N = 2^14 where this takes 0.64 (2.1 with a launch per step); for
// ten the parts also spread over twice the compute units (105 -> 25 us).
template <int LOGN>
__global__ __launch_bounds__(Ntt<LOGN>::T) void k_encrypt(const uint32_t *pt, Tables T, const uint32_t *keys,
                                                          uint32_t *ct) {
  using C = Ntt<LOGN>;
  extern __shared__ uint32_t lds[];
  const uint32_t i = blockIdx.x % kL, k = (blockIdx.x / kL) & 1u;
  const uint64_t t = blockIdx.x / (2 * kL);
  const Prime P = T.p[i];
  uint32_t *o = ct + ((t * 2 + k) * kL + i) * C::N;
  const uint8_t *su = (const uint8_t *)o, *se = su + C::N;
  // part 0 uses b (the third key polynomial set), part 1 a
  const uint32_t *key = keys + ((uint64_t)(2 - k) * kL + i) * C::N;
  uint32_t v[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    const uint32_t x = su[threadIdx.x + c * C::T];
    v[c] = x ? x - 1u : P.q - 1u;
  }
  ntt_forward<LOGN>(v, lds, T.psi + (uint64_t)i * C::N, P.q);
#pragma unroll
  for (int c = 0; c < 16; ++c) v[c] = mont_q(key[ntt_pos<LOGN>(c)], v[c], P.q, P.qinv);
  ntt_inverse<LOGN>(v, lds, T.ipsi + (uint64_t)i * C::N, P);
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    const uint32_t x = se[threadIdx.x + c * C::T];
    v[c] = add_q(v[c], x >= kEta ? x - kEta : P.q + x - kEta, P.q);
  }
  if (k == 0) {
    const uint32_t *m = pt + (t * kL + i) * C::N;
#pragma unroll
    for (int c = 0; c < 16; ++c) v[c] = add_q(v[c], m[threadIdx.x + c * C::T], P.q);
  }
  __syncthreads();  // every sample of the region is read
#pragma unroll
  for (int c = 0; c < 16; ++c) o[threadIdx.x + c * C::T] = v[c];
}

// pt = c0 + INTT(NTT(c1) s) for one (ciphertext, prime), one launch instead of
// four.
template <int LOGN>
__global__ __launch_bounds__(Ntt<LOGN>::T) void k_decrypt(const uint32_t *ct, Tables T, const uint32_t *s, uint32_t *pt) {
  using C = Ntt<LOGN>;
  extern __shared__ uint32_t lds[];
  const uint32_t i = blockIdx.x % kL;
  const uint64_t t = blockIdx.x / kL;
  const Prime P = T.p[i];
  const uint32_t *c0 = ct + (t * 2 * kL + i) * C::N, *c1 = c0 + (uint64_t)kL * C::N;
  const uint32_t *key = s + (uint64_t)i * C::N;
  uint32_t v[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) v[c] = c1[threadIdx.x + c * C::T];
  ntt_forward<LOGN>(v, lds, T.psi + (uint64_t)i * C::N, P.q);
#pragma unroll
  for (int c = 0; c < 16; ++c) v[c] = mont_q(key[ntt_pos<LOGN>(c)], v[c], P.q, P.qinv);
  ntt_inverse<LOGN>(v, lds, T.ipsi + (uint64_t)i * C::N, P);
  uint32_t *o = pt + (t * kL + i) * C::N;
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    const uint32_t j = threadIdx.x + c * C::T;
    o[j] = add_q(v[c], c0[j], P.q);
  }
}

// ---- pointwise ----------------------------------------------------------------
// Key generation in the NTT domain: b = -a s + e, then a, b, s into
// Montgomery form.  All [L][N].
__global__ void k_keygen_finish(uint32_t n, Tables T, uint32_t *s, uint32_t *a, const uint32_t *e, uint32_t *b) {
  const uint64_t idx = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (uint64_t)kL * n) return;
  const Prime P = T.p[idx / n];
  const uint32_t sm = mont_q(s[idx], P.r2, P.q, P.qinv);  // s R
  const uint32_t am = mont_q(a[idx], P.r2, P.q, P.qinv);
  const uint32_t as = mont_q(am, s[idx], P.q, P.qinv);   // a s
  const uint32_t bv = sub_q(e[idx], as, P.q);
  b[idx] = mont_q(bv, P.r2, P.q, P.qinv);
  a[idx] = am;
  s[idx] = sm;
}

// out = x + y over sets of L residue polynomials of N = 2^log_n: `n` groups of
// four coefficients (VEC: 16-byte aligned buffers) or single ones per thread.
template <bool VEC>
__global__ __launch_bounds__(256) void k_add(uint32_t log_n, uint64_t n, Tables T, const uint32_t *x, const uint32_t *y,
                                             uint32_t *out) {
  const uint64_t idx = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= n) return;
  const uint32_t q = T.p[(idx >> (VEC ? log_n - 2 : log_n)) % kL].q;
  if constexpr (VEC) {
    const uint4 a = ((const uint4 *)x)[idx], b = ((const uint4 *)y)[idx];
    ((uint4 *)out)[idx] = make_uint4(add_q(a.x, b.x, q), add_q(a.y, b.y, q), add_q(a.z, b.z, q), add_q(a.w, b.w, q));
  } else {
    out[idx] = add_q(x[idx], y[idx], q);
  }
}

// ---- encoding FFT ---------------------------------------------------------------
// One block per vector; n = N/2 complex values in LDS.  The evaluation points
// zeta^(5^k) (zeta = e^(i pi / N)) are zeta^(1 + 4 t) with t = (5^k mod 2N -
// 1) / 4, so with u_j = m_j + i m_(j + n):
//   z_k = sum_j u_j zeta^j omega^(t j),  omega = e^(2 pi i / n),
// a length-n DFT of the twisted u read at t_k.  Encoding inverts it.
struct Cx {
  double re, im;
};
__device__ __forceinline__ Cx cmul(Cx a, Cx b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }

// Radix-2 DIT FFT of length n = 2^LOG (bit-reversed order in, natural out) by
// n / 8 threads; sign +1 for sum x_j w^(t j), -1 for the conjugate.  tw[k] =
// e^(2 pi i k / n), k < n/2.  Each thread runs up to three stages on eight
// values in registers: the vector crosses LDS every three stages instead of
// every one (13 at n = 2^13), by the same butterflies on the same values.  The
// values come from LDS and end in registers: value k of thread t is x[fft_pos(k)].
// One block per vector, so what a block issues bounds it: encoding and decoding
// a vector of 2^13 slots took 83 and 78 us and take 25 and 27.
template <int LOG>
struct Fft {
  static constexpr uint32_t n = 1u << LOG, T = n / 8;
  static constexpr int kLast = LOG % 3 == 0 ? 3 : 2;  // stages of the last pass (and of the one before, LOG % 3 == 1)
  static constexpr uint32_t kLds = n + n / 8;         // one value of padding after every 8
};
__device__ __forceinline__ uint32_t pad8(uint32_t i) { return i + (i >> 3); }
// Pass of R stages from half-length 2^E on: set k of 8 >> R per thread.
template <int LOG, int R, int E>
__device__ __forceinline__ uint32_t fft_base(int set) {
  const uint32_t id = threadIdx.x + Fft<LOG>::T * set;
  return ((id >> E) << (E + R)) + (id & ((1u << E) - 1u));
}
template <int LOG, int R, int E>
__device__ __forceinline__ void fft_pass(Cx (&v)[8], const Cx *x, const Cx *tw, int sign) {
#pragma unroll
  for (int set = 0; set < (8 >> R); ++set) {
    const uint32_t base = fft_base<LOG, R, E>(set), off = base & ((1u << E) - 1u);
    Cx *p = v + (set << R);
#pragma unroll
    for (int c = 0; c < (1 << R); ++c) p[c] = x[pad8(base + (c << E))];
#pragma unroll
    for (int i = 0; i < R; ++i) {
#pragma unroll
      for (int c = 0; c < (1 << R); ++c) {
        if (c & (1 << i)) continue;
        const uint32_t k = off + ((uint32_t)(c & ((1 << i) - 1)) << E);
        Cx w = tw[k << (LOG - E - i - 1)];
        if (sign < 0) w.im = -w.im;
        const Cx y = cmul(p[c + (1 << i)], w), u = p[c];
        p[c] = {u.re + y.re, u.im + y.im};
        p[c + (1 << i)] = {u.re - y.re, u.im - y.im};
      }
    }
  }
}
template <int LOG, int R, int E>
__device__ __forceinline__ void fft_store(const Cx (&v)[8], Cx *x) {
#pragma unroll
  for (int k = 0; k < 8; ++k) x[pad8(fft_base<LOG, R, E>(k >> R) + ((k & ((1 << R) - 1)) << E))] = v[k];
}
template <int LOG>
__device__ __forceinline__ uint32_t fft_pos(int k) {
  constexpr int R = Fft<LOG>::kLast, E = LOG - R;
  return fft_base<LOG, R, E>(k >> R) + ((k & ((1 << R) - 1)) << E);
}
template <int LOG, int E = 0>
__device__ __forceinline__ void fft_lds(Cx (&v)[8], Cx *x, const Cx *tw, int sign) {
  constexpr int left = LOG - E, R = left == 2 || left == 4 ? 2 : 3;
  __syncthreads();
  fft_pass<LOG, R, E>(v, x, tw, sign);
  if constexpr (left > R) {
    // a thread stores where it has read, so no other thread's values are lost
    fft_store<LOG, R, E>(v, x);
    fft_lds<LOG, E + R>(v, x, tw, sign);
  }
}

// z: [count][n_values] doubles (n_values <= N/2) -> pt [count][L][N].
template <int LOGN>
__global__ __launch_bounds__(Fft<LOGN - 1>::T) void k_encode(const double *z, uint32_t n_values, double scale,
                                                             const uint32_t *perm, const Cx *tw, const Cx *zeta,
                                                             Tables T, uint32_t *pt) {
  constexpr int LOG = LOGN - 1;
  constexpr uint32_t N = 1u << LOGN, n = N / 2;
  extern __shared__ Cx x[];
  const double *zz = z + (uint64_t)blockIdx.x * n_values;
#pragma unroll
  for (int k8 = 0; k8 < 8; ++k8) {
    const uint32_t k = threadIdx.x + k8 * Fft<LOG>::T;
    x[pad8(__brev(perm[k]) >> (32 - LOG))] = {k < n_values ? zz[k] * scale : 0.0, 0.0};
  }
  Cx v[8];
  fft_lds<LOG>(v, x, tw, -1);
  uint32_t *o = pt + (uint64_t)blockIdx.x * kL * N;
  const double inv_n = 1.0 / (double)n;
#pragma unroll
  for (int k8 = 0; k8 < 8; ++k8) {
    const uint32_t j = fft_pos<LOG>(k8);
    Cx c = v[k8];
    c.re *= inv_n;
    c.im *= inv_n;
    const Cx zc = {zeta[j].re, -zeta[j].im};  // zeta^-j
    const Cx u = cmul(c, zc);
    const int64_t lo = (int64_t)rint(u.re), hi = (int64_t)rint(u.im);
#pragma unroll
    for (int i = 0; i < kL; ++i) {
      o[(uint64_t)i * N + j] = to_residue(lo, T.p[i]);
      o[(uint64_t)i * N + j + n] = to_residue(hi, T.p[i]);
    }
  }
}

// Centered value of the residues r_i of one coefficient, as a double:
// Garner's mixed-radix digits, the integer x = d0 + q0 (d1 + q1 d2) in 128
// bits, x - Q when x > Q/2.
struct Crt {
  uint32_t q0_inv_q1;    // q0^-1 2^32 mod q1
  uint32_t q0q1_inv_q2;  // (q0 q1)^-1 2^32 mod q2
  uint32_t q0_q2;        // q0 2^32 mod q2
  uint64_t Q_lo, Q_hi;
};
__device__ __forceinline__ double crt_center(uint32_t r0, uint32_t r1, uint32_t r2, const Tables &T, const Crt &C) {
  // the primes lie between 2^29 and 2^30, so a residue of one is below twice another
  const uint32_t q0 = T.p[0].q, q1 = T.p[1].q, q2 = T.p[2].q;
  const uint32_t d0 = r0;
  const uint32_t d1 = mont_q(sub_q(r1, once(d0, q1), q1), C.q0_inv_q1, q1, T.p[1].qinv);
  // d2 = ((r2 - d0) q0^-1 - d1) q1^-1 mod q2 = (r2 - d0 - q0 d1) (q0 q1)^-1
  const uint32_t t = mont_q(once(d1, q2), C.q0_q2, q2, T.p[2].qinv);
  const uint32_t v = sub_q(sub_q(r2, once(d0, q2), q2), t, q2);
  const uint32_t d2 = mont_q(v, C.q0q1_inv_q2, q2, T.p[2].qinv);
  const unsigned __int128 x =
      (unsigned __int128)d0 + (unsigned __int128)q0 * ((unsigned __int128)d1 + (unsigned __int128)q1 * d2);
  const unsigned __int128 Q = ((unsigned __int128)C.Q_hi << 64) | C.Q_lo;
  const bool neg = x > (Q >> 1);
  const unsigned __int128 mag = neg ? Q - x : x;
  const double d = (double)(uint64_t)(mag >> 64) * 18446744073709551616.0 + (double)(uint64_t)mag;
  return neg ? -d : d;
}

// pt [count][L][N] -> z [count][n_values].
template <int LOGN>
__global__ __launch_bounds__(Fft<LOGN - 1>::T) void k_decode(const uint32_t *pt, uint32_t n_values, double inv_scale,
                                                             const uint32_t *perm, const Cx *tw, const Cx *zeta,
                                                             Tables T, Crt C, double *z) {
  constexpr int LOG = LOGN - 1;
  constexpr uint32_t N = 1u << LOGN, n = N / 2;
  extern __shared__ Cx x[];
  const uint32_t *p = pt + (uint64_t)blockIdx.x * kL * N;
#pragma unroll
  for (int k8 = 0; k8 < 8; ++k8) {
    const uint32_t j = threadIdx.x + k8 * Fft<LOG>::T;
    const double lo = crt_center(p[j], p[N + j], p[2 * N + j], T, C);
    const double hi = crt_center(p[j + n], p[N + j + n], p[2 * N + j + n], T, C);
    x[pad8(__brev(j) >> (32 - LOG))] = cmul({lo * inv_scale, hi * inv_scale}, zeta[j]);
  }
  Cx v[8];
  fft_lds<LOG>(v, x, tw, +1);
  __syncthreads();
#pragma unroll
  for (int k8 = 0; k8 < 8; ++k8) x[pad8(fft_pos<LOG>(k8))] = v[k8];
  __syncthreads();
  double *zz = z + (uint64_t)blockIdx.x * n_values;
  for (uint32_t k = threadIdx.x; k < n_values; k += Fft<LOG>::T) zz[k] = x[pad8(perm[k])].re;
}

// ---- host -----------------------------------------------------------------------
thread_local std::string g_err;
int fail(int code, const std::string &msg) {
  g_err = msg;
  return code;
}
#define CK_TRY(expr)                                          \
  do {                                                        \
    hipError_t e_ = (expr);                                   \
    if (e_ != hipSuccess) return fail(HE_ERR_DEVICE, hipGetErrorString(e_)); \
  } while (0)

uint64_t pow_mod(uint64_t b, uint64_t e, uint64_t m) {
  uint64_t r = 1 % m;
  b %= m;
  while (e) {
    if (e & 1) r = (unsigned __int128)r * b % m;
    b = (unsigned __int128)b * b % m;
    e >>= 1;
  }
  return r;
}
bool is_prime32(uint64_t q) {
  if (q < 2 || q % 2 == 0) return q == 2;
  // deterministic Miller-Rabin for q < 2^32 with bases 2, 7, 61
  uint64_t d = q - 1;
  int s = 0;
  while (d % 2 == 0) {
    d /= 2;
    ++s;
  }
  for (uint64_t a : {2ull, 7ull, 61ull}) {
    if (a % q == 0) continue;
    uint64_t x = pow_mod(a, d, q);
    if (x == 1 || x == q - 1) continue;
    bool comp = true;
    for (int r = 1; r < s; ++r) {
      x = (unsigned __int128)x * x % q;
      if (x == q - 1) {
        comp = false;
        break;
      }
    }
    if (comp) return false;
  }
  return true;
}
uint32_t bitrev(uint32_t x, uint32_t bits) {
  uint32_t r = 0;
  for (uint32_t b = 0; b < bits; ++b) r |= ((x >> b) & 1u) << (bits - 1 - b);
  return r;
}

}  // namespace

struct he_ckks {
  uint32_t log_n = 0, n = 0, scale_bits = 0;
  uint64_t seed = 0;
  Tables T{};
  Crt C{};
  uint32_t *d_tab = nullptr;   // psi and ipsi, each with its Shoup companion: 2 [L][N][2]
  uint32_t *d_keys = nullptr;  // s, a, b: 3 [L][N] (NTT domain, Montgomery form)
  uint32_t *d_perm = nullptr;  // t_k for k < N/2
  Cx *d_tw = nullptr;          // e^(2 pi i k / (N/2)), k < N/4
  Cx *d_zeta = nullptr;        // zeta^j, j < N/2
};

namespace {

inline uint32_t blocks(uint64_t n, uint32_t per) { return (uint32_t)((n + per - 1) / per); }

// f(integral_constant<log_n>) for this context's ring.
template <typename F>
void for_ring(uint32_t log_n, F f) {
  if (log_n == 12) f(std::integral_constant<int, 12>{});
  else if (log_n == 13) f(std::integral_constant<int, 13>{});
  else f(std::integral_constant<int, 14>{});
}

}  // namespace

extern "C" {

int he_ckks_create(uint32_t log_n, uint32_t scale_bits, uint64_t seed, he_ckks **out) {
  if (!out) return fail(HE_ERR_ARG, "null out");
  // Q is about 2^90: within the 128-bit classical security bounds of the
  // homomorphic encryption standard for a ternary secret (log Q at most 109
  // at N = 2^12, 218 at 2^13, 438 at 2^14), far outside them at N = 2^10 or
  // 2^11 (27 and 54), so smaller rings are refused.
  if (log_n < 12 || log_n > 14) return fail(HE_ERR_ARG, "log_n must be in [12, 14]");
  if (scale_bits < 10 || scale_bits > 60) return fail(HE_ERR_ARG, "scale_bits must be in [10, 60]");
  auto *c = new he_ckks();
  c->log_n = log_n;
  c->n = 1u << log_n;
  c->scale_bits = scale_bits;
  c->seed = seed;
  const uint32_t N = c->n;
  // primes: the largest below 2^30 that are 1 mod 2N
  std::vector<uint32_t> qs;
  for (uint64_t q = ((1ull << kPrimeBits) - 1) / (2 * N) * (2 * N) + 1; qs.size() < kL; q -= 2 * N)
    if (q < (1ull << kPrimeBits) && is_prime32(q)) qs.push_back((uint32_t)q);
  std::vector<uint32_t> tab(4ull * kL * N);
  for (int i = 0; i < kL; ++i) {
    const uint64_t q = qs[i];
    Prime &P = c->T.p[i];
    P.q = (uint32_t)q;
    uint32_t inv = 1;  // q^-1 mod 2^32 by Newton
    for (int k = 0; k < 5; ++k) inv *= 2u - (uint32_t)q * inv;
    P.qinv = 0u - inv;
    P.r1 = (uint32_t)((1ull << 32) % q);
    P.r2 = (uint32_t)(((unsigned __int128)1 << 64) % q);
    P.ninv = (uint32_t)pow_mod(N, q - 2, q);
    P.ninv_s = (uint32_t)(((uint64_t)P.ninv << 32) / q);
    uint64_t psi = 0;
    for (uint64_t g = 2; g < q; ++g) {
      const uint64_t cand = pow_mod(g, (q - 1) / (2 * N), q);
      if (pow_mod(cand, N, q) == q - 1) {
        psi = cand;
        break;
      }
    }
    const uint64_t ipsi = pow_mod(psi, q - 2, q);
    for (uint32_t k = 0; k < N; ++k) {
      const uint32_t e = bitrev(k, log_n);
      const uint64_t w = pow_mod(psi, e, q), iw = pow_mod(ipsi, e, q);
      uint32_t *t = &tab[2 * ((uint64_t)i * N + k)], *it = t + 2ull * kL * N;
      t[0] = (uint32_t)w;
      t[1] = (uint32_t)((w << 32) / q);
      it[0] = (uint32_t)iw;
      it[1] = (uint32_t)((iw << 32) / q);
    }
  }
  {
    const uint64_t q0 = qs[0], q1 = qs[1], q2 = qs[2];
    // in Montgomery form
    c->C.q0_inv_q1 = (uint32_t)((pow_mod(q0 % q1, q1 - 2, q1) << 32) % q1);
    c->C.q0q1_inv_q2 = (uint32_t)((pow_mod((unsigned __int128)q0 * q1 % q2, q2 - 2, q2) << 32) % q2);
    c->C.q0_q2 = (uint32_t)((q0 % q2 << 32) % q2);
    const unsigned __int128 Q = (unsigned __int128)q0 * q1 * q2;
    c->C.Q_lo = (uint64_t)Q;
    c->C.Q_hi = (uint64_t)(Q >> 64);
  }
  // encoding tables
  const uint32_t n = N / 2;
  std::vector<uint32_t> perm(n);
  uint64_t e = 1;
  for (uint32_t k = 0; k < n; ++k) {
    perm[k] = (uint32_t)((e - 1) / 4);
    e = e * 5 % (2ull * N);
  }
  std::vector<Cx> tw(n / 2), zeta(n);
  for (uint32_t k = 0; k < n / 2; ++k) tw[k] = {std::cos(2.0 * M_PI * k / n), std::sin(2.0 * M_PI * k / n)};
  for (uint32_t j = 0; j < n; ++j) zeta[j] = {std::cos(M_PI * j / N), std::sin(M_PI * j / N)};

  auto cleanup = [&](int rc) {
    he_ckks_free(c);
    return rc;
  };
  // The N/2-point FFT holds up to 144 KiB of LDS, the NTT up to 68 KiB: ask
  // for that much dynamic LDS (best effort; a size the device refuses shows
  // up as a launch error of the kernel).
  for_ring(log_n, [](auto ln) {
    constexpr int LN = decltype(ln)::value;
    const int fft = (int)(Fft<LN - 1>::kLds * sizeof(Cx)), ntt = (int)(Ntt<LN>::kLds * 4);
    (void)hipFuncSetAttribute((const void *)k_encode<LN>, hipFuncAttributeMaxDynamicSharedMemorySize, fft);
    (void)hipFuncSetAttribute((const void *)k_decode<LN>, hipFuncAttributeMaxDynamicSharedMemorySize, fft);
    (void)hipFuncSetAttribute((const void *)k_ntt<LN>, hipFuncAttributeMaxDynamicSharedMemorySize, ntt);
    (void)hipFuncSetAttribute((const void *)k_encrypt<LN>, hipFuncAttributeMaxDynamicSharedMemorySize, ntt);
    (void)hipFuncSetAttribute((const void *)k_decrypt<LN>, hipFuncAttributeMaxDynamicSharedMemorySize, ntt);
  });
  (void)hipGetLastError();
  if (hipMalloc(&c->d_tab, tab.size() * 4) != hipSuccess || hipMalloc(&c->d_keys, 3ull * kL * N * 4) != hipSuccess ||
      hipMalloc(&c->d_perm, n * 4) != hipSuccess || hipMalloc(&c->d_tw, tw.size() * sizeof(Cx)) != hipSuccess ||
      hipMalloc(&c->d_zeta, n * sizeof(Cx)) != hipSuccess)
    return cleanup(fail(HE_ERR_OOM, "out of device memory"));
  if (hipMemcpy(c->d_tab, tab.data(), tab.size() * 4, hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(c->d_perm, perm.data(), n * 4, hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(c->d_tw, tw.data(), tw.size() * sizeof(Cx), hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(c->d_zeta, zeta.data(), n * sizeof(Cx), hipMemcpyHostToDevice) != hipSuccess)
    return cleanup(fail(HE_ERR_DEVICE, "copy of the tables failed"));
  c->T.psi = (const uint2 *)c->d_tab;
  c->T.ipsi = c->T.psi + (uint64_t)kL * N;
  // keys: s (ternary), e (centered binomial), a (uniform); b = -a s + e
  uint32_t *s = c->d_keys, *a = s + kL * N, *b = a + kL * N, *ek = nullptr;
  if (hipMalloc(&ek, (size_t)kL * N * 4) != hipSuccess) return cleanup(fail(HE_ERR_OOM, "out of device memory"));
  const uint32_t g = blocks(N, 256);
  hipLaunchKernelGGL(k_sample, dim3(g), dim3(256), 0, 0, 0, seed, 0ull, N, c->T, s);
  hipLaunchKernelGGL(k_sample, dim3(g), dim3(256), 0, 0, 1, seed, kKeyEBase, N, c->T, ek);
  hipLaunchKernelGGL(k_sample, dim3(g), dim3(256), 0, 0, 2, seed, kKeyABase, N, c->T, a);
  for_ring(log_n, [&](auto ln) {
    constexpr int LN = decltype(ln)::value;
    for (uint32_t *x : {s, a, ek})
      hipLaunchKernelGGL(k_ntt<LN>, dim3(kL), dim3(Ntt<LN>::T), Ntt<LN>::kLds * 4, 0, x, c->T);
  });
  hipError_t err = hipGetLastError();
  if (err == hipSuccess) {
    hipLaunchKernelGGL(k_keygen_finish, dim3(blocks((uint64_t)kL * N, 256)), dim3(256), 0, 0, N, c->T, s, a, ek, b);
    err = hipGetLastError();
  }
  if (err == hipSuccess) err = hipDeviceSynchronize();
  hipFree(ek);
  if (err != hipSuccess) return cleanup(fail(HE_ERR_DEVICE, hipGetErrorString(err)));
  *out = c;
  return HE_OK;
}

void he_ckks_free(he_ckks *c) {
  if (!c) return;
  hipFree(c->d_tab);
  hipFree(c->d_keys);
  hipFree(c->d_perm);
  hipFree(c->d_tw);
  hipFree(c->d_zeta);
  delete c;
}

int he_ckks_params(const he_ckks *c, uint32_t *n, uint32_t *primes, uint32_t *scale_bits) {
  if (!c) return fail(HE_ERR_ARG, "null context");
  if (n) *n = c->n;
  if (primes)
    for (int i = 0; i < kL; ++i) primes[i] = c->T.p[i].q;
  if (scale_bits) *scale_bits = c->scale_bits;
  return HE_OK;
}

int he_ckks_encode(const he_ckks *c, const double *z, uint64_t count, uint32_t n_values, uint32_t *pt,
                   hipStream_t s) {
  if (!c) return fail(HE_ERR_ARG, "null context");
  if (n_values > c->n / 2) return fail(HE_ERR_ARG, "n_values exceeds N/2 slots");
  if (count == 0) return HE_OK;
  if (!pt || (n_values && !z)) return fail(HE_ERR_ARG, "null z or pt");
  if (count > 0x7FFFFFFFull) return fail(HE_ERR_ARG, "count too large");
  for_ring(c->log_n, [&](auto ln) {
    constexpr int LN = decltype(ln)::value;
    hipLaunchKernelGGL(k_encode<LN>, dim3((uint32_t)count), dim3(Fft<LN - 1>::T), Fft<LN - 1>::kLds * sizeof(Cx), s, z,
                       n_values, std::ldexp(1.0, (int)c->scale_bits), c->d_perm, c->d_tw, c->d_zeta, c->T, pt);
  });
  CK_TRY(hipGetLastError());
  return HE_OK;
}

int he_ckks_decode(const he_ckks *c, const uint32_t *pt, uint64_t count, uint32_t n_values, double *z,
                   hipStream_t s) {
  if (!c) return fail(HE_ERR_ARG, "null context");
  if (n_values > c->n / 2) return fail(HE_ERR_ARG, "n_values exceeds N/2 slots");
  if (count == 0 || n_values == 0) return HE_OK;
  if (!pt || !z) return fail(HE_ERR_ARG, "null pt or z");
  if (count > 0x7FFFFFFFull) return fail(HE_ERR_ARG, "count too large");
  for_ring(c->log_n, [&](auto ln) {
    constexpr int LN = decltype(ln)::value;
    hipLaunchKernelGGL(k_decode<LN>, dim3((uint32_t)count), dim3(Fft<LN - 1>::T), Fft<LN - 1>::kLds * sizeof(Cx), s,
                       pt, n_values, std::ldexp(1.0, -(int)c->scale_bits), c->d_perm, c->d_tw, c->d_zeta, c->T, c->C,
                       z);
  });
  CK_TRY(hipGetLastError());
  return HE_OK;
}

int he_ckks_encrypt(he_ckks *c, const uint32_t *pt, uint64_t count, uint64_t seed, uint64_t offset, uint32_t *ct,
                    hipStream_t s) {
  if (!c) return fail(HE_ERR_ARG, "null context");
  if (count == 0) return HE_OK;
  if (!pt || !ct) return fail(HE_ERR_ARG, "null pt or ct");
  if (count * 2 * kL > 0x7FFFFFFFull || count * c->n > 0xFFFFFFFFull) return fail(HE_ERR_ARG, "count too large");
  const uint64_t quads = count * (c->n / 4);
  hipLaunchKernelGGL(k_sample_enc, dim3(blocks(quads, 256)), dim3(256), 0, s, seed, offset, c->log_n, quads, ct);
  CK_TRY(hipGetLastError());
  for_ring(c->log_n, [&](auto ln) {
    constexpr int LN = decltype(ln)::value;
    hipLaunchKernelGGL(k_encrypt<LN>, dim3((uint32_t)(count * kL * 2)), dim3(Ntt<LN>::T), Ntt<LN>::kLds * 4, s, pt,
                       c->T, c->d_keys, ct);
  });
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    // ct holds u, e0 and e1 in clear: they must not reach the caller
    (void)he::launch_fill(ct, 2 * count * kL * (uint64_t)c->n, 0u, s);
    return fail(HE_ERR_DEVICE, hipGetErrorString(e));
  }
  return HE_OK;
}

int he_ckks_add(const he_ckks *c, const uint32_t *x, const uint32_t *y, uint64_t count, uint32_t *out,
                hipStream_t s) {
  if (!c) return fail(HE_ERR_ARG, "null context");
  if (count == 0) return HE_OK;
  if (!x || !y || !out) return fail(HE_ERR_ARG, "null x, y or out");
  const uint64_t words = 2 * count * kL * (uint64_t)c->n;
  if ((((uintptr_t)x | (uintptr_t)y | (uintptr_t)out) & 15u) == 0)
    hipLaunchKernelGGL(k_add<true>, dim3(blocks(words / 4, 256)), dim3(256), 0, s, c->log_n, words / 4, c->T, x, y, out);
  else
    hipLaunchKernelGGL(k_add<false>, dim3(blocks(words, 256)), dim3(256), 0, s, c->log_n, words, c->T, x, y, out);
  CK_TRY(hipGetLastError());
  return HE_OK;
}

int he_ckks_decrypt(const he_ckks *c, const uint32_t *ct, uint64_t count, uint32_t *pt, hipStream_t s) {
  if (!c) return fail(HE_ERR_ARG, "null context");
  if (count == 0) return HE_OK;
  if (!ct || !pt) return fail(HE_ERR_ARG, "null ct or pt");
  if (count * kL > 0x7FFFFFFFull) return fail(HE_ERR_ARG, "count too large");
  for_ring(c->log_n, [&](auto ln) {
    constexpr int LN = decltype(ln)::value;
    hipLaunchKernelGGL(k_decrypt<LN>, dim3((uint32_t)(count * kL)), dim3(Ntt<LN>::T), Ntt<LN>::kLds * 4, s, ct, c->T,
                       c->d_keys, pt);
  });
  CK_TRY(hipGetLastError());
  return HE_OK;
}

const char *he_ckks_last_error(void) { return g_err.c_str(); }

}  // extern "C"
