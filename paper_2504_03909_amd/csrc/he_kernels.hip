// gfx950 kernels of the Paillier histogram path: fixed-point encoding,
// encryption (CRT and public-key), Montgomery conversion, histogram
// aggregation (bucketing + chunked ciphertext products) and CRT decryption.
//
// Layout conventions: one big integer per 16-lane group (see mont.hpp);
// 256-thread blocks = 4 waves = 16 groups; every group owns one LDS row.
// Kernels keep all 64 lanes of a wave active until they return; groups with
// no work compute on a valid dummy item and do not store.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <map>
#include <mutex>
#include <tuple>

#include "he_internal.hpp"
#include "hist_bucket.hpp"
#include "hist_pair.hpp"
#include "mont.hpp"
#include "mont29.hpp"

namespace he {

static_assert(kWindow == kWindowBits, "window width mismatch");

// ------------------------------------------------------------- small helpers
// Limb t of a little-endian buffer of `nl` limbs, zero past the end.
template <int K, int G = 16>
__device__ __forceinline__ void ld_part(uint32_t (&x)[K], const uint32_t *p, int nl) {
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const int t = (int)glane<G>() * K + j;
    x[j] = t < nl ? p[t] : 0u;
  }
}

// x = v mod N for a signed 64-bit v (|v| < N).
template <int K, int G = 16>
__device__ __forceinline__ void signed_mod(uint32_t (&x)[K], int64_t v, const uint32_t (&N)[K]) {
  const uint64_t mag = v < 0 ? (uint64_t)0 - (uint64_t)v : (uint64_t)v;
  uint32_t a[K];
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const int t = (int)glane<G>() * K + j;
    a[j] = t == 0 ? (uint32_t)mag : (t == 1 ? (uint32_t)(mag >> 32) : 0u);
  }
  if (v < 0) {
    uint32_t d[K];
    sub_plain<K, G>(d, N, a);
    copy(x, d);
  } else {
    copy(x, a);
  }
}

// x += 1 (no reduction).
template <int K, int G = 16>
__device__ __forceinline__ void add_one(uint32_t (&x)[K]) {
  uint32_t one[K];
  set_small<K, G>(one, 1u);
  add_plain<K, G>(x, x, one);
}

// Limbs [first, first + G K) of the seeded stream integer
// X = sum_j w(seed, base + j) 2^(64 j), each lane taking its K limbs;
// limbs at or past `nl` are zero.
template <int K, int G = 16>
__device__ __forceinline__ void seeded_limbs(uint32_t (&x)[K], uint64_t seed, uint64_t base,
                                             int first, int nl) {
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const int t = first + (int)glane<G>() * K + j;
    const uint64_t w = splitmix64(seed, base + (uint64_t)(t >> 1));
    x[j] = t < nl ? (uint32_t)((t & 1) ? (w >> 32) : w) : 0u;
  }
}

__device__ __forceinline__ uint32_t group_in_wave() { return (threadIdx.x >> 4) & 3u; }

// ------------------------------------------------------------------- encode
__global__ void k_encode(const double *__restrict__ x, uint64_t count, uint32_t frac_bits,
                         int64_t *__restrict__ m, uint32_t *__restrict__ n_bad) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) {
    const double v = ldexp(x[i], (int)frac_bits);  // exact scaling by a power of two
    if (!(fabs(v) < 9223372036854775808.0)) {
      m[i] = INT64_MIN;
      if (n_bad) atomicAdd(n_bad, 1u);
    } else {
      m[i] = (int64_t)rint(v);  // round to nearest, ties to even
    }
  }
}

// ----------------------------------------------------- private-key exponentiation
// k_pow: x_u <- x_u^(e_P) mod P for units u = (ciphertext i, prime P) at 2 to 16
// lanes per integer, the radix-2^29 exponentiation alone (the products around
// it run in the 16-lane kernels below, so this kernel holds nothing but the
// exponentiation's own state).  Powers mod P^2 and mod n^2, and mod P with one
// integer per lane, run in k_pow_pair (pow_pair.hpp).  Unit (i, w) reads
// in_limbs limbs at in + (2 i + w) in_stride (zero-extended to S32) and writes
// S32 canonical limbs at out + (2 i + w) out_stride.  Work unit = (prime, 64/G
// consecutive ciphertexts), so the modulus and exponent are the same for the
// whole wave.  For secret exponents: every table entry is read.  At most 3 waves per SIMD:
// the 18-limb-per-lane shape needs about 168 VGPRs to run its step loops
// without spills.  With `next` (a counter zeroed before the launch) the waves
// claim units as they finish them, so they end together; without, wave w takes
// units w, w + waves, ...
struct PowArgs {
  DMod mod[2];
  DExp exp[2];
  const uint32_t *in;
  uint32_t *out;
  uint32_t in_stride, in_limbs, out_stride;
  uint64_t count;
  uint32_t *tabs;
  uint32_t *next;
};

template <int S32, int G>
__global__ __launch_bounds__(kBlockThreads, 3) void k_pow(PowArgs a) {
  constexpr int K32 = S32 / G, NG = 64 / G, GB = kBlockThreads / G;
  constexpr int S29 = he29::limbs_for_group(S32, G), ROW = 2 * S29 > S32 ? 2 * S29 : S32;
  __shared__ __align__(16) uint32_t lds_all[GB * ROW + S29];
  uint32_t *const zeros = lds_all + GB * ROW;
  zero_lds(zeros, S29);
  const uint32_t g = (threadIdx.x & 63u) / G;
  uint32_t *lds = lds_all + (threadIdx.x / G) * ROW;
  const uint64_t gw = (uint64_t)blockIdx.x * 4 + wave_in_block();
  const uint64_t nw = (uint64_t)gridDim.x * 4;
  uint32_t *tab = a.tabs + (gw * NG + g) * (uint64_t)((kTable + 1) * S29);
  const uint64_t nunits = 2 * ((a.count + NG - 1) / NG);
  for (uint64_t qd = a.next ? claim_unit(a.next) : gw; qd < nunits; qd = a.next ? claim_unit(a.next) : qd + nw) {
    const int which = (int)(qd & 1);
    uint64_t i = (qd >> 1) * NG + g;
    const bool valid = i < a.count;
    if (!valid) i = a.count - 1;
    const uint64_t u = i * 2 + which;
    uint32_t x[K32];
    ld_part<K32, G>(x, a.in + u * a.in_stride, (int)a.in_limbs);
    pow29<K32, G>(x, a.exp[which], tab, a.mod[which], lds, zeros);
    if (valid) st<K32, G>(a.out + u * a.out_stride, x);
  }
}

// ----------------------------------------------------------- CRT encryption
// For each (ciphertext i, prime P):
//   c_P = (1 + m n) r^n mod P^2,  r^n mod P^2 = (r^(Q mod (P-1)) mod P)^P mod P^2
// (x -> x^P mod P^2 depends only on x mod P), and 1 + m n = 1 + P (m Q mod P)
// mod P^2.  k_enc_r reduces r mod P, k_pow_joint computes omega = r^n mod P^2
// as two digits base P (with secret digits, in two steps: k_pow t = r^(Q mod
// (P-1)) mod P, k_pow_pair t^P), and k_enc_crt_b forms c_P = omega (1 + P (m Q
// mod P)) and combines c_p, c_q by the CRT.

// r mod P for each (ciphertext i, prime P) into tq[2 i + P] (S_P limbs): r's
// S_P-limb words w_k (two for an explicit r, three for the seeded one), each
// times R^k mod P by a Montgomery product with R^(k+1) mod P, summed.  One
// 16-lane group per (i, P).
template <int KP>
__global__ __launch_bounds__(kBlockThreads) void k_enc_r(DKey key, uint64_t count, const uint32_t *__restrict__ r,
                                                        uint64_t seed, uint64_t roff, uint32_t *__restrict__ tq) {
  constexpr int SP = 16 * KP, L = 32 * KP;
  __shared__ __align__(16) uint32_t lds_all[16 * SP];
  const uint32_t gi = wave_in_block() * 4 + group_in_wave();
  uint32_t *lds = lds_all + gi * SP;
  uint64_t u = (uint64_t)blockIdx.x * 16 + gi;
  const bool valid = u < 2 * count;
  if (!valid) u = 2 * count - 1;
  const uint64_t i = u >> 1;
  const DPrime &P = key.pr[u & 1];
  const Mod<KP> Mp = load_mod<KP>(P.P.N, P.P.ninv);
  const uint64_t W = (uint64_t)SP + 1;  // stream words per r
  const uint64_t base = (roff + i) * W;
  const int words = r ? 2 : 3;
  uint32_t x[KP], t[KP], c[KP];
  set_zero(x);
#pragma unroll 1
  for (int k = 0; k < words; ++k) {
    if (r)
      ld<KP>(t, r + i * L + k * SP);
    else
      seeded_limbs<KP>(t, seed, base, k * SP, 2 * SP + 2);
    ld<KP>(c, k == 0 ? P.P.R1 : (k == 1 ? P.P.R2 : P.P.R3));
    mont_mul<KP>(t, t, c, Mp, lds);
    add_mod<KP>(x, x, t, Mp);
  }
  if (valid) st<KP>(tq + u * SP, x);
}

// c_P = omega_P (1 + P (m Q mod P)) mod P^2 for both primes, then
// c = c_q + q^2 ((c_p - c_q) (q^2)^-1 mod p^2), the CRT to mod n^2.  One
// 16-lane group per ciphertext.
template <int KP>
__global__ __launch_bounds__(kBlockThreads) void k_enc_crt_b(DKey key, const int64_t *__restrict__ m,
                                                            const uint32_t *__restrict__ cpq, uint64_t count,
                                                            uint32_t *__restrict__ ct) {
  constexpr int KP2 = 2 * KP, KN2 = 4 * KP, SP2 = 32 * KP, SN2 = 64 * KP;
  __shared__ __align__(16) uint32_t lds_all[16 * SN2];
  const uint32_t gi = wave_in_block() * 4 + group_in_wave();
  uint32_t *lds = lds_all + gi * SN2;
  uint64_t i = (uint64_t)blockIdx.x * 16 + gi;
  const bool valid = i < count;
  if (!valid) i = count - 1;
  const int64_t mi = m ? m[i] : 0;
  uint32_t cw[2][KP2];
#pragma unroll 1
  for (int which = 0; which < 2; ++which) {
    // omega = a + e P (its digits), f = 1 + P u with u = m Q mod P:
    // omega f = a + P (e + a u mod P) mod P^2
    const DPrime &P = key.pr[which];
    const uint32_t *om = cpq + (i * 2 + which) * SP2;
    uint32_t f[KP2], a2[KP2], c2[KP2];
    {
      const Mod<KP> Mp = load_mod<KP>(P.P.N, P.P.ninv);
      uint32_t u[KP], a[KP], e[KP];
      signed_mod<KP>(u, mi, Mp.n);
      ld<KP>(a, P.QR2_P);
      mont_mul<KP>(u, u, a, Mp, lds);  // u R
      ld<KP>(a, om);
      mont_mul<KP>(u, u, a, Mp, lds);  // a u
      ld<KP>(e, om + SP2 / 2);
      add_mod<KP>(u, u, e, Mp);
      relayout<KP, KP2>(f, u, lds);
      relayout<KP, KP2>(a2, a, lds);
    }
    const Mod<KP2> M2 = load_mod<KP2>(P.P2.N, P.P2.ninv);
    ld<KP2>(c2, P.PR_P2);
    mont_mul<KP2>(f, f, c2, M2, lds);
    add_plain<KP2>(cw[which], f, a2);
  }
  const DPrime &Pp = key.pr[0];
  const Mod<KP2> M2 = load_mod<KP2>(Pp.P2.N, Pp.P2.ninv);
  uint32_t c[KP2], a[KP2], b[KP2];
  ld<KP2>(c, key.Cq);
  mont_mul<KP2>(a, cw[0], c, M2, lds);
  mont_mul<KP2>(b, cw[1], c, M2, lds);
  sub_mod<KP2>(a, a, b, M2);
  const Mod<KN2> Mn2 = load_mod<KN2>(key.n2.N, key.n2.ninv);
  uint32_t u[KN2], cq4[KN2], k4[KN2];
  relayout<KP2, KN2>(u, a, lds);
  relayout<KP2, KN2>(cq4, cw[1], lds);
  ld<KN2>(k4, key.q2R_n2);
  mont_mul<KN2>(u, u, k4, Mn2, lds);
  add_plain<KN2>(u, u, cq4);
  if (valid) st<KN2>(ct + i * SN2, u);
}

// ------------------------------------------------------ public-key encryption
// c = (1 + (m mod n) n) r^n mod n^2 by one exponentiation mod n^2, in three
// launches like the CRT path: k_pub_pre reduces r mod n (r^n mod n^2 depends
// only on r mod n), k_pow_pair raises it to n in two digits base n (its units
// of both "primes" are n, so a unit pair covers two consecutive ciphertexts),
// k_pub_post multiplies by 1 + (m mod n) n.  One 16-lane group per ciphertext
// in the light kernels.  x has count + (count & 1) rows: an odd count's last row is repeated, so the
// exponentiation's last unit pair reads and writes a row of its own.
template <int KP>
__global__ __launch_bounds__(kBlockThreads) void k_pub_pre(DKey key, uint64_t count, const uint32_t *__restrict__ r,
                                                          uint64_t seed, uint64_t roff, uint32_t *__restrict__ x) {
  constexpr int KN = 2 * KP, L = 32 * KP;
  __shared__ __align__(16) uint32_t lds_all[16 * L];
  const uint32_t gi = wave_in_block() * 4 + group_in_wave();
  uint32_t *lds = lds_all + gi * L;
  const uint64_t rows = count + (count & 1);
  uint64_t row = (uint64_t)blockIdx.x * 16 + gi;
  const bool valid = row < rows;
  if (!valid) row = rows - 1;
  const uint64_t i = row < count ? row : count - 1;
  const uint64_t W = (uint64_t)L / 2 + 1;
  const Mod<KN> M = load_mod<KN>(key.n.N, key.n.ninv);
  // r's L-limb words w_k (one for an explicit r, two for the seeded one), each
  // times R^k mod n by a Montgomery product with R^(k+1) mod n, summed
  uint32_t v[KN], t[KN], c[KN];
  set_zero(v);
#pragma unroll 1
  for (int k = 0; k < (r ? 1 : 2); ++k) {
    if (r)
      ld<KN>(t, r + i * L);
    else
      seeded_limbs<KN>(t, seed, (roff + i) * W, k * L, L + 2);
    ld<KN>(c, k == 0 ? key.n.R1 : key.n.R2);
    mont_mul<KN>(t, t, c, M, lds);
    add_mod<KN>(v, v, t, M);
  }
  if (valid) st<KN>(x + row * L, v);
}

// ct = (a + e n) (1 + m n) = a + n (e + a m mod n) mod n^2.
template <int KP>
__global__ __launch_bounds__(kBlockThreads) void k_pub_post(DKey key, const int64_t *__restrict__ m, uint64_t count,
                                                           const uint32_t *__restrict__ x, uint32_t *__restrict__ ct) {
  constexpr int KN = 2 * KP, KN2 = 4 * KP, SN2 = 64 * KP, L = 32 * KP;
  __shared__ __align__(16) uint32_t lds_all[16 * SN2];
  const uint32_t gi = wave_in_block() * 4 + group_in_wave();
  uint32_t *lds = lds_all + gi * SN2;
  uint64_t i = (uint64_t)blockIdx.x * 16 + gi;
  const bool valid = i < count;
  if (!valid) i = count - 1;
  uint32_t f[KN2], a2[KN2], c2[KN2];
  {
    const Mod<KN> Mn = load_mod<KN>(key.n.N, key.n.ninv);
    uint32_t u[KN], a[KN], e[KN];
    signed_mod<KN>(u, m ? m[i] : 0, Mn.n);
    ld<KN>(a, key.n.R2);
    mont_mul<KN>(u, u, a, Mn, lds);  // m R
    ld<KN>(a, x + i * SN2);
    mont_mul<KN>(u, u, a, Mn, lds);  // a m
    ld<KN>(e, x + i * SN2 + L);
    add_mod<KN>(u, u, e, Mn);
    relayout<KN, KN2>(f, u, lds);
    relayout<KN, KN2>(a2, a, lds);
  }
  const Mod<KN2> M = load_mod<KN2>(key.n2.N, key.n2.ninv);
  ld<KN2>(c2, key.nR_n2);
  mont_mul<KN2>(f, f, c2, M, lds);
  add_plain<KN2>(f, f, a2);
  if (valid) st<KN2>(ct + i * SN2, f);
}

// ------------------------------------------------ obfuscated encryption
// ct = (1 + (m mod n) n) rho mod n^2 with a precomputed obfuscator
// rho = r^n mod n^2 (canonical).  Since (1 + m n) rho = rho + n (m rho) and
// n x mod n^2 = n (x mod n), ct = rho + n t mod n^2 with t = m rho mod n:
// three products mod n (rho R mod n from rho's halves, then times m) and
// one mod n^2 (n t), instead of three mod n^2.  Without m: m = 2^63, the offset of
// a packed slot, for packing one ciphertext to one.
template <int KP>
__global__ __launch_bounds__(kBlockThreads) void k_enc_obf(DKey key, const int64_t *__restrict__ m,
                                                          uint64_t count, const uint32_t *rho,
                                                          uint32_t *ct) {
  constexpr int KN = 2 * KP, KN2 = 4 * KP, SN2 = 64 * KP, L = 32 * KP;
  __shared__ __align__(16) uint32_t lds_all[16 * SN2];
  const uint32_t gi = wave_in_block() * 4 + group_in_wave();
  uint32_t *lds = lds_all + gi * SN2;
  uint64_t i = (uint64_t)blockIdx.x * 16 + gi;
  const bool valid = i < count;
  if (!valid) i = count - 1;
  uint32_t t2[KN2];
  {
    // t = m rho mod n: s = rho0 R + rho1 R^2 = rho R (mod n) from the halves
    // rho = rho0 + rho1 R (R = 2^(32 L)), then t = s (m mod n) R^-1
    const Mod<KN> Mn = load_mod<KN>(key.n.N, key.n.ninv);
    uint32_t a[KN], b[KN], c[KN];
    ld<KN>(a, rho + i * SN2);
    ld<KN>(c, key.n.R2);
    mont_mul<KN>(a, a, c, Mn, lds);
    ld<KN>(b, rho + i * SN2 + L);
    ld<KN>(c, key.n.R3);
    mont_mul<KN>(b, b, c, Mn, lds);
    add_mod<KN>(a, a, b, Mn);
    if (m) {
      signed_mod<KN>(b, m[i], Mn.n);
    } else {
#pragma unroll
      for (int j = 0; j < KN; ++j) b[j] = (int)glane() * KN + j == 1 ? 0x80000000u : 0u;
    }
    mont_mul<KN>(a, a, b, Mn, lds);
    relayout<KN, KN2>(t2, a, lds);
  }
  // ct = rho + n t mod n^2 (n t by one product with n R' mod n^2)
  const Mod<KN2> M = load_mod<KN2>(key.n2.N, key.n2.ninv);
  uint32_t x[KN2], c[KN2];
  ld<KN2>(c, key.nR_n2);
  mont_mul<KN2>(t2, t2, c, M, lds);
  ld<KN2>(x, rho + i * SN2);
  add_mod<KN2>(x, x, t2, M);
  if (valid) st<KN2>(ct + i * SN2, x);
}

// J = Q^-1 R mod n^2 for Q < n^2; false (group-uniform) where Q is no unit.  The
// inverse is taken mod n only -- half the limbs and half the steps of the serial
// binary algorithm, about a quarter of its time -- and lifted: with y = Q^-1 mod
// n, Q^-1 = y (2 - Q y) mod n^2, four products.  Q is a unit mod n^2 where it is
// one mod n.
template <int KP>
__device__ __forceinline__ bool inverse_n2(uint32_t (&J)[4 * KP], const uint32_t (&Q)[4 * KP], const DKey &key,
                                           const Mod<4 * KP> &M, uint32_t *lds, bool active) {
  constexpr int KN = 2 * KP, KN2 = 4 * KP, L = 32 * KP;
  bool ok;
  uint32_t t[KN2], u[KN2], c2[KN2];
  {
    const Mod<KN> Mn = load_mod<KN>(key.n.N, key.n.ninv);
    uint32_t lo[KN], hi[KN], c[KN];
    relayout<KN2, KN>(lo, Q, lds);
    relayout<KN2, KN>(hi, Q, lds, L);
    ld<KN>(c, key.n.R1);
    mont_mul<KN>(lo, lo, c, Mn, lds);
    ld<KN>(c, key.n.R2);
    mont_mul<KN>(hi, hi, c, Mn, lds);
    add_mod<KN>(lo, lo, hi, Mn);  // Q mod n
    ok = mont_inverse<KN>(hi, lo, Mn, key.n.R2, lds, active);
    set_small<KN>(c, 1u);
    mont_mul<KN>(hi, hi, c, Mn, lds);
    relayout<KN, KN2>(t, hi, lds);  // y
  }
  ld<KN2>(c2, key.n2.R2);
  mont_mul<KN2>(t, t, c2, M, lds);  // y R
  mont_mul<KN2>(J, Q, t, M, lds);   // Q y
  set_small<KN2>(u, 2u);
  sub_mod<KN2>(u, u, J, M);
  mont_mul<KN2>(u, u, c2, M, lds);
  mont_mul<KN2>(J, t, u, M, lds);
  return ok;
}

// ------------------------------------------------------ ciphertext division
// out[i] = num[i] den[i]^-1 mod n^2, i.e. an encryption of m_num - m_den.
// Montgomery's batch-inversion trick per group of `batch` consecutive
// elements: prefix products Q_j = Q_(j-1) a_j R^-1 (Q_0 = a_0, stored in
// `out`), one inversion J = Q_last^-1 R, then backwards a_j^-1 R =
// J Q_(j-1) R^-1 and J <- J a_j R^-1 = Q_(j-1)^-1 R -- four Montgomery
// products per element plus one inversion per batch.  A batch whose product
// is not invertible is redone element by element; elements whose den is
// not a unit mod n^2 get 0 and are counted into *n_bad.
template <int KP>
__global__ __launch_bounds__(kBlockThreads) void k_ct_div(DKey key, const uint32_t *__restrict__ num,
                                                         const uint32_t *__restrict__ den, uint64_t count,
                                                         uint32_t batch, uint32_t *__restrict__ out,
                                                         uint32_t *__restrict__ n_bad) {
  constexpr int KN2 = 4 * KP, SN2 = 64 * KP;
  __shared__ __align__(16) uint32_t lds_all[16 * SN2];
  const uint32_t gi = wave_in_block() * 4 + group_in_wave();
  uint32_t *lds = lds_all + gi * SN2;
  const uint64_t first = ((uint64_t)blockIdx.x * 16 + gi) * batch;
  const uint32_t len = first < count ? (uint32_t)min((uint64_t)batch, count - first) : 0u;
  const Mod<KN2> M = load_mod<KN2>(key.n2.N, key.n2.ninv);

  // forward: prefix products
  uint32_t Q[KN2], a[KN2], t[KN2];
  set_zero(Q);
  set_zero(a);
  if (len) {
    ld<KN2>(Q, den + first * SN2);
    st<KN2>(out + first * SN2, Q);
  }
#pragma unroll 1
  for (uint32_t j = 1; j < batch; ++j) {
    const bool v = j < len;
    if (v) ld<KN2>(a, den + (first + j) * SN2);
    mont_mul<KN2>(t, Q, a, M, lds);
    select(Q, v, t, Q);
    if (v) st<KN2>(out + (first + j) * SN2, Q);
  }

  uint32_t J[KN2];
  const bool ok = inverse_n2<KP>(J, Q, key, M, lds, len > 0u);

  // backward
  uint32_t p[KN2], ainv[KN2];
  set_zero(p);
#pragma unroll 1
  for (uint32_t j = batch; j-- > 0u;) {
    const bool v = ok && j < len;
    if (j > 0u) {
      if (v) ld<KN2>(t, out + (first + j - 1) * SN2);
      mont_mul<KN2>(ainv, J, t, M, lds);
      if (v) ld<KN2>(a, den + (first + j) * SN2);
      mont_mul<KN2>(t, J, a, M, lds);
      select(J, v, t, J);
    } else {
      copy(ainv, J);
    }
    if (v) ld<KN2>(p, num + (first + j) * SN2);
    mont_mul<KN2>(p, p, ainv, M, lds);
    if (v) st<KN2>(out + (first + j) * SN2, p);
  }

  // element-by-element retry for batches that held a non-unit
  const bool retry = len > 0u && !ok;
  if (wave_any(retry)) {
#pragma unroll 1
    for (uint32_t j = 0; j < batch; ++j) {
      const bool v = retry && j < len;
      if (v) {
        ld<KN2>(a, den + (first + j) * SN2);
        ld<KN2>(p, num + (first + j) * SN2);
      }
      const bool ok1 = inverse_n2<KP>(J, a, key, M, lds, v);
      mont_mul<KN2>(p, p, J, M, lds);
      if (!ok1) set_zero(p);
      if (v) st<KN2>(out + (first + j) * SN2, p);
      if (v && !ok1 && glane() == 0 && n_bad) atomicAdd(n_bad, 1u);
    }
  }
}

// ------------------------------------------------------ split finding
// Best split per (node, feature) and per node from decrypted histograms:
// exact int64 prefix sums over the bins, XGBoost's gain in IEEE double with
// no contraction (every operation rounded as written), the largest gain with
// the lowest bin, then the lowest feature, on ties.  One block per node; each
// wave takes every fourth feature, lane l holds bins 4l .. 4l + 3.
struct SplitCand {
  double gain;
  int32_t feature, bin;
  int64_t gl, hl;
};

__device__ __forceinline__ bool split_better(const SplitCand &a, const SplitCand &b, bool by_feature) {
  if (a.gain > b.gain) return true;
  if (a.gain < b.gain || a.bin < 0) return false;
  if (b.bin < 0) return true;
  return by_feature ? a.feature < b.feature : a.bin < b.bin;
}

__device__ __forceinline__ SplitCand shfl_xor_cand(const SplitCand &c, int m) {
  SplitCand o;
  o.gain = __shfl_xor(c.gain, m, 64);
  o.feature = __shfl_xor(c.feature, m, 64);
  o.bin = __shfl_xor(c.bin, m, 64);
  o.gl = __shfl_xor(c.gl, m, 64);
  o.hl = __shfl_xor(c.hl, m, 64);
  return o;
}

__device__ __forceinline__ double split_term(double g, double h, double lam) {
#pragma clang fp contract(off)
  return (g * g) / (h + lam);
}

__global__ __launch_bounds__(kBlockThreads) void k_split(const int64_t *hist, const int64_t *minus, uint32_t F,
                                                        uint32_t B, double scale, double lam, double gamma,
                                                        double mcw, int64_t *derived, SplitCand *out_feat,
                                                        SplitCand *out_node) {
#pragma clang fp contract(off)
  __shared__ SplitCand waves[kBlockThreads / 64];
  const uint64_t node = blockIdx.x;
  const uint32_t w = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  const SplitCand none = {-__builtin_inf(), -1, -1, 0, 0};
  SplitCand best = none;
  for (uint32_t f = w; f < F; f += kBlockThreads / 64) {
    const uint64_t base = (node * F + f) * (uint64_t)B * 2;
    int64_t g[4], h[4], sg = 0, sh = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t b = lane * 4 + k;
      g[k] = h[k] = 0;
      if (b < B) {
        g[k] = hist[base + 2 * b];
        h[k] = hist[base + 2 * b + 1];
        if (minus) {
          g[k] -= minus[base + 2 * b];
          h[k] -= minus[base + 2 * b + 1];
        }
        if (derived) {
          derived[base + 2 * b] = g[k];
          derived[base + 2 * b + 1] = h[k];
        }
      }
      sg += g[k];
      sh += h[k];
    }
    // inclusive scan of the lane sums over the wave
    int64_t pg = sg, ph = sh;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int64_t tg = __shfl_up(pg, d, 64), th = __shfl_up(ph, d, 64);
      if ((int)lane >= d) {
        pg += tg;
        ph += th;
      }
    }
    const int64_t G = __shfl(pg, 63, 64), H = __shfl(ph, 63, 64);
    const double fg = (double)G * scale, fh = (double)H * scale;
    const double tp = split_term(fg, fh, lam);
    int64_t gl = pg - sg, hl = ph - sh;
    SplitCand c = none;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t b = lane * 4 + k;
      gl += g[k];
      hl += h[k];
      if (b + 1 < B) {
        const double fgl = (double)gl * scale, fhl = (double)hl * scale;
        const double fgr = (double)(G - gl) * scale, fhr = (double)(H - hl) * scale;
        if (fhl >= mcw && fhr >= mcw && fhl + lam > 0.0 && fhr + lam > 0.0) {
          const double gain = 0.5 * ((split_term(fgl, fhl, lam) + split_term(fgr, fhr, lam)) - tp) - gamma;
          if (gain > c.gain) c = {gain, (int32_t)f, (int32_t)b, gl, hl};
        }
      }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
      const SplitCand o = shfl_xor_cand(c, m);
      if (split_better(o, c, false)) c = o;
    }
    if (lane == 0 && out_feat) out_feat[node * F + f] = c;
    if (split_better(c, best, true)) best = c;
  }
  if (lane == 0) waves[w] = best;
  __syncthreads();
  if (threadIdx.x == 0) {
    SplitCand b = waves[0];
    for (uint32_t i = 1; i < kBlockThreads / 64; ++i)
      if (split_better(waves[i], b, true)) b = waves[i];
    out_node[node] = b;
  }
}

// ------------------------------------------------ ciphertext products
// out[i] = a[i] b[i] mod n^2 (canonical in and out): the encrypted sum of two
// ciphertext arrays.  MM(a, b) = a b R^-1, then MM(., R^2) = a b.
template <int KP>
__global__ __launch_bounds__(kBlockThreads) void k_ct_mul(DKey key, const uint32_t *a, const uint32_t *b,
                                                         uint64_t count, uint32_t *out) {
  constexpr int KN2 = 4 * KP, SN2 = 64 * KP;
  __shared__ __align__(16) uint32_t lds_all[16 * SN2];
  const uint32_t gi = wave_in_block() * 4 + group_in_wave();
  uint32_t *lds = lds_all + gi * SN2;
  uint64_t i = (uint64_t)blockIdx.x * 16 + gi;
  const bool valid = i < count;
  if (!valid) i = count - 1;
  const Mod<KN2> M = load_mod<KN2>(key.n2.N, key.n2.ninv);
  uint32_t x[KN2], y[KN2];
  ld<KN2>(x, a + i * SN2);
  ld<KN2>(y, b + i * SN2);
  mont_mul<KN2>(x, x, y, M, lds);
  ld<KN2>(y, key.n2.R2);
  mont_mul<KN2>(x, x, y, M, lds);
  if (valid) st<KN2>(out + i * SN2, x);
}

// ------------------------------------------------------ packing
// Folds `slots` consecutive ciphertexts into one (public key only):
// prod_j c_j^(2^(64 j)) (1 + K n) mod n^2 with K = sum_j 2^(64 j + 63), an
// encryption of sum_j 2^(64 j) (m_j + 2^63), by Horner's rule from the top
// slot down (64 squarings per slot) in two digits base n, 16 lanes per packed
// ciphertext.  The last packed ciphertext may hold fewer slots; the wave's loops
// run over `slots` and its missing slots multiply by one.  The slot count
// leaves one wave per SIMD (pack_slots), so a squaring's latency, 72 steps of
// 27 multiply-adds, bounds it: 32,768 ciphertexts at 8 slots 3.5 -> 2.5 ms
// against squarings of one 144-limb integer.  One slot needs no squaring, and the
// way into and out of the two digits would be most of its time (30,000 ciphertexts
// 0.35 ms): k_enc_obf multiplies by 1 + K n mod n instead (0.16 ms).
template <int KP>
__global__ __launch_bounds__(kBlockThreads, 2) void k_pack(DKey key, const uint32_t *__restrict__ ct, uint64_t count,
                                                          uint32_t slots, uint32_t *__restrict__ packed) {
  constexpr int KN2 = 4 * KP, SN2 = 64 * KP, L = 32 * KP;
  using E = GroupPair<L, 8>;
  constexpr int S = E::S, K = E::K;
  static_assert(E::kLds >= SN2, "the row also holds 32-bit limbs mod n^2");
  __shared__ __align__(16) uint32_t lds_all[16 * E::kLds + S];
  uint32_t *const zeros = lds_all + 16 * E::kLds;
  zero_lds(zeros, S);
  const uint32_t gi = wave_in_block() * 4 + group_in_wave();
  uint32_t *lds = lds_all + gi * E::kLds;
  const uint64_t n_packed = (count + slots - 1) / slots;
  uint64_t p = (uint64_t)blockIdx.x * 16 + gi;
  const bool valid = p < n_packed;
  if (!valid) p = n_packed - 1;
  const uint64_t first = p * slots;
  const uint32_t my_slots = (uint32_t)min((uint64_t)slots, count - first);
  E eng(UnitArgs{key.pair_n.c[he29::pair_variant(8)], key.pair_n.ninv, nullptr}, lds, zeros);
  // the pair of x R in y and z, ready as a product's operand: x = x0 + x1
  // 2^(32 L), each half by its piece's constant
  auto operand = [&](const uint32_t *x) __attribute__((always_inline)) {
    uint32_t t[K];
    uint64_t C[K];
    eng.load_piece(x);
    eng.fetch(0, true);
    eng.mul();
#pragma unroll
    for (int j = 0; j < K; ++j) t[j] = eng.r[j];
    eng.load_piece(x + L);
    eng.fetch(1, true);
    eng.mul();
#pragma unroll
    for (int j = 0; j < K; ++j) C[j] = (uint64_t)eng.r[j] + t[j];
    settle29<K, 8>(eng.r, C);
    st29<K, 16>(lds, eng.r);
    __builtin_amdgcn_wave_barrier();
    ld29<K, 16>(eng.y, lds);
    ld29<K, 8>(eng.z, lds);
    __builtin_amdgcn_wave_barrier();
  };
  uint32_t acc[K];
#pragma unroll 1
  for (uint32_t j = slots; j-- > 0;) {
    // a slot this packed ciphertext does not have: its first row is read (in
    // bounds) and the Montgomery one taken
    const bool have = j < my_slots;
    operand(ct + (first + (have ? j : 0u)) * SN2);
    if (!have) eng.fetch(he29::kPairR, true);
    if (j + 1 == slots) {
#pragma unroll
      for (int i = 0; i < K; ++i) acc[i] = eng.y[i];
    } else {
      uint32_t y[K], z[K];
#pragma unroll
      for (int i = 0; i < K; ++i) {
        y[i] = eng.y[i];
        z[i] = eng.z[i];
        eng.r[i] = acc[i];
      }
#pragma unroll 1
      for (int t = 0; t < 64; ++t) eng.sq();
#pragma unroll
      for (int i = 0; i < K; ++i) {
        eng.y[i] = y[i];
        eng.z[i] = z[i];
      }
      eng.mul();
#pragma unroll
      for (int i = 0; i < K; ++i) acc[i] = eng.r[i];
    }
  }
  // times f = 1 + K n: K has bit 31 of every odd limb below 2 my_slots
  {
    uint32_t f[KN2], c[KN2];
    const Mod<KN2> M32 = load_mod<KN2>(key.n2.N, key.n2.ninv);
#pragma unroll
    for (int i = 0; i < KN2; ++i) {
      const uint32_t idx = glane() * KN2 + i;
      f[i] = ((idx & 1u) && (idx >> 1) < my_slots) ? 0x80000000u : 0u;
    }
    ld<KN2>(c, key.nR_n2);
    mont_mul<KN2>(f, f, c, M32, lds);  // K n mod n^2
    add_one<KN2>(f);
    uint32_t *row = packed + p * SN2;  // f waits in the output row
    if (valid) st<KN2>(row, f);
    __threadfence_block();
    operand(row);
  }
#pragma unroll
  for (int i = 0; i < K; ++i) eng.r[i] = acc[i];
  eng.mul();
  eng.finish(packed + p * SN2, valid);
}

// Slot values of decrypted packed plaintexts raw[n_packed][L]: value i is
// the 64-bit field (i mod slots) of plaintext i / slots, minus 2^63.  A
// plaintext with bits above its last slot (a slot sum outside the signed
// 64-bit range at the top, or a negative total) is counted into *n_overflow.
__global__ void k_unpack(const uint32_t *__restrict__ raw, uint64_t count, uint32_t slots, uint32_t L,
                         int64_t *__restrict__ m, uint32_t *__restrict__ n_overflow) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const uint64_t p = i / slots;
  const uint32_t j = (uint32_t)(i - p * slots);
  const uint32_t my_slots = (uint32_t)min((uint64_t)slots, count - p * slots);
  const uint32_t *w = raw + p * L;
  const uint64_t v = (uint64_t)w[2 * j] | ((uint64_t)w[2 * j + 1] << 32);
  m[i] = (int64_t)(v ^ 0x8000000000000000ull);
  if (j == my_slots - 1 && n_overflow) {
    bool high = false;
    for (uint32_t k = 2 * my_slots; k < L; ++k) high = high || w[k] != 0u;
    if (high) atomicAdd(n_overflow, 1u);
  }
}

// ------------------------------------------------------ Montgomery conversion
// x -> x R' mod n^2 (to_mont) or x R'^-1 mod n^2, R' the radix-2^29 factor of
// the histogram kernels' G-lane groups; canonical 32-bit limbs in and out.
template <int KP, int G>
__global__ __launch_bounds__(kBlockThreads) void k_mont_convert(DKey key, const uint32_t *in, uint64_t count,
                                                               uint32_t *out, int to_mont) {
  constexpr int SN2 = 64 * KP, K32 = SN2 / G, GB = kBlockThreads / G;
  constexpr int S29 = he29::limbs_for_group(SN2, G), K = S29 / G, ROW = S29 > SN2 ? S29 : SN2;
  __shared__ __align__(16) uint32_t lds_all[GB * ROW];
  uint32_t *lds = lds_all + (threadIdx.x / G) * ROW;
  uint64_t i = (uint64_t)blockIdx.x * GB + threadIdx.x / G;
  const bool valid = i < count;
  if (!valid) i = count - 1;
  const Mod29<K> M = load_mod29<K, G>(key.n2);
  uint32_t x[K32], t[K], c[K];
  ld<K32, G>(x, in + i * SN2);
  to29<K32, K, G>(t, x, lds);
  if (to_mont)
    ld29<K, G>(c, key.n2.R2_29[he29::variant(G)]);
  else
    set_small<K, G>(c, 1u);
  mm29<K, G>(t, t, c, M, lds);
  canon29<K, G>(t, M);
  to32<K, K32, G>(x, t, lds);
  if (valid) st<K32, G>(out + i * SN2, x);
}

// -------------------------------------------------------------- decryption
// For (ciphertext i, prime P): x = c^(P-1) mod P^2 = a + e P (k_pow_pair, from
// the ciphertext's four pieces of S_P limbs), then m_P = ((x - 1) / P) h_P mod
// P, and Garner's combination of m_p, m_q.

// m_P = ((x_P - 1) / P) h_P mod P from x_P = a + e P (the exact division as (x -
// 1) P^-1 = e + (a - 1) P^-1 mod 2^(32 S_P), a low-half product; e itself for a
// unit), then m = m_q + q ((m_p - m_q) q^-1 mod p) and the signed decode.
template <int KP>
__global__ __launch_bounds__(kBlockThreads) void k_dec_b(DKey key, const uint32_t *__restrict__ xpq,
                                                        uint64_t count, int64_t *__restrict__ mout,
                                                        uint32_t *__restrict__ raw,
                                                        uint32_t *__restrict__ n_overflow) {
  constexpr int KN = 2 * KP, SP2 = 32 * KP, SN = 32 * KP;
  __shared__ __align__(16) uint32_t lds_all[16 * SN];
  const uint32_t gi = wave_in_block() * 4 + group_in_wave();
  uint32_t *lds = lds_all + gi * SN;
  uint64_t i = (uint64_t)blockIdx.x * 16 + gi;
  const bool valid = i < count;
  if (!valid) i = count - 1;
  uint32_t mpq[2][KP];
#pragma unroll 1
  for (int which = 0; which < 2; ++which) {
    const DPrime &P = key.pr[which];
    uint32_t a[KP], one[KP], k[KP], c[KP];
    const uint32_t *x = xpq + (i * 2 + which) * SP2;
    ld<KP>(a, x);
    set_small<KP>(one, 1u);
    sub_plain<KP>(a, a, one);  // mod 2^(32 S_P)
    ld<KP>(c, P.Pinv);
    st<KP>(lds, a);
    __builtin_amdgcn_wave_barrier();
    mul_lo_lds<KP>(k, lds, c);
    __builtin_amdgcn_wave_barrier();
    ld<KP>(c, x + SP2 / 2);
    add_plain<KP>(k, k, c);
    const Mod<KP> Mp = load_mod<KP>(P.P.N, P.P.ninv);
    ld<KP>(c, P.hR_P);
    mont_mul<KP>(mpq[which], k, c, Mp, lds);
  }
  const DPrime &Pp = key.pr[0];
  const Mod<KP> Mp = load_mod<KP>(Pp.P.N, Pp.P.ninv);
  uint32_t mp[KP], mq[KP], c[KP];
  copy(mp, mpq[0]);
  copy(mq, mpq[1]);
  ld<KP>(c, Pp.P.R2);
  mont_mul<KP>(mp, mp, c, Mp, lds);
  uint32_t mqr[KP];
  mont_mul<KP>(mqr, mq, c, Mp, lds);
  sub_mod<KP>(mp, mp, mqr, Mp);
  ld<KP>(c, key.qinv_p);
  mont_mul<KP>(mp, mp, c, Mp, lds);  // u = (m_p - m_q) q^-1 mod p
  const Mod<KN> Mn = load_mod<KN>(key.n.N, key.n.ninv);
  uint32_t u[KN], v[KN], cn[KN];
  relayout<KP, KN>(u, mp, lds);
  relayout<KP, KN>(v, mq, lds);
  ld<KN>(cn, key.qR_n);
  mont_mul<KN>(u, u, cn, Mn, lds);  // q u (exact, < n)
  add_plain<KN>(u, u, v);           // m in [0, n)
  if (raw && valid) st<KN>(raw + i * SN, u);
  // signed decode: m >= (n + 1) / 2 means m - n
  ld<KN>(cn, key.half);
  const bool below_half = bcast_last(sub_plain<KN>(v, u, cn) ? 1u : 0u) != 0u;
  uint32_t mag[KN];
  sub_plain<KN>(mag, Mn.n, u);
  select(mag, below_half, u, mag);
  bool high = false;
#pragma unroll
  for (int j = 0; j < KN; ++j) high = high || ((glane() * KN + j) >= 2 && mag[j] != 0u);
  high = row_any(high);
  const uint64_t lo64 = (uint64_t)bcast_first(mag[0]) | ((uint64_t)bcast_first(mag[1]) << 32);
  int64_t val;
  bool ovf;
  if (below_half) {
    ovf = high || (lo64 >> 63);
    val = ovf ? INT64_MAX : (int64_t)lo64;
  } else {
    ovf = high || lo64 > (1ull << 63);
    val = ovf ? INT64_MIN : (int64_t)((uint64_t)0 - lo64);
  }
  if (valid && glane() == 0) {
    mout[i] = val;
    if (ovf && n_overflow) atomicAdd(n_overflow, 1u);
  }
}

// ------------------------------------------------------------ histograms
__global__ void k_fill(uint32_t *p, uint64_t n, uint32_t v) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

constexpr int kJobsPerSetup = 24;
struct JobPack {
  DJob j[kJobsPerSetup];
};
// n jobs from the kernel's arguments to dst, and `words` words at zero cleared.
__global__ __launch_bounds__(256) void k_job_setup(JobPack pack, uint32_t n, DJob *dst, uint32_t *zero,
                                                   uint64_t words) {
  if (blockIdx.x == 0 && threadIdx.x < n) dst[threadIdx.x] = pack.j[threadIdx.x];
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < words; i += (uint64_t)gridDim.x * 256) zero[i] = 0;
}

// Bin counts of one (job, feature, sample block) into counts[fb].  Samples
// whose row is not resident or whose bin is out of range are skipped and
// counted into the job's n_bad (bucket_sample).
__global__ __launch_bounds__(256) void k_hist_count(HistWs ws) {
  __shared__ uint32_t h[256];
  __shared__ uint32_t nbad;
  const uint64_t blk = blockIdx.x;
  const uint32_t jn = find_job(ws.jobs, ws.n_jobs, &DJob::blk_off, blk);
  const DJob J = ws.jobs[jn];
  uint32_t f;
  uint64_t s0, s1;
  bucket_block(blk - J.blk_off, J.nblk, J.n, kSampleBlock, f, s0, s1);
  h[threadIdx.x] = 0;
  if (threadIdx.x == 0) nbad = 0;
  __syncthreads();
  const uint8_t *bf = J.bins + (uint64_t)f * J.ld;
  for (uint64_t s = s0 + threadIdx.x; s < s1; s += 256) {
    uint32_t row, bin;
    if (bucket_sample(J.idx, bf, ws.rows, J.B, s, row, bin))
      atomicAdd(&h[bin], 1u);
    else
      atomicAdd(&nbad, 1u);
  }
  __syncthreads();
  if (threadIdx.x < J.B && h[threadIdx.x])
    atomicAdd(&ws.counts[J.fb_off + (uint64_t)f * J.B + threadIdx.x], h[threadIdx.x]);
  if (threadIdx.x == 0 && nbad && J.n_bad) atomicAdd(J.n_bad, nbad);
}

// The length class of a bin's items (the longest class first in their order).
__device__ __forceinline__ uint32_t item_class(uint32_t cnt, uint32_t nch) {
  return min((cnt + nch - 1) / nch, (uint32_t)kHistClasses - 1u);
}

// Per (job, feature): exclusive scan of the bin counts (the bins' sample runs
// in bin order), the bins in decreasing order of their counts (border,
// k_hist_final's entry order; ties: lower bin first), each bin's items and
// their length's class count.  The last block to finish turns the class
// counts into each class's first item, longest first, so that the items of the
// whole batch run from long to short: a wave's consecutive items are of equal
// length, and the launch ends on its shortest ones.
__global__ __launch_bounds__(256) void k_hist_scan(HistWs ws) {
  __shared__ uint32_t sc[256], cn[256], last;
  const uint64_t jf = blockIdx.x;
  const uint32_t jn = find_job(ws.jobs, ws.n_jobs, &DJob::f_off, jf);
  const DJob J = ws.jobs[jn];
  const uint32_t f = (uint32_t)(jf - J.f_off);
  const uint64_t e = J.fb_off + (uint64_t)f * J.B + threadIdx.x;
  const uint32_t t = threadIdx.x;
  const uint32_t cnt = t < J.B ? ws.counts[e] : 0u;
  cn[t] = cnt;
  sc[t] = cnt;
  __syncthreads();
  uint32_t rank = 0;
  if (t < J.B)
    for (uint32_t b = 0; b < J.B; ++b) {
      const uint32_t c = cn[b];
      rank += (c > cnt || (c == cnt && b < t)) ? 1u : 0u;
    }
  const uint32_t chunk = ws.stretch ? item_chunk(cnt, rank, ws.chunk) : ws.chunk;
  const uint32_t nch = (cnt + chunk - 1) / chunk;
  for (uint32_t d = 1; d < 256; d <<= 1) {  // inclusive Hillis-Steele scan
    const uint32_t a = t >= d ? sc[t - d] : 0u;
    __syncthreads();
    sc[t] += a;
    __syncthreads();
  }
  if (t < J.B) {
    ws.offs[e] = sc[t] - cnt;
    ws.cursor[e] = sc[t] - cnt;
    ws.fch[e] = nch;
    ws.border[e - t + rank] = t;
    if (nch) atomicAdd(&ws.cls[item_class(cnt, nch)], nch);
  }
  __threadfence();
  __syncthreads();
  if (t == 0) last = atomicAdd(ws.scanned, 1u) + 1u == (uint32_t)ws.total_f ? 1u : 0u;
  __syncthreads();
  if (!last) return;
  __threadfence();
  // thread t: classes kHistClasses - 1 - 4 t and the three below it
  uint32_t v[4], sum = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[i] = atomicAdd(&ws.cls[kHistClasses - 1 - 4 * t - i], 0u);
    sum += v[i];
  }
  sc[t] = sum;
  __syncthreads();
  for (uint32_t d = 1; d < 256; d <<= 1) {
    const uint32_t a = t >= d ? sc[t - d] : 0u;
    __syncthreads();
    sc[t] += a;
    __syncthreads();
  }
  uint32_t first = sc[t] - sum;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    ws.cls[kHistClasses - 1 - 4 * t - i] = first;
    first += v[i];
  }
  if (t == 255) {
    *ws.n_items = sc[255];
    *ws.next = 0;  // k_hist_chunk's work counter
  }
}

// Items of one (job, feature): every bin's sample run split into its nch
// chunks of equal length (to one sample), each at most `chunk` samples, at the
// next free items of its length's class.
__device__ __forceinline__ void hist_items(const HistWs &ws, uint64_t jf) {
  __shared__ uint32_t at[256];
  const DJob J = ws.jobs[find_job(ws.jobs, ws.n_jobs, &DJob::f_off, jf)];
  const uint32_t f = (uint32_t)(jf - J.f_off);
  const uint64_t e0 = J.fb_off + (uint64_t)f * J.B;
  if (threadIdx.x < J.B) {
    const uint32_t cnt = ws.counts[e0 + threadIdx.x], nch = ws.fch[e0 + threadIdx.x];
    const uint32_t first = nch ? atomicAdd(&ws.cls[item_class(cnt, nch)], nch) : 0u;
    ws.fitem[e0 + threadIdx.x] = first;
    at[threadIdx.x] = first;
  }
  __syncthreads();
  for (uint32_t b = threadIdx.x >> 6; b < J.B; b += 4) {  // a wave per bin
    const uint32_t nch = ws.fch[e0 + b], cnt = ws.counts[e0 + b], first = at[b];
    const uint64_t start = J.perm_off + (uint64_t)f * J.n + ws.offs[e0 + b];
    for (uint32_t c = threadIdx.x & 63u; c < nch; c += 64) {
      const uint32_t lo = (uint32_t)((uint64_t)c * cnt / nch), hi = (uint32_t)((uint64_t)(c + 1) * cnt / nch);
      ws.items[first + c] = HistItem{start + lo, hi - lo, 0};
    }
  }
}

// Scatter of the samples' pairs (their row, or their place among the gathered
// ones) into per-(feature, bin) runs of perm, skipping the samples k_hist_count
// skipped (bucket_sample), so each run receives exactly the samples counted for
// its bin.  The first total_f blocks write the work items.
__global__ __launch_bounds__(256) void k_hist_scatter(HistWs ws) {
  if (blockIdx.x < ws.total_f) {
    hist_items(ws, blockIdx.x);
    return;
  }
  __shared__ uint32_t h[256], base[256];
  const uint64_t blk = blockIdx.x - ws.total_f;
  const uint32_t jn = find_job(ws.jobs, ws.n_jobs, &DJob::blk_off, blk);
  const DJob J = ws.jobs[jn];
  uint32_t f;
  uint64_t s0, s1;
  bucket_block(blk - J.blk_off, J.nblk, J.n, kSampleBlock, f, s0, s1);
  h[threadIdx.x] = 0;
  __syncthreads();
  const uint8_t *bf = J.bins + (uint64_t)f * J.ld;
  constexpr int kPer = kSampleBlock / 256;
  uint32_t rows[kPer], bn[kPer], rk[kPer];
  bool ok[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const uint64_t s = s0 + threadIdx.x + (uint64_t)k * 256;
    ok[k] = s < s1 && bucket_sample(J.idx, bf, ws.rows, J.B, s, rows[k], bn[k]);
    if (ws.gather) rows[k] = (uint32_t)(J.s_off + s);
    if (ok[k]) rk[k] = atomicAdd(&h[bn[k]], 1u);
  }
  __syncthreads();
  const uint64_t e0 = J.fb_off + (uint64_t)f * J.B;
  if (threadIdx.x < J.B && h[threadIdx.x]) base[threadIdx.x] = atomicAdd(&ws.cursor[e0 + threadIdx.x], h[threadIdx.x]);
  __syncthreads();
  uint32_t *pf = ws.perm + J.perm_off + (uint64_t)f * J.n;
#pragma unroll
  for (int k = 0; k < kPer; ++k)
    if (ok[k]) pf[bucket_slot(base[bn[k]], rk[k])] = rows[k];
}

// Final product over the chunks of one (job, feature, bin), conversion out of
// Montgomery form, and the store into the job's histogram.  A block takes
// one rank of one (job, feature) among the first kFinalSolo ranks, else four
// consecutive ranks, one per wave; the units go rank-major over all
// (job, feature) pairs, so the heaviest bins start first.
//  * A block's own entry: its 16 groups are (slot g/h) x (8 runs); the
//    entry's nch partials are cut into P runs of equal length (to one), P
//    the largest power of two that is at most 8 and at most nch / 2, each
//    run's product is one group's chain (about nch / P products instead of
//    nch / 2), and the P products are joined in log2(P) levels through LDS.
//  * A wave's entry: its 4 groups are (slot) x (first or second half of the
//    partials), the halves joined at the end.
template <int KP>
__global__ __launch_bounds__(kBlockThreads, 2) void k_hist_final(DPair pc, HistWs ws) {
  using E = GroupPair<32 * KP, 8>;
  constexpr int S = E::S, K = E::K, ROW = 2 * S, S2 = 64 * KP, GW = 4, kWaves = kBlockThreads / 64, kParts = 2 * kWaves;
  __shared__ __align__(16) uint32_t lds_all[kWaves * GW * E::kLds + S];
  uint32_t *const zeros = lds_all + kWaves * GW * E::kLds;
  zero_lds(zeros, S);
  const uint32_t wv = wave_in_block();
  const uint32_t g = (threadIdx.x & 63u) / 16u;
  uint32_t *lds = lds_all + (wv * GW + g) * E::kLds;
  const uint32_t slot = g & 1u, half = g >> 1, part = 2 * wv + half;
  const uint32_t *consts = pc.c[kHistVariant];
  E eng(UnitArgs{consts, pc.ninv, nullptr}, lds, zeros);
  const uint32_t *one = consts + 2 * he29::kPairR * S;  // Montgomery form of 1
  // product over n partials from the p0-th on, `trip` of them for the wave;
  // past this group's n the multiplier is the Montgomery form of 1
  auto chain = [&](uint64_t p0, uint32_t n, uint32_t trip) __attribute__((always_inline)) {
    auto at = [&](uint32_t k) { return k < n ? ws.partials + ((p0 + k) * 2 + slot) * ROW : one; };
    ld29<K, 16>(eng.r, at(0));
#pragma unroll 1
    for (uint32_t k = 1; k < trip; ++k) {
      const uint32_t *p = at(k);
      ld29<K, 16>(eng.y, p);
      ld29<K, 8>(eng.z, p);
      eng.mul();
    }
  };
  // r <- r times the pair in LDS row `other`, where `keep`
  auto join_row = [&](bool keep) __attribute__((always_inline)) {
    uint32_t old[K];
#pragma unroll
    for (int j = 0; j < K; ++j) old[j] = eng.r[j];
    eng.mul();
    select(eng.r, keep, eng.r, old);
  };
  const uint64_t solo = ws.total_f * kFinalSolo;
  const uint64_t units = solo + ws.total_f * ((256 - kFinalSolo) / kWaves);  // ranks past a job's bins are skipped
  for (uint64_t u = blockIdx.x; u < units; u += gridDim.x) {
    const bool whole = u < solo;  // block-uniform
    const uint64_t v = whole ? u : u - solo;
    const uint64_t jf = v % ws.total_f;
    const uint32_t r = whole ? (uint32_t)(v / ws.total_f) : kFinalSolo + kWaves * (uint32_t)(v / ws.total_f) + wv;
    const DJob J = ws.jobs[find_job(ws.jobs, ws.n_jobs, &DJob::f_off, jf)];
    if (whole && r >= J.B) continue;  // block-uniform
    const uint64_t fb_f = (jf - J.f_off) * J.B;  // the feature's first entry within the job
    if (whole) {
      const uint32_t bin = ws.border[J.fb_off + fb_f + r];
      const uint64_t e = J.fb_off + fb_f + bin;
      const uint32_t nch = ws.fch[e], first = ws.fitem[e];
      uint32_t P = 1;
      while (P < (uint32_t)kParts && 4 * P <= nch) P *= 2;
      const bool mine = part < P;
      const uint32_t lo = mine ? (uint32_t)((uint64_t)part * nch / P) : 0u;
      const uint32_t len = mine ? (uint32_t)((uint64_t)(part + 1) * nch / P) - lo : 0u;
      const uint32_t maxlen = (nch + P - 1) / P;
      const bool wave_on = 2 * wv < P;  // wave-uniform: the wave holds a run
      uint64_t done = 0;
      if (wave_on) {
        chain((uint64_t)first + lo, len, maxlen);
        done += maxlen ? maxlen - 1 : 0;
      }
      // level d joins run p with run p + d for p a multiple of 2d; only the
      // even runs (half 0 of a wave) ever join, so a wave joins or not as a
      // whole
      for (uint32_t d = 1; d < P; d <<= 1) {  // block-uniform
        if (wave_on) st29<K, 16>(lds, eng.r);
        __syncthreads();
        const bool wave_join = (2 * wv) % (2 * d) == 0 && 2 * wv + d < P;
        if (wave_join) {
          const uint32_t q = part + d;  // in range for the joining (even) runs
          const uint32_t qr = half == 0 ? (q >> 1) * GW + ((q & 1u) << 1 | slot) : wv * GW + g;
          ld29<K, 16>(eng.y, lds_all + qr * E::kLds);
          ld29<K, 8>(eng.z, lds_all + qr * E::kLds);
        }
        __syncthreads();
        if (wave_join) {
          join_row(half == 0);
          ++done;
        }
      }
      if (wv == 0) {
        eng.finish(J.hist + ((fb_f + bin) * 2 + slot) * S2, half == 0);
        ++done;
      }
      if (ws.mm_count && glane<16>() == 0) {
        if (wave_on) atomicAdd(&ws.mm_count[1], (unsigned long long)done);
        if (wv == 0 && half == 0) {
          atomicAdd(&ws.mm_count[0], (unsigned long long)(nch ? nch - 1 : 0));
          atomicAdd(&ws.mm_count[2], 1ull);
        }
      }
      __syncthreads();  // the rows are reused by the block's next unit
    } else if (r < J.B) {  // wave-uniform
      const uint32_t bin = ws.border[J.fb_off + fb_f + r];
      const uint64_t e = J.fb_off + fb_f + bin;
      const uint32_t nch = ws.fch[e], first = ws.fitem[e];
      const uint32_t n_lo = (nch + 1) >> 1, n_hi = nch >> 1;
      chain((uint64_t)first + (half ? n_lo : 0u), half ? n_hi : n_lo, n_lo);
      if (n_hi) {  // wave-uniform: join the halves
        st29<K, 16>(lds, eng.r);
        __builtin_amdgcn_wave_barrier();
        ld29<K, 16>(eng.y, lds_all + (wv * GW + (g ^ 2u)) * E::kLds);
        ld29<K, 8>(eng.z, lds_all + (wv * GW + (g ^ 2u)) * E::kLds);
        __builtin_amdgcn_wave_barrier();
        join_row(half == 0);
      }
      eng.finish(J.hist + ((fb_f + bin) * 2 + slot) * S2, half == 0);
      if (ws.mm_count && glane<16>() == 0) {
        const uint64_t done = (n_lo ? n_lo - 1 : 0) + (n_hi ? 1 : 0) + 1;
        atomicAdd(&ws.mm_count[1], (unsigned long long)done);
        if (half == 0) {
          atomicAdd(&ws.mm_count[0], (unsigned long long)(nch ? nch - 1 : 0));
          atomicAdd(&ws.mm_count[2], 1ull);
        }
      }
    }
  }
}

// ------------------------------------------------ integer multiply probe
// Independent 32x32->64 multiply-adds, 8 chains per lane, for the measured
// peak of the VALU integer multiplier (the roofline denominator).
__global__ __launch_bounds__(256) void k_probe_mul(uint64_t iters, uint32_t *sink) {
  uint64_t a0 = threadIdx.x, a1 = a0 + 1, a2 = a0 + 2, a3 = a0 + 3, a4 = a0 + 4, a5 = a0 + 5,
           a6 = a0 + 6, a7 = a0 + 7;
  uint32_t x = 0x9E3779B9u ^ blockIdx.x, y = 0x85EBCA6Bu + threadIdx.x;
  for (uint64_t i = 0; i < iters; ++i) {
    a0 = (uint64_t)x * y + a0;
    a1 = (uint64_t)x * (y + 1) + a1;
    a2 = (uint64_t)x * (y + 2) + a2;
    a3 = (uint64_t)x * (y + 3) + a3;
    a4 = (uint64_t)x * (y + 4) + a4;
    a5 = (uint64_t)x * (y + 5) + a5;
    a6 = (uint64_t)x * (y + 6) + a6;
    a7 = (uint64_t)x * (y + 7) + a7;
    x = (uint32_t)a0;
  }
  const uint64_t s = a0 ^ a1 ^ a2 ^ a3 ^ a4 ^ a5 ^ a6 ^ a7;
  if (s == 0x123456789ull) sink[0] = (uint32_t)s;  // keeps the chains alive
}

// ================================================================ launchers
int device_cus() {
  static int cus = 0;
  if (!cus) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
      cus = 1;
  }
  return cus;
}
static inline uint32_t blocks_for(uint64_t n, uint64_t per) { return (uint32_t)((n + per - 1) / per); }

hipError_t launch_encode(const double *x, uint64_t count, uint32_t frac_bits, int64_t *m,
                         uint32_t *n_bad, hipStream_t s) {
  if (!count) return hipSuccess;
  const uint32_t grid = (uint32_t)std::min<uint64_t>(blocks_for(count, 256), 65536);
  hipLaunchKernelGGL(k_encode, dim3(grid), dim3(256), 0, s, x, count, frac_bits, m, n_bad);
  return hipGetLastError();
}

const void *pow_lane16(int SN, int L, PairPow which);
const void *pow_lane32(int SN, int L, PairPow which);
const void *pow_twin32(int SN, int L, PairPow which);
const void *pow_group(int SN, int L, PairPow which);
const void *pow_pair_kernel(int SN, int L, PairPow which) {
  for (auto f : {pow_lane16, pow_lane32, pow_twin32, pow_group})
    if (const void *k = f(SN, L, which)) return k;
  return nullptr;
}

// Base limbs of an exponentiation of `kind`: n (1) or p, q.
static int pow_base(int KP, int kind) { return kind == 1 ? 32 * KP : 16 * KP; }

// The exponentiation kernel of `kind` at G lanes per integer, null if not
// built.  Mod P (4) and the lift (0), the two steps of an encryption whose
// digits are secret, read their tables masked; an encryption that need not hide
// them takes kind 3; decryption is kind 2, or masked 5; the public exponent n
// is never secret.  Mod P: k_pow from 2 lanes on, one residue per lane below.
template <int S32>
static const void *pow_mod_kernel(int G) {
  switch (G) {
    case 2: return (const void *)k_pow<S32, 2>;
    case 4: return (const void *)k_pow<S32, 4>;
    case 8: return (const void *)k_pow<S32, 8>;
    case 16: return (const void *)k_pow<S32, 16>;
    default: return nullptr;
  }
}
static const void *pow_kernel(int KP, int kind, int G) {
  const int SN = pow_base(KP, kind);
  if (kind == 3) return pow_pair_kernel(SN, G, PairPow::kJoint);
  if (kind == 1 || kind == 2) return pow_pair_kernel(SN, G, PairPow::kSliding);
  if (kind != 4) return pow_pair_kernel(SN, G, PairPow::kMasked);
  if (G == 1) return pow_pair_kernel(SN, 0, PairPow::kMasked);
  return KP == 1 ? pow_mod_kernel<16>(G) : pow_mod_kernel<32>(G);
}
bool pow_shape_valid(int KP, int kind, int G) { return pow_kernel(KP, kind, G) != nullptr; }

// One launch of an exponentiation over the unit pairs [first, first + count).
static hipError_t launch_pow(int KP, const DKey &k, int kind, const uint32_t *in, uint32_t *out, uint64_t first,
                             uint64_t count, uint32_t *tabs, uint32_t *next, const PowLaunch &l, hipStream_t s) {
  const uint32_t SN = (uint32_t)pow_base(KP, kind);
  const void *fn = pow_kernel(KP, kind, l.G);
  if (!fn) return hipErrorInvalidValue;
  if (kind == 4 && l.G > 1) {
    PowArgs a{};
    for (int w = 0; w < 2; ++w) {
      a.mod[w] = k.pr[w].P;
      a.exp[w] = k.pr[w].e_enc;
    }
    a.in = in + first * 2 * SN;
    a.out = out + first * 2 * SN;
    a.in_stride = a.in_limbs = a.out_stride = SN;
    a.count = count;
    a.tabs = tabs;
    a.next = next;
    void *args[] = {&a};
    return hipLaunchKernel(fn, dim3(l.grid), dim3(kBlockThreads), args, l.dyn, s);
  }
  PairPowArgs a{};
  const int v = kind == 4 ? 0 : he29::pair_variant(l.G / 2);
  for (int w = 0; w < 2; ++w) {
    const DPair &pc = kind == 1 ? k.pair_n : k.pr[w].pair;
    a.consts[w] = pc.c[v];
    a.ninv[w] = pc.ninv;
    switch (kind) {
      case 0: a.exp[w] = k.pr[w].e_lift; break;
      case 1: a.exp[w] = k.e_n; break;
      case 2:
      case 5: a.exp[w] = k.pr[w].e_dec; break;
      case 3: a.exp[w] = k.pr[w].joint; break;
      default: a.exp[w] = k.pr[w].e_enc;
    }
  }
  const bool dec = kind == 2 || kind == 5;
  a.pieces = dec ? 4 : 1;
  a.in_w = dec ? 0 : SN;
  a.in_i = dec ? 4 * SN : 2 * SN;
  a.out_w = kind == 4 ? SN : 2 * SN;
  a.out_i = 2 * a.out_w;
  a.in = in + first * a.in_i;
  a.out = out + first * a.out_i;
  a.count = count;
  a.tabs = tabs;
  a.next = next;
  void *args[] = {&a};
  return hipLaunchKernel(fn, dim3(l.grid), dim3(kBlockThreads), args, l.dyn, s);
}

// The plan's launches over `count` unit pairs: the first main_count at
// p.main, the rest at p.tail, each with its work counter in p.ctr when given
// (cleared here, in stream order).  Kind 4 works on tq in place, 0 and 3 read tq,
// 2 and 5 the ciphertexts, 1 the rows of r mod n; all but 4 write two digits.
hipError_t launch_pow_kind(int KP, const DKey &k, int kind, const uint32_t *in, uint32_t *out, uint64_t count,
                           uint32_t *tab, const PowPlan &p, hipStream_t s) {
  if (!count) return hipSuccess;
  const uint64_t mc = p.tail.G ? std::min(p.main_count, count) : count;
  if (p.ctr) {
    const hipError_t e = launch_fill(p.ctr, 2, 0u, s);
    if (e != hipSuccess) return e;
  }
  if (mc) {
    const hipError_t e = launch_pow(KP, k, kind, in, out, 0, mc, tab, p.ctr, p.main, s);
    if (e != hipSuccess) return e;
  }
  if (mc < count) return launch_pow(KP, k, kind, in, out, mc, count - mc, tab, p.ctr ? p.ctr + 1 : nullptr, p.tail, s);
  return hipSuccess;
}

hipError_t launch_enc_r(int KP, const DKey &k, uint64_t count, const uint32_t *r, uint64_t seed, uint64_t roff,
                        uint32_t *tq, hipStream_t s) {
  if (!count) return hipSuccess;
  if (KP == 1)
    hipLaunchKernelGGL(k_enc_r<1>, dim3(blocks_for(2 * count, 16)), dim3(kBlockThreads), 0, s, k, count, r, seed,
                       roff, tq);
  else
    hipLaunchKernelGGL(k_enc_r<2>, dim3(blocks_for(2 * count, 16)), dim3(kBlockThreads), 0, s, k, count, r, seed,
                       roff, tq);
  return hipGetLastError();
}

template <int KP>
static hipError_t enc_crt(const DKey &k, const int64_t *m, uint64_t count, const uint32_t *r, uint64_t seed,
                          uint64_t roff, uint32_t *tq, uint32_t *cpq, uint32_t *ct, uint32_t *tab,
                          const PowPlan &p1, const PowPlan &p2, hipStream_t s) {
  hipLaunchKernelGGL(k_enc_r<KP>, dim3(blocks_for(2 * count, 16)), dim3(kBlockThreads), 0, s, k, count, r, seed,
                     roff, tq);
  hipError_t e = k.ct ? launch_pow_kind(KP, k, 4, tq, tq, count, tab, p1, s) : hipSuccess;
  if (e != hipSuccess) return e;
  e = launch_pow_kind(KP, k, pow_lift_kind(k), tq, cpq, count, tab, p2, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_enc_crt_b<KP>, dim3(blocks_for(count, 16)), dim3(kBlockThreads), 0, s, k, m,
                     (const uint32_t *)cpq, count, ct);
  return hipGetLastError();
}
hipError_t launch_enc_crt(int KP, const DKey &k, const int64_t *m, uint64_t count, const uint32_t *r, uint64_t seed,
                          uint64_t roff, uint32_t *tq, uint32_t *cpq, uint32_t *ct, uint32_t *tab,
                          const PowPlan &p1, const PowPlan &p2, hipStream_t s) {
  if (!count) return hipSuccess;
  return KP == 1 ? enc_crt<1>(k, m, count, r, seed, roff, tq, cpq, ct, tab, p1, p2, s)
                 : enc_crt<2>(k, m, count, r, seed, roff, tq, cpq, ct, tab, p1, p2, s);
}

template <int KP>
static hipError_t enc_pub(const DKey &k, const int64_t *m, uint64_t count, const uint32_t *r, uint64_t seed,
                          uint64_t roff, uint32_t *x, uint32_t *ct, uint32_t *tab, const PowPlan &p, hipStream_t s) {
  const uint64_t rows = count + (count & 1);
  uint32_t *digits = x + rows * 32 * KP;
  hipLaunchKernelGGL(k_pub_pre<KP>, dim3(blocks_for(rows, 16)), dim3(kBlockThreads), 0, s, k, count,
                     r, seed, roff, x);
  const hipError_t e = launch_pow_kind(KP, k, 1, x, digits, rows / 2, tab, p, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_pub_post<KP>, dim3(blocks_for(count, 16)), dim3(kBlockThreads), 0, s, k, m, count,
                     (const uint32_t *)digits, ct);
  return hipGetLastError();
}
hipError_t launch_enc_pub(int KP, const DKey &k, const int64_t *m, uint64_t count, const uint32_t *r, uint64_t seed,
                          uint64_t roff, uint32_t *x, uint32_t *ct, uint32_t *tab, const PowPlan &p, hipStream_t s) {
  if (!count) return hipSuccess;
  return KP == 1 ? enc_pub<1>(k, m, count, r, seed, roff, x, ct, tab, p, s)
                 : enc_pub<2>(k, m, count, r, seed, roff, x, ct, tab, p, s);
}

hipError_t launch_enc_obf(int KP, const DKey &k, const int64_t *m, uint64_t count, const uint32_t *rho,
                          uint32_t *ct, hipStream_t s) {
  if (!count) return hipSuccess;
  const dim3 grid(blocks_for(count, 16));
  if (KP == 1)
    hipLaunchKernelGGL(k_enc_obf<1>, grid, dim3(kBlockThreads), 0, s, k, m, count, rho, ct);
  else
    hipLaunchKernelGGL(k_enc_obf<2>, grid, dim3(kBlockThreads), 0, s, k, m, count, rho, ct);
  return hipGetLastError();
}

hipError_t launch_ct_div(int KP, const DKey &k, const uint32_t *num, const uint32_t *den, uint64_t count,
                         uint32_t batch, uint32_t *out, uint32_t *n_bad, hipStream_t s) {
  if (!count) return hipSuccess;
  const uint64_t groups = (count + batch - 1) / batch;
  const dim3 grid(blocks_for(groups, 16));
  if (KP == 1)
    hipLaunchKernelGGL(k_ct_div<1>, grid, dim3(kBlockThreads), 0, s, k, num, den, count, batch, out, n_bad);
  else
    hipLaunchKernelGGL(k_ct_div<2>, grid, dim3(kBlockThreads), 0, s, k, num, den, count, batch, out, n_bad);
  return hipGetLastError();
}

hipError_t launch_split(const int64_t *hist, const int64_t *minus, uint32_t nodes, uint32_t F, uint32_t B,
                        double scale, double lam, double gamma, double mcw, int64_t *derived, void *out_feat,
                        void *out_node, hipStream_t s) {
  if (!nodes) return hipSuccess;
  hipLaunchKernelGGL(k_split, dim3(nodes), dim3(kBlockThreads), 0, s, hist, minus, F, B, scale, lam, gamma, mcw,
                     derived, (SplitCand *)out_feat, (SplitCand *)out_node);
  return hipGetLastError();
}

hipError_t launch_ct_mul(int KP, const DKey &k, const uint32_t *a, const uint32_t *b, uint64_t count,
                         uint32_t *out, hipStream_t s) {
  if (!count) return hipSuccess;
  const dim3 grid(blocks_for(count, 16));
  if (KP == 1)
    hipLaunchKernelGGL(k_ct_mul<1>, grid, dim3(kBlockThreads), 0, s, k, a, b, count, out);
  else
    hipLaunchKernelGGL(k_ct_mul<2>, grid, dim3(kBlockThreads), 0, s, k, a, b, count, out);
  return hipGetLastError();
}

hipError_t launch_pack(int KP, const DKey &k, const uint32_t *ct, uint64_t count, uint32_t slots,
                       uint32_t *packed, hipStream_t s) {
  if (!count) return hipSuccess;
  if (slots == 1) return launch_enc_obf(KP, k, nullptr, count, ct, packed, s);
  const dim3 grid(blocks_for((count + slots - 1) / slots, 16));
  if (KP == 1)
    hipLaunchKernelGGL(k_pack<1>, grid, dim3(kBlockThreads), 0, s, k, ct, count, slots, packed);
  else
    hipLaunchKernelGGL(k_pack<2>, grid, dim3(kBlockThreads), 0, s, k, ct, count, slots, packed);
  return hipGetLastError();
}

hipError_t launch_unpack(const uint32_t *raw, uint64_t count, uint32_t slots, uint32_t L, int64_t *m,
                         uint32_t *n_overflow, hipStream_t s) {
  if (!count) return hipSuccess;
  hipLaunchKernelGGL(k_unpack, dim3(blocks_for(count, 256)), dim3(256), 0, s, raw, count, slots, L, m, n_overflow);
  return hipGetLastError();
}

uint32_t pack_slots(int n_bits, uint64_t count) {
  static int cus = 0;
  if (!cus) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
      cus = 1;
  }
  // enough packed ciphertexts for one 16-lane group per wave slot of a
  // wave per SIMD; beyond that, as many slots as the plaintext holds
  const uint64_t groups = (uint64_t)cus * 4 * 4;
  const uint64_t s = (count + groups - 1) / groups;
  return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(s, (uint64_t)(n_bits - 1) / 64));
}

hipError_t launch_mont_convert(int KP, const DKey &k, const uint32_t *in, uint64_t count,
                               uint32_t *out, bool to_mont, hipStream_t s) {
  if (!count) return hipSuccess;
  const dim3 grid(blocks_for(count, kBlockThreads / kHistGroup));
  if (KP == 1)
    hipLaunchKernelGGL((k_mont_convert<1, kHistGroup>), grid, dim3(kBlockThreads), 0, s, k, in, count, out,
                       (int)to_mont);
  else
    hipLaunchKernelGGL((k_mont_convert<2, kHistGroup>), grid, dim3(kBlockThreads), 0, s, k, in, count, out,
                       (int)to_mont);
  return hipGetLastError();
}

template <int KP>
static hipError_t dec(const DKey &k, const uint32_t *ct, uint64_t count, uint32_t *xpq, int64_t *m,
                      uint32_t *raw, uint32_t *n_overflow, uint32_t *tab, const PowPlan &p, hipStream_t s) {
  const hipError_t e = launch_pow_kind(KP, k, pow_dec_kind(k), ct, xpq, count, tab, p, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_dec_b<KP>, dim3(blocks_for(count, 16)), dim3(kBlockThreads), 0, s, k,
                     (const uint32_t *)xpq, count, m, raw, n_overflow);
  return hipGetLastError();
}
hipError_t launch_dec(int KP, const DKey &k, const uint32_t *ct, uint64_t count, uint32_t *xpq,
                      int64_t *m, uint32_t *raw, uint32_t *n_overflow, uint32_t *tab, const PowPlan &p,
                      hipStream_t s) {
  if (!count) return hipSuccess;
  return KP == 1 ? dec<1>(k, ct, count, xpq, m, raw, n_overflow, tab, p, s)
                 : dec<2>(k, ct, count, xpq, m, raw, n_overflow, tab, p, s);
}

hipError_t launch_fill(uint32_t *p, uint64_t n, uint32_t v, hipStream_t s) {
  if (!n) return hipSuccess;
  const uint32_t grid = (uint32_t)std::min<uint64_t>(blocks_for(n, 256), 4096);
  hipLaunchKernelGGL(k_fill, dim3(grid), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

template <int KP>
static hipError_t hist(const DKey &k, uint64_t pairs, const DJob *host_jobs, const HistWs &ws, const HistLaunch &l,
                       hipStream_t s) {
  constexpr int G = kHistLanes;
  for (uint32_t j0 = 0; j0 < ws.n_jobs; j0 += kJobsPerSetup) {
    JobPack pack;
    const uint32_t n = std::min<uint32_t>(kJobsPerSetup, ws.n_jobs - j0);
    for (uint32_t j = 0; j < n; ++j) pack.j[j] = host_jobs[j0 + j];
    const uint64_t words = j0 ? 0 : ws.total_fb + kHistClasses + 1;  // counts, classes, the scan's block count
    hipLaunchKernelGGL(k_job_setup, dim3(j0 ? 1 : (uint32_t)std::min<uint64_t>(blocks_for(words, 1024), 1024)),
                       dim3(256), 0, s, pack, n, ws.jobs + j0, ws.counts, words);
  }
  if (ws.total_blocks)
    hipLaunchKernelGGL(k_hist_count, dim3((uint32_t)ws.total_blocks), dim3(256), 0, s, ws);
  hipLaunchKernelGGL(k_hist_scan, dim3((uint32_t)ws.total_f), dim3(256), 0, s, ws);
  hipLaunchKernelGGL(k_hist_scatter, dim3((uint32_t)(ws.total_f + ws.total_blocks)), dim3(256), 0, s, ws);
  if (ws.total_blocks) {
    if (ws.pairs) {
      hipLaunchKernelGGL((k_hist_pairs<KP, G>), dim3(blocks_for(pairs, kBlockThreads / (2 * G))), dim3(kBlockThreads),
                         0, s, k.pair_n, ws.ct, (int)ws.mont, ws, pairs);
      hipLaunchKernelGGL((k_hist_chunk<KP, G, false>), dim3(l.grid), dim3(kBlockThreads), l.dyn, s, k.pair_n, ws);
    } else {
      hipLaunchKernelGGL((k_hist_chunk<KP, G, true>), dim3(l.grid), dim3(kBlockThreads), l.dyn, s, k.pair_n, ws);
    }
  }
  const uint64_t final_units = ws.total_f * (kFinalSolo + (256 - kFinalSolo) / 4);
  const uint32_t fgrid = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(final_units, 1u << 20));
  hipLaunchKernelGGL(k_hist_final<KP>, dim3(fgrid), dim3(kBlockThreads), 0, s, k.pair_n, ws);
  return hipGetLastError();
}
hipError_t launch_hist(int KP, const DKey &k, uint64_t pairs, const DJob *host_jobs, const HistWs &ws,
                       const HistLaunch &l, hipStream_t s) {
  return KP == 1 ? hist<1>(k, pairs, host_jobs, ws, l, s) : hist<2>(k, pairs, host_jobs, ws, l, s);
}

hipError_t launch_probe_mul(uint64_t iters, uint32_t grid, uint32_t *sink, hipStream_t s) {
  hipLaunchKernelGGL(k_probe_mul, dim3(grid), dim3(256), 0, s, iters, sink);
  return hipGetLastError();
}


// Elements per inversion batch of k_ct_div: enough groups for about two
// waves per SIMD, each group then chains as many elements as needed.
uint32_t ct_div_batch(uint64_t count) {
  static int cus = 0;
  if (!cus) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
      cus = 1;
  }
  const uint64_t groups = (uint64_t)cus * 4 * 2 * 4;
  return (uint32_t)std::max<uint64_t>(1, (count + groups - 1) / groups);
}


// Resident blocks of the exponentiation of `kind` at G lanes with `dyn` bytes
// of dynamic LDS.
uint32_t pow_resident_blocks(int KP, int kind, int G, uint32_t dyn) {
  static std::mutex mu;
  static std::map<std::tuple<const void *, uint32_t>, uint32_t> cache;
  const void *fn = pow_kernel(KP, kind, G);
  std::lock_guard<std::mutex> lk(mu);
  auto it = cache.find({fn, dyn});
  if (it != cache.end()) return it->second;
  int nb = 0;
  if (!fn || hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, kBlockThreads, dyn) != hipSuccess || nb < 1) nb = 1;
  const uint32_t r = (uint32_t)(nb * device_cus());
  cache[{fn, dyn}] = r;
  return r;
}

// Dynamic LDS that makes at most `waves` blocks of `fn` fit a compute unit
// (0 if its own occupancy `natural` is already at most that).
static uint32_t cap_dyn_lds(const void *fn, int natural, int waves) {
  if (waves <= 0 || natural <= waves) return 0;
  int dev = 0, lds_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&lds_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) != hipSuccess ||
      lds_cu <= 0)
    return 0;
  hipFuncAttributes fa{};
  if (hipFuncGetAttributes(&fa, fn) != hipSuccess) return 0;
  const int64_t per_block = lds_cu / (waves + 1) + 1;
  const int64_t dyn = per_block - (int64_t)fa.sharedSizeBytes;
  return dyn > 0 ? (uint32_t)((dyn + 255) / 256 * 256) : 0u;
}

// Dynamic LDS that caps the exponentiation at `waves` blocks (= waves per SIMD)
// per compute unit: enough that waves + 1 blocks do not fit.  0 when waves
// is 0 or the kernel's own occupancy is at most `waves`.
uint32_t pow_dyn_lds(int KP, int kind, int G, int waves) {
  if (waves <= 0 || !pow_shape_valid(KP, kind, G)) return 0;
  return cap_dyn_lds(pow_kernel(KP, kind, G),
                     (int)(pow_resident_blocks(KP, kind, G, 0) / (uint32_t)device_cus()), waves);
}

template <int KP>
static const void *hist_kernel(bool direct) {
  return direct ? (const void *)k_hist_chunk<KP, kHistLanes, true> : (const void *)k_hist_chunk<KP, kHistLanes, false>;
}
static const void *hist_kernel(int KP, bool direct) { return KP == 1 ? hist_kernel<1>(direct) : hist_kernel<2>(direct); }
uint32_t hist_resident_blocks(int KP, bool direct, uint32_t dyn) {
  static std::mutex mu;
  static std::map<std::tuple<int, bool, uint32_t>, uint32_t> cache;
  std::lock_guard<std::mutex> lk(mu);
  auto it = cache.find({KP, direct, dyn});
  if (it != cache.end()) return it->second;
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, hist_kernel(KP, direct), kBlockThreads, dyn) != hipSuccess ||
      nb < 1)
    nb = 1;
  const uint32_t r = (uint32_t)(nb * device_cus());
  cache[{KP, direct, dyn}] = r;
  return r;
}
uint32_t hist_dyn_lds(int KP, bool direct, int waves) {
  return waves <= 0 ? 0
                    : cap_dyn_lds(hist_kernel(KP, direct),
                                  (int)(hist_resident_blocks(KP, direct, 0) / (uint32_t)device_cus()), waves);
}

uint64_t table_bytes_per_block(int KP, int kind, int G) {
  // radix-2^29 limbs per table entry: two digits, or one residue mod P
  const int SN = pow_base(KP, kind);
  const uint64_t S = kind != 4 ? 2ull * he29::pair_limbs(SN, he29::pair_variant(G / 2))
                               : (G == 1 ? (uint64_t)he29::pair_limbs(SN, 0) : (uint64_t)he29::limbs_for_group(SN, G));
  return (uint64_t)(kBlockThreads / G) * (kTable + 1) * S * sizeof(uint32_t);
}

}  // namespace he
