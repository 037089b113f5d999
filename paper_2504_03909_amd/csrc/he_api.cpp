// Host runtime behind the C ABI in include/he.h: key objects with their
// device-resident constants, per-stream workspaces, argument checks and
// kernel dispatch.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <cmath>
#include <map>
#include <tuple>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/he.h"
#include "he_internal.hpp"
#include "hostbn.hpp"
#include "keysetup.hpp"

using hebn::Limbs;

struct he_key {
  uint32_t n_bits = 0;
  bool priv = false;
  Limbs n, p, q;
  int device = 0;
  void *blob = nullptr;   // device copy of every constant below
  he::DKey dk{};
};

namespace {

thread_local std::string g_last_error;

int fail(int code, const std::string &msg) {
  g_last_error = msg;
  return code;
}

#define HE_TRY_HIP(expr)                                                       \
  do {                                                                         \
    hipError_t e_ = (expr);                                                    \
    if (e_ != hipSuccess)                                                      \
      return fail(HE_ERR_DEVICE, std::string(#expr ": ") + hipGetErrorString(e_)); \
  } while (0)

he::DMod mk_mod(const uint32_t *base, const hekey::ModOff &o) {
  he::DMod m{base + o.N, base + o.R1, base + o.R2, base + o.R3, o.ninv, {}, {}, {}};
  for (int v = 0; v < he29::kVariants; ++v) {
    if (!o.N29[v]) continue;
    m.N29[v] = base + o.N29[v];
    m.R1_29[v] = base + o.R1_29[v];
    m.R2_29[v] = base + o.R2_29[v];
  }
  return m;
}
he::DExp mk_exp(const uint32_t *base, const hekey::ExpOff &o) {
  return he::DExp{base + o.e, o.nwin, base + o.ops, o.nops};
}

he::DPair mk_pair(const uint32_t *base, const hekey::PairOff &o) {
  he::DPair d{};
  for (int v = 0; v < he29::kPairVariants; ++v) d.c[v] = base + o.c[v];
  d.ninv = o.ninv;
  return d;
}

// Builds every constant of the key and uploads them to the current device.
int build_key(he_key *k) {
  const hekey::KeyConsts kc = hekey::derive(k->n_bits, k->n, k->p, k->q, k->priv);
  const hekey::Blob &b = kc.blob;
  const hekey::ModOff &on = kc.n, &on2 = kc.n2;
  const hekey::ExpOff &oe = kc.e_n;
  const hekey::PrimeOff &op = kc.pr[0], &oq = kc.pr[1];
  const size_t o_nR = kc.nR_n2, o_half = kc.half, o_Cq = kc.Cq, o_q2R = kc.q2R_n2, o_qinv = kc.qinv_p,
               o_qR = kc.qR_n;
  HE_TRY_HIP(hipGetDevice(&k->device));
  HE_TRY_HIP(hipMalloc(&k->blob, b.words.size() * sizeof(uint32_t)));
  HE_TRY_HIP(hipMemcpy(k->blob, b.words.data(), b.words.size() * sizeof(uint32_t), hipMemcpyHostToDevice));
  const uint32_t *base = (const uint32_t *)k->blob;
  he::DKey &d = k->dk;
  d.n_bits = k->n_bits;
  d.has_priv = k->priv;
  d.n = mk_mod(base, on);
  d.n2 = mk_mod(base, on2);
  d.pair_n = mk_pair(base, kc.pair_n);
  d.e_n = mk_exp(base, oe);
  d.nR_n2 = base + o_nR;
  d.half = base + o_half;
  if (k->priv) {
    const hekey::PrimeOff *po[2] = {&op, &oq};
    for (int w = 0; w < 2; ++w) {
      he::DPrime &P = d.pr[w];
      P.P = mk_mod(base, po[w]->P);
      P.P2 = mk_mod(base, po[w]->P2);
      P.pair = mk_pair(base, po[w]->pair);
      P.e_enc = mk_exp(base, po[w]->e_enc);
      P.e_lift = mk_exp(base, po[w]->e_lift);
      P.e_dec = mk_exp(base, po[w]->e_dec);
      P.joint = mk_exp(base, po[w]->joint);
      P.QR2_P = base + po[w]->QR2_P;
      P.PR_P2 = base + po[w]->PR_P2;
      P.Pinv = base + po[w]->Pinv;
      P.hR_P = base + po[w]->hR_P;
    }
    d.Cq = base + o_Cq;
    d.q2R_n2 = base + o_q2R;
    d.qinv_p = base + o_qinv;
    d.qR_n = base + o_qR;
  }
  return HE_OK;
}

int make_key(uint32_t n_bits, const Limbs &p, const Limbs &q, bool priv, he_key **out) {
  he_key *k = new (std::nothrow) he_key();
  if (!k) return fail(HE_ERR_OOM, "out of host memory");
  k->n_bits = n_bits;
  k->priv = priv;
  if (priv) {
    k->p = p;
    k->q = q;
    k->n = hebn::mul(p, q);
  } else {
    k->n = p;
  }
  int rc;
  try {
    rc = build_key(k);
  } catch (const std::exception &e) {
    rc = fail(HE_ERR_KEY, std::string("key setup: ") + e.what());
  }
  if (rc != HE_OK) {
    if (k->blob) hipFree(k->blob);
    delete k;
    return rc;
  }
  *out = k;
  return HE_OK;
}

bool valid_bits(uint32_t n_bits) { return n_bits == 1024 || n_bits == 2048; }
int kp_of(const he_key *k) { return k->n_bits == 2048 ? 2 : 1; }

// ---------------------------------------------------------------- workspace
// Grow-only device buffers, one set per stream.  Growing synchronises the
// stream first so that no queued kernel still uses the old buffer.
struct Buf {
  void *p = nullptr;
  size_t bytes = 0;
};
struct Workspace {
  Buf tab, tmp, hist, unpack, ctr;  // ctr: the exponentiation launches' work counters
};
std::mutex g_ws_mu;
std::map<std::pair<int, hipStream_t>, Workspace *> g_ws;

Workspace *workspace(hipStream_t s) {
  int dev = 0;
  hipGetDevice(&dev);
  std::lock_guard<std::mutex> lk(g_ws_mu);
  auto &w = g_ws[{dev, s}];
  if (!w) w = new Workspace();
  return w;
}

int ensure(Buf &b, size_t bytes, hipStream_t s) {
  if (b.bytes >= bytes) return HE_OK;
  if (b.p) {
    HE_TRY_HIP(hipStreamSynchronize(s));
    HE_TRY_HIP(hipFree(b.p));
    b.p = nullptr;
    b.bytes = 0;
  }
  size_t want = std::max(bytes, b.bytes * 3 / 2);
  if (hipMalloc(&b.p, want) != hipSuccess) {
    hipGetLastError();
    b.p = nullptr;
    if (hipMalloc(&b.p, bytes) != hipSuccess) {
      hipGetLastError();
      b.p = nullptr;
      return fail(HE_ERR_OOM, "workspace allocation of " + std::to_string(bytes) + " bytes failed");
    }
    want = bytes;
  }
  b.bytes = want;
  return HE_OK;
}

// ------------------------------------------------- exponentiation launch shapes
// Tuned shapes (lanes per integer, waves per SIMD) of the exponentiations per
// (device, key size, kind, count class), filled by he_crt_autotune and
// he_crt_set_shape; count class = bit length of the count.  A kind is one set of
// kernels (he_internal.hpp), so a shape timed on one is never used for another.
struct PowShape {
  int G = 0, waves = 0;  // G 0: the default plan; waves 0: the kernel's own occupancy
  int tailG = 0;         // lanes per integer of the last partial round's launch (0: no separate launch)
};
std::mutex g_pow_mu;
std::map<std::tuple<int, int, int, int>, PowShape> g_pow_tuned;

// The widths that he_crt_set_shape takes and the autotuner tries and returns:
// every built one but two lanes where the power's modulus has 64 32-bit limbs
// (the lift and decryption at 2048 bits, public-key encryption at 1024).  A pin
// holds for a whole class of counts, and there two lanes are the best only where
// the count just fills a wave per SIMD with them (at 16,384 of 2048 bits 7.95
// against two rounds at four lanes of 8.3 ms); the default plan takes them there.
bool pow_shape_named(int KP, int kind, int G) {
  const int S32 = kind == 4 ? 16 * KP : (kind == 1 ? 64 * KP : 32 * KP);
  return he::pow_shape_valid(KP, kind, G) && !(S32 == 64 && G == 2);
}

int count_class(uint64_t count) {
  int b = 0;
  while (count) {
    ++b;
    count >>= 1;
  }
  return b;
}

he::PowLaunch pow_launch_at(int KP, int kind, uint64_t count, PowShape sh) {
  const uint32_t dyn = he::pow_dyn_lds(KP, kind, sh.G, sh.waves);
  const uint64_t per_wave = 64 / sh.G;
  const uint64_t work_blocks = (2 * ((count + per_wave - 1) / per_wave) + 3) / 4;
  const uint32_t grid =
      (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(he::pow_resident_blocks(KP, kind, sh.G, dyn), work_blocks));
  return he::PowLaunch{sh.G, grid, dyn};
}

// The launches of shape `sh` over `count` ciphertexts.  With sh.tailG, the
// ciphertexts that fill whole rounds of the main launch's resident waves
// (as many units of 64 / G integers of one prime as a whole number of
// units per wave) go to the main launch and the rest, less than one round,
// to a launch at sh.tailG lanes per integer, whose fewer integers per wave
// spread that remainder over more waves.  No split when there is no whole
// round or no remainder.
he::PowPlan pow_plan_at(int KP, int kind, uint64_t count, PowShape sh) {
  he::PowPlan p{pow_launch_at(KP, kind, count, sh), count, he::PowLaunch{0, 0, 0}};
  if (sh.tailG == 0 || sh.tailG == p.main.G || !he::pow_shape_valid(KP, kind, sh.tailG)) return p;
  const uint64_t per_wave = 64 / p.main.G;
  const uint64_t units = 2 * ((count + per_wave - 1) / per_wave);
  const uint64_t waves = 4ull * p.main.grid;
  const uint64_t rounds = units / waves;
  if (rounds == 0 || units % waves == 0) return p;
  p.main_count = rounds * waves / 2 * per_wave;  // < count: at least one unit pair is left
  p.tail = pow_launch_at(KP, kind, count - p.main_count, PowShape{sh.tailG, 0, 0});
  return p;
}

// Window-table bytes a plan's launches need (they run one after the other).
uint64_t plan_table_bytes(int KP, int kind, const he::PowPlan &p) {
  uint64_t b = (uint64_t)p.main.grid * he::table_bytes_per_block(KP, kind, p.main.G);
  if (p.tail.G) b = std::max<uint64_t>(b, (uint64_t)p.tail.grid * he::table_bytes_per_block(KP, kind, p.tail.G));
  return b;
}

// Launch plan of an exponentiation no shape was tuned or pinned for.  A wave
// on a SIMD of its own issues nearly as fast as two, so a launch's time is
// first + (n - 1) more, n the waves the fullest SIMD gets: `first` is one wave
// alone (for wide groups the latency of their steps), `more` what each further
// wave adds once latencies are covered.  Narrow groups need fewer instructions
// per integer (more / 64 G falls with G), wide ones fill the device with fewer
// integers and leave a smaller last wave.  Tried: every width for the whole
// count, and every width for as many whole waves per SIMD as the count holds
// with the rest in a second launch at a wider one.
// The constants are milliseconds measured at one and at several waves per
// SIMD (MI355X, about 2.15 GHz under this load); only their ratios matter.
// E.g. 200,000 encryptions' powers at 2048 bits: 196,608 at one lane and the rest
// at 8 take 98 ms; in one launch 109 ms at one lane (an uneven last wave), 119
// at 2 and 132 at 8.
struct PowCost {
  int G;
  double first, more;
};
const std::vector<PowCost> &pow_costs(int KP, int kind) {
  // Masked tables: every window reads 32 entries, which narrow groups, with more
  // integers per wave, wait for longest (`first` between a few waves and one on
  // every SIMD, e.g. 1.05 and 1.7 at four lanes mod a 512-bit prime).
  static const std::vector<PowCost> mod16 = {{1, 2.5, 2.55}, {2, 2.0, 1.65}, {4, 1.15, .6}, {8, 1.2, .45}, {16, 1.53, .42}};
  static const std::vector<PowCost> mod32 = {{1, 11, 10.4}, {2, 6.5, 7.7}, {4, 3.5, 2.7}, {8, 3.3, 1.8}, {16, 3.4, 1.5}};
  static const std::vector<PowCost> mask16 = {{1, 5.2, 5.25}, {2, 2.7, 2.55}, {4, 1.9, 1.05}, {8, 1.6, .7}, {16, 1.34, .55}};
  static const std::vector<PowCost> mask32 = {{1, 32, 22.5}, {2, 14, 12.7}, {4, 8.4, 6.3}, {8, 5, 3.35}, {16, 4.2, 2.3}};
  static const std::vector<PowCost> pair16 = {{1, 1.93, 1.72}, {2, 1.2, .98}, {4, .88, .55}, {8, .72, .41}, {16, .78, .38}};
  static const std::vector<PowCost> pair32 = {{1, 13.1, 12.1}, {2, 7.95, 7.1}, {4, 4.7, 3.6}, {8, 2.9, 2.1}, {16, 2.58, 1.53}};
  static const std::vector<PowCost> joint16 = {{1, 2.5, 2.2}, {2, 1.65, 1.35}, {4, 1.12, .74}, {8, .93, .54}, {16, .98, .46}};
  static const std::vector<PowCost> joint32 = {{1, 17.0, 15.4}, {2, 10.2, 9.2}, {4, 6.0, 4.75}, {8, 3.65, 2.75}, {16, 3.2, 1.95}};
  static const std::vector<PowCost> pair64 = {{8, 17.1, 13.7}, {16, 11.1, 8.0}};
  if (kind == 4) return KP == 1 ? mod16 : mod32;
  if (kind == 0 || kind == 5) return KP == 1 ? mask16 : mask32;
  if (kind == 1) return KP == 1 ? pair32 : pair64;
  if (kind == 3) return KP == 1 ? joint16 : joint32;
  return KP == 1 ? pair16 : pair32;
}

he::PowPlan default_pow_plan(int KP, int kind, uint64_t count) {
  const uint64_t simds = 4ull * (uint64_t)he::device_cus();
  auto waves = [](int G, uint64_t n) { return 2 * ((n + 64 / G - 1) / (64 / G)); };
  auto cost = [&](const PowCost &c, uint64_t n) {
    return c.first + (double)((waves(c.G, n) + simds - 1) / simds - 1) * c.more;
  };
  double best = 1e300;
  int G = 16, tailG = 0;
  uint64_t main_count = count;
  for (const PowCost &c : pow_costs(KP, kind)) {
    if (cost(c, count) < best) {
      best = cost(c, count);
      G = c.G;
      tailG = 0;
      main_count = count;
    }
    const uint64_t whole = waves(c.G, count) / simds * simds / 2 * (64 / c.G);
    if (whole == 0 || whole >= count) continue;
    for (const PowCost &t : pow_costs(KP, kind)) {
      if (t.G <= c.G || cost(c, whole) + cost(t, count - whole) >= best) continue;
      best = cost(c, whole) + cost(t, count - whole);
      G = c.G;
      tailG = t.G;
      main_count = whole;
    }
  }
  he::PowPlan p{pow_launch_at(KP, kind, main_count, PowShape{G, 0, 0}), main_count, he::PowLaunch{0, 0, 0}, nullptr};
  if (tailG) p.tail = pow_launch_at(KP, kind, count - main_count, PowShape{tailG, 0, 0});
  return p;
}

// The tuned or pinned shape of an exponentiation over `count` ciphertexts
// (units), G 0 (the default plan) if there is none.
PowShape pow_shape_set(int KP, int kind, uint64_t count) {
  int dev = 0;
  (void)hipGetDevice(&dev);
  std::lock_guard<std::mutex> lk(g_pow_mu);
  auto it = g_pow_tuned.find({dev, KP, kind, count_class(count)});
  return it != g_pow_tuned.end() ? it->second : PowShape{};
}

// The shape whose pin gives the plan that `count` has now: G 0 for a default plan
// of two launches, or of a width no pin names.
PowShape pow_pin(int KP, int kind, uint64_t count) {
  const PowShape sh = pow_shape_set(KP, kind, count);
  if (sh.G) return sh;
  const he::PowPlan p = default_pow_plan(KP, kind, count);
  return p.tail.G || !pow_shape_named(KP, kind, p.main.G) ? PowShape{} : PowShape{p.main.G, 0, 0};
}

// The launches of an exponentiation over `count` ciphertexts (units): those of
// the shape set for its class, else default_pow_plan's.
he::PowPlan pow_plan(int KP, int kind, uint64_t count) {
  const PowShape sh = pow_shape_set(KP, kind, count);
  return sh.G ? pow_plan_at(KP, kind, count, sh) : default_pow_plan(KP, kind, count);
}

// Workspace for the window tables of a call's exponentiations (one after the
// other), 0.6 to 1.25 GB where one lane per integer fills the device.  Without
// room for them the largest launches are halved until they fit: waves claim their
// units, so any number of blocks does the same work.
struct KindPlan {
  int kind;
  he::PowPlan *plan;  // main.G 0: a step the call does not have
};
int ensure_tables(Buf &b, int KP, std::initializer_list<KindPlan> plans, hipStream_t s) {
  for (;;) {
    uint64_t bytes = 0;
    for (const KindPlan &k : plans)
      if (k.plan->main.G) bytes = std::max(bytes, plan_table_bytes(KP, k.kind, *k.plan));
    const int rc = ensure(b, bytes, s);
    if (rc != HE_ERR_OOM) return rc;
    bool halved = false;
    for (const KindPlan &k : plans)
      for (he::PowLaunch *l : {&k.plan->main, &k.plan->tail}) {
        if (!l->G || l->grid < 2 || l->grid * he::table_bytes_per_block(KP, k.kind, l->G) <= bytes / 2) continue;
        l->grid = (l->grid + 1) / 2;
        halved = true;
      }
    if (!halved) return rc;
  }
}

// m == nullptr encrypts zeros (the obfuscators r^n mod n^2).
int encrypt_impl(const he_key *key, const int64_t *m, uint64_t count, const uint32_t *r,
                 uint64_t r_seed, uint64_t r_offset, uint32_t *ct, hipStream_t stream, bool force_pub) {
  if (!key) return fail(HE_ERR_ARG, "null key");
  if (count == 0) return HE_OK;
  if (!ct) return fail(HE_ERR_ARG, "null ct");
  Workspace *w = workspace(stream);
  const int KP = kp_of(key);
  const size_t L = key->n_bits / 32;
  if (key->priv && !force_pub) {
    // secret digits: r^(Q mod (P-1)) mod P, then its power P; else both at once
    const he::DKey dk = key->dk;
    const int kind = he::pow_lift_kind(dk);
    he::PowPlan p1{}, p2 = pow_plan(KP, kind, count);
    if (dk.ct) p1 = pow_plan(KP, 4, count);
    int rc = ensure(w->ctr, 256, stream);
    if (rc) return rc;
    p1.ctr = (uint32_t *)w->ctr.p;
    p2.ctr = p1.ctr + 2;
    // omega / c_P per (ciphertext, prime) (2L limbs per ciphertext), then
    // r mod P / t per (ciphertext, prime) (L limbs)
    rc = ensure(w->tmp, count * 3 * L * sizeof(uint32_t), stream);
    if (rc) return rc;
    rc = ensure_tables(w->tab, KP, {{4, &p1}, {kind, &p2}}, stream);
    if (rc) return rc;
    uint32_t *cpq = (uint32_t *)w->tmp.p, *tq = cpq + count * 2 * L;
    HE_TRY_HIP(he::launch_enc_crt(KP, dk, m, count, r, r_seed, r_offset, tq, cpq, ct, (uint32_t *)w->tab.p,
                                  p1, p2, stream));
  } else {
    // the exponentiation's units pair consecutive ciphertexts (both "primes"
    // of a public-key unit pair are n^2)
    he::PowPlan p = pow_plan(KP, 1, (count + 1) / 2);
    int rc = ensure(w->ctr, 256, stream);
    if (rc) return rc;
    p.ctr = (uint32_t *)w->ctr.p;
    // r mod n, then r^n mod n^2: count + (count & 1) rows of L and of 2L limbs
    rc = ensure(w->tmp, (count + 1) * 3 * L * sizeof(uint32_t), stream);
    if (rc) return rc;
    rc = ensure_tables(w->tab, KP, {{1, &p}}, stream);
    if (rc) return rc;
    HE_TRY_HIP(he::launch_enc_pub(KP, key->dk, m, count, r, r_seed, r_offset, (uint32_t *)w->tmp.p, ct,
                                  (uint32_t *)w->tab.p, p, stream));
  }
  return HE_OK;
}

}  // namespace

// ===================================================================== ABI
extern "C" {

const char *he_last_error(void) { return g_last_error.c_str(); }

int he_keygen(uint32_t n_bits, uint64_t seed, he_key **out) {
  if (!out) return fail(HE_ERR_ARG, "null out");
  if (!valid_bits(n_bits)) return fail(HE_ERR_ARG, "n_bits must be 1024 or 2048");
  try {
    const uint32_t half = n_bits / 2;
    Limbs p, q;
    for (uint64_t a = 0;; ++a) {
      p = hebn::prime_candidate(seed, 0, a, half);
      if (hebn::is_probable_prime(p)) break;
    }
    const Limbs one = hebn::from_u64(1);
    for (uint64_t a = 0;; ++a) {
      q = hebn::prime_candidate(seed, 1, a, half);
      if (hebn::cmp(q, p) == 0 || !hebn::is_probable_prime(q)) continue;
      Limbs g = hebn::gcd(hebn::mul(p, q), hebn::mul(hebn::sub(p, one), hebn::sub(q, one)));
      if (hebn::cmp(g, one) == 0) break;
    }
    return make_key(n_bits, p, q, true, out);
  } catch (const std::exception &e) {
    return fail(HE_ERR_KEY, std::string("keygen: ") + e.what());
  }
}

int he_key_import(uint32_t n_bits, const uint32_t *p, const uint32_t *q, he_key **out) {
  if (!out || !p) return fail(HE_ERR_ARG, "null argument");
  if (!valid_bits(n_bits)) return fail(HE_ERR_ARG, "n_bits must be 1024 or 2048");
  const size_t L = n_bits / 32;
  try {
    const Limbs one = hebn::from_u64(1);
    if (!q) {
      Limbs n = hebn::from_words(p, L);
      if (!hebn::is_odd(n) || hebn::bit_length(n) != n_bits)
        return fail(HE_ERR_KEY, "n must be odd with exactly n_bits bits");
      return make_key(n_bits, n, Limbs(), false, out);
    }
    Limbs P = hebn::from_words(p, L / 2), Q = hebn::from_words(q, L / 2);
    if (!hebn::is_odd(P) || !hebn::is_odd(Q) || hebn::cmp(P, one) <= 0 || hebn::cmp(Q, one) <= 0)
      return fail(HE_ERR_KEY, "p and q must be odd and > 1");
    if (hebn::cmp(P, Q) == 0) return fail(HE_ERR_KEY, "p == q");
    Limbs n = hebn::mul(P, Q);
    if (hebn::bit_length(n) != n_bits) return fail(HE_ERR_KEY, "p q must have exactly n_bits bits");
    Limbs g = hebn::gcd(n, hebn::mul(hebn::sub(P, one), hebn::sub(Q, one)));
    if (hebn::cmp(g, one) != 0) return fail(HE_ERR_KEY, "gcd(pq, (p-1)(q-1)) != 1");
    return make_key(n_bits, P, Q, true, out);
  } catch (const std::exception &e) {
    return fail(HE_ERR_KEY, std::string("import: ") + e.what());
  }
}

int he_key_export(const he_key *key, uint32_t *n, uint32_t *p, uint32_t *q) {
  if (!key) return fail(HE_ERR_ARG, "null key");
  const size_t L = key->n_bits / 32;
  if ((p || q) && !key->priv) return fail(HE_ERR_NOPRIV, "public key has no p, q");
  if (n) hebn::to_words(key->n, n, L);
  if (p) hebn::to_words(key->p, p, L / 2);
  if (q) hebn::to_words(key->q, q, L / 2);
  return HE_OK;
}

int he_key_set_constant_time(he_key *key, int on) {
  if (!key) return fail(HE_ERR_ARG, "null key");
  key->dk.ct = on ? 1 : 0;
  return HE_OK;
}

uint32_t he_key_bits(const he_key *key) { return key ? key->n_bits : 0; }
int he_key_has_private(const he_key *key) { return key && key->priv ? 1 : 0; }

void he_key_free(he_key *key) {
  if (!key) return;
  if (key->blob) hipFree(key->blob);
  delete key;
}

int he_encode(const double *x, uint64_t count, uint32_t frac_bits, int64_t *m, uint32_t *n_bad,
              hipStream_t stream) {
  if (count == 0) return HE_OK;
  if (!x || !m) return fail(HE_ERR_ARG, "null x or m");
  if (frac_bits > 62) return fail(HE_ERR_ARG, "frac_bits must be <= 62");
  HE_TRY_HIP(he::launch_encode(x, count, frac_bits, m, n_bad, stream));
  return HE_OK;
}

int he_encrypt(const he_key *key, const int64_t *m, uint64_t count, const uint32_t *r, uint64_t r_seed,
               uint64_t r_offset, uint32_t *ct, hipStream_t stream) {
  if (count && !m) return fail(HE_ERR_ARG, "null m");
  return encrypt_impl(key, m, count, r, r_seed, r_offset, ct, stream, false);
}

int he_obfuscators(const he_key *key, uint64_t count, const uint32_t *r, uint64_t r_seed, uint64_t r_offset,
                   uint32_t *rho, hipStream_t stream) {
  return encrypt_impl(key, nullptr, count, r, r_seed, r_offset, rho, stream, false);
}

int he_encrypt_obfuscated(const he_key *key, const int64_t *m, uint64_t count, const uint32_t *rho,
                          uint32_t *ct, hipStream_t stream) {
  if (!key) return fail(HE_ERR_ARG, "null key");
  if (count == 0) return HE_OK;
  if (!m || !rho || !ct) return fail(HE_ERR_ARG, "null m, rho or ct");
  HE_TRY_HIP(he::launch_enc_obf(kp_of(key), key->dk, m, count, rho, ct, stream));
  return HE_OK;
}

int he_encrypt_public(const he_key *key, const int64_t *m, uint64_t count, const uint32_t *r,
                      uint64_t r_seed, uint64_t r_offset, uint32_t *ct, hipStream_t stream) {
  if (count && !m) return fail(HE_ERR_ARG, "null m");
  return encrypt_impl(key, m, count, r, r_seed, r_offset, ct, stream, true);
}

int he_hist_subtract(const he_key *key, const uint32_t *parent, const uint32_t *child, uint64_t count,
                     uint32_t batch, uint32_t *out, uint32_t *n_bad, hipStream_t stream) {
  if (!key) return fail(HE_ERR_ARG, "null key");
  if (count == 0) return HE_OK;
  if (!parent || !child || !out) return fail(HE_ERR_ARG, "null parent, child or out");
  const uint64_t bytes = count * (key->n_bits / 16) * sizeof(uint32_t);
  auto overlap = [bytes](const void *x, const void *y) {
    const uintptr_t a = (uintptr_t)x, b = (uintptr_t)y;
    return a < b + bytes && b < a + bytes;
  };
  if (overlap(out, parent) || overlap(out, child)) return fail(HE_ERR_ARG, "out overlaps parent or child");
  if (batch == 0) batch = he::ct_div_batch(count);
  if ((count + batch - 1) / batch > (uint64_t)16 * 0x7FFFFFFF) return fail(HE_ERR_ARG, "batch too small");
  HE_TRY_HIP(he::launch_ct_div(kp_of(key), key->dk, parent, child, count, batch, out, n_bad, stream));
  return HE_OK;
}

static_assert(sizeof(he_split) == 32, "he_split layout");

int he_split_find(const int64_t *hist, const int64_t *minus, uint32_t nodes, uint32_t n_features, uint32_t n_bins,
                  uint32_t frac_bits, double lambda, double gamma, double min_child_weight, int64_t *derived,
                  he_split *out_feature, he_split *out_node, hipStream_t stream) {
  if (nodes == 0 || n_features == 0) return HE_OK;
  if (!hist || !out_node) return fail(HE_ERR_ARG, "null hist or out_node");
  if (n_bins < 1 || n_bins > 256) return fail(HE_ERR_ARG, "n_bins must be in [1, 256]");
  if (frac_bits > 62) return fail(HE_ERR_ARG, "frac_bits must be at most 62");
  if (!(lambda >= 0.0) || !(min_child_weight >= 0.0) || !(gamma == gamma))
    return fail(HE_ERR_ARG, "lambda and min_child_weight must be >= 0, gamma a number");
  HE_TRY_HIP(he::launch_split(hist, minus, nodes, n_features, n_bins, std::ldexp(1.0, -(int)frac_bits), lambda,
                              gamma, min_child_weight, derived, out_feature, out_node, stream));
  return HE_OK;
}

int he_ct_mul(const he_key *key, const uint32_t *a, const uint32_t *b, uint64_t count, uint32_t *out,
              hipStream_t stream) {
  if (!key) return fail(HE_ERR_ARG, "null key");
  if (count == 0) return HE_OK;
  if (!a || !b || !out) return fail(HE_ERR_ARG, "null a, b or out");
  HE_TRY_HIP(he::launch_ct_mul(kp_of(key), key->dk, a, b, count, out, stream));
  return HE_OK;
}

int he_to_mont(const he_key *key, const uint32_t *in, uint64_t count, uint32_t *out, hipStream_t stream) {
  if (!key) return fail(HE_ERR_ARG, "null key");
  if (count == 0) return HE_OK;
  if (!in || !out) return fail(HE_ERR_ARG, "null buffer");
  HE_TRY_HIP(he::launch_mont_convert(kp_of(key), key->dk, in, count, out, true, stream));
  return HE_OK;
}

int he_from_mont(const he_key *key, const uint32_t *in, uint64_t count, uint32_t *out, hipStream_t stream) {
  if (!key) return fail(HE_ERR_ARG, "null key");
  if (count == 0) return HE_OK;
  if (!in || !out) return fail(HE_ERR_ARG, "null buffer");
  HE_TRY_HIP(he::launch_mont_convert(kp_of(key), key->dk, in, count, out, false, stream));
  return HE_OK;
}

int he_decrypt(const he_key *key, const uint32_t *ct, uint64_t count, int64_t *m, uint32_t *raw,
               uint32_t *n_overflow, hipStream_t stream) {
  if (!key) return fail(HE_ERR_ARG, "null key");
  if (!key->priv) return fail(HE_ERR_NOPRIV, "decryption needs p and q");
  if (count == 0) return HE_OK;
  if (!ct || !m) return fail(HE_ERR_ARG, "null ct or m");
  Workspace *w = workspace(stream);
  const int KP = kp_of(key);
  const size_t L = key->n_bits / 32;
  const he::DKey dk = key->dk;
  const int kind = he::pow_dec_kind(dk);
  he::PowPlan p = pow_plan(KP, kind, count);
  int rc = ensure(w->ctr, 256, stream);
  if (rc) return rc;
  p.ctr = (uint32_t *)w->ctr.p;
  // c^(P-1) mod P^2 per (ciphertext, prime): 2L limbs per ciphertext
  rc = ensure(w->tmp, count * 2 * L * sizeof(uint32_t), stream);
  if (rc) return rc;
  rc = ensure_tables(w->tab, KP, {{kind, &p}}, stream);
  if (rc) return rc;
  HE_TRY_HIP(he::launch_dec(KP, dk, ct, count, (uint32_t *)w->tmp.p, m, raw, n_overflow,
                            (uint32_t *)w->tab.p, p, stream));
  return HE_OK;
}

}  // extern "C"

// ------------------------------------------------- allocation-free decryption
// Scratch of he_decrypt_noalloc: c mod p^2 and c mod q^2, then their powers
// (2L words per ciphertext, at most half of the array), followed by the
// exponentiation window tables of the persistent launch, whose grid is cut
// to what the rest of the array holds.  One copy per device, held until the
// process ends; in host code `scratch` only names the symbol, its device
// address comes from hipGetSymbolAddress.
namespace {
constexpr size_t kNoAllocBytes = size_t(64) << 20;
constexpr int kNoAllocDevices = 64;
}  // namespace
static __device__ __align__(256) uint8_t scratch[kNoAllocBytes];
namespace {
std::mutex g_scratch_mu;
void *g_scratch_ptr[kNoAllocDevices] = {};

// Device address of this device's copy of `scratch` (looked up once per device).
int scratch_address(void **out) {
  int dev = 0;
  HE_TRY_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kNoAllocDevices)
    return fail(HE_ERR_DEVICE, "device index " + std::to_string(dev) + " beyond the allocation-free path's table");
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    HE_TRY_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return fail(HE_ERR_DEVICE, "hipGetSymbolAddress returned a null address for the scratch array");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return HE_OK;
}
}  // namespace

extern "C" {

int he_decrypt_noalloc(const he_key *key, const uint32_t *ct, uint64_t count, int64_t *m, uint32_t *raw,
                       uint32_t *n_overflow, hipStream_t stream) {
  if (!key) return fail(HE_ERR_ARG, "null key");
  if (!key->priv) return fail(HE_ERR_NOPRIV, "decryption needs p and q");
  if (count == 0) return HE_OK;
  if (!ct || !m) return fail(HE_ERR_ARG, "null ct or m");
  const int KP = kp_of(key);
  const size_t L = key->n_bits / 32;
  const uint64_t max_count = (kNoAllocBytes / 2) / (2 * L * sizeof(uint32_t));
  if (count > max_count)
    return fail(HE_ERR_ARG, "he_decrypt_noalloc: count " + std::to_string(count) + " exceeds the maximum of " +
                                std::to_string(max_count) + " ciphertexts at " + std::to_string(key->n_bits) +
                                "-bit keys (fixed scratch of " + std::to_string(kNoAllocBytes >> 20) + " MiB)");
  void *base = nullptr;
  int rc = scratch_address(&base);
  if (rc) return rc;
  const size_t xpq_bytes = (count * 2 * L * sizeof(uint32_t) + 255) / 256 * 256;
  // One launch whose grid is cut to the tables the scratch holds, at the
  // narrowest width that still puts a wave on every SIMD (a table holds as
  // many integers at every width, so wider groups mean more waves).
  const uint64_t cus = (uint64_t)he::device_cus();
  const he::DKey dk = key->dk;
  const int kind = he::pow_dec_kind(dk);
  he::PowLaunch l{};
  for (int G : {2, 4, 8, 16}) {
    l = pow_launch_at(KP, kind, count, PowShape{G, 0, 0});
    const uint64_t fit = (kNoAllocBytes - xpq_bytes) / he::table_bytes_per_block(KP, kind, G);
    if (fit == 0) return fail(HE_ERR_ARG, "he_decrypt_noalloc: no room for one block's window tables");
    l.grid = (uint32_t)std::min<uint64_t>(fit, l.grid);
    if (l.grid >= cus) break;
  }
  uint32_t *xpq = (uint32_t *)base;
  uint32_t *tab = (uint32_t *)((char *)base + xpq_bytes);
  // static units: no work counter in the scratch
  HE_TRY_HIP(he::launch_dec(KP, dk, ct, count, xpq, m, raw, n_overflow, tab,
                            he::PowPlan{l, count, he::PowLaunch{0, 0, 0}, nullptr}, stream));
  return HE_OK;
}

uint32_t he_pack_slots(const he_key *key, uint64_t count) {
  if (!key) return 0;
  return he::pack_slots((int)key->n_bits, count);
}

int he_pack(const he_key *key, const uint32_t *ct, uint64_t count, uint32_t slots, uint32_t *packed,
            hipStream_t stream) {
  if (!key) return fail(HE_ERR_ARG, "null key");
  if (slots < 1 || slots > (key->n_bits - 1) / 64) return fail(HE_ERR_ARG, "slots must be in [1, (n_bits - 1) / 64]");
  if (count == 0) return HE_OK;
  if (!ct || !packed) return fail(HE_ERR_ARG, "null ct or packed");
  HE_TRY_HIP(he::launch_pack(kp_of(key), key->dk, ct, count, slots, packed, stream));
  return HE_OK;
}

int he_decrypt_packed(const he_key *key, const uint32_t *packed, uint64_t count, uint32_t slots, int64_t *m,
                      uint32_t *n_overflow, hipStream_t stream) {
  if (!key) return fail(HE_ERR_ARG, "null key");
  if (!key->priv) return fail(HE_ERR_NOPRIV, "decryption needs p and q");
  if (slots < 1 || slots > (key->n_bits - 1) / 64) return fail(HE_ERR_ARG, "slots must be in [1, (n_bits - 1) / 64]");
  if (count == 0) return HE_OK;
  if (!packed || !m) return fail(HE_ERR_ARG, "null packed or m");
  const uint64_t n_packed = (count + slots - 1) / slots;
  const size_t L = key->n_bits / 32;
  Workspace *w = workspace(stream);
  const size_t raw_bytes = (n_packed * L * sizeof(uint32_t) + 255) & ~(size_t)255;
  int rc = ensure(w->unpack, raw_bytes + n_packed * sizeof(int64_t), stream);
  if (rc) return rc;
  uint32_t *raw = (uint32_t *)w->unpack.p;
  int64_t *whole = (int64_t *)((char *)w->unpack.p + raw_bytes);  // signed decode of the whole plaintext, unused
  rc = he_decrypt(key, packed, n_packed, whole, raw, nullptr, stream);
  if (rc) return rc;
  HE_TRY_HIP(he::launch_unpack(raw, count, slots, (uint32_t)L, m, n_overflow, stream));
  return HE_OK;
}

int he_hist_aggregate(const he_key *key, const uint32_t *ct, uint64_t rows, int ct_form,
                      const he_hist_job *jobs, uint32_t n_jobs, hipStream_t stream) {
  return he_hist_aggregate_ex(key, ct, rows, ct_form, jobs, n_jobs, 0, stream);
}

}  // extern "C"

namespace {
size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

// Device layout of one histogram batch: job descriptors, flat per-(feature,
// bin) arrays, work items, the permutation and the partial products.
struct HistLayout {
  std::vector<he::DJob> dj;
  uint64_t total_fb = 0, total_f = 0, total_blocks = 0, total_perm = 0, items_cap = 0;
  uint64_t contributions = 0, rows = 0;
  size_t o_jobs = 0, o_counts = 0, o_offs = 0, o_cursor = 0, o_fch = 0, o_fitem = 0, o_border = 0, o_nitems = 0,
         o_items = 0, o_perm = 0, o_part = 0, o_pairs = 0, bytes = 0;
  uint32_t chunk = 64, runs = 1;
  int waves = 0;          // product kernel: waves per SIMD cap (0: none)
  uint64_t pairs = 0;     // ciphertext pairs converted: every row, or (gather) the jobs' samples
  bool gather = false, mont = false, stretch = false;
  bool direct = false;    // no pairs: the products read the resident ciphertexts
};

// Work shapes callers may name: 16 lanes per sample, or 8 at 2048-bit keys.
bool hist_shape_valid(int KP, int lanes) { return lanes == 16 || (lanes == 8 && KP == 2); }
// Groups per (item, slot) of a work shape: `split` times one (8 lanes per
// sample: 4 per ciphertext) or two (16 lanes).
uint32_t hist_runs(uint32_t split, int lanes) { return split * (lanes == 8 ? 1u : 2u); }

int plan_layout(const he_key *key, const uint32_t *ct, uint64_t rows, int ct_form, const he_hist_job *jobs,
                uint32_t n_jobs, uint32_t chunk, uint32_t split, int lanes, HistLayout &lay, bool direct = false) {
  if (!key) return fail(HE_ERR_ARG, "null key");
  if (!jobs) return fail(HE_ERR_ARG, "null jobs");
  if (ct_form != HE_FORM_CANONICAL && ct_form != HE_FORM_MONT) return fail(HE_ERR_ARG, "bad ct_form");
  if (chunk == 0) chunk = 64;
  if (chunk > (1u << 20)) return fail(HE_ERR_ARG, "chunk too large");
  if (split != 1 && split != 2) return fail(HE_ERR_ARG, "split must be 1 or 2");
  const size_t S = 2 * (key->n_bits / 32);
  lay = HistLayout{};
  lay.dj.assign(n_jobs, he::DJob{});
  lay.rows = rows;
  lay.chunk = chunk;
  lay.runs = hist_runs(split, lanes);
  lay.mont = ct_form == HE_FORM_MONT;
  uint64_t samples = 0;
  for (uint32_t j = 0; j < n_jobs; ++j) {
    const he_hist_job &J = jobs[j];
    const std::string tag = "job " + std::to_string(j) + ": ";
    if (J.n_features == 0 || J.n_bins == 0 || J.n_bins > 256)
      return fail(HE_ERR_ARG, tag + "need n_features >= 1 and 1 <= n_bins <= 256");
    if (!J.hist || !J.bins || (J.n_samples && !J.sample_idx)) return fail(HE_ERR_ARG, tag + "null pointer");
    if (J.n_samples > rows || J.n_samples >= (1ull << 32)) return fail(HE_ERR_ARG, tag + "n_samples exceeds rows");
    if (J.n_samples && !ct) return fail(HE_ERR_ARG, "null ct");
    if (J.bins_ld < rows) return fail(HE_ERR_ARG, tag + "bins_ld < rows");
    he::DJob &d = lay.dj[j];
    d.idx = J.sample_idx;
    d.bins = J.bins;
    d.hist = J.hist;
    d.n = J.n_samples;
    d.ld = J.bins_ld;
    d.F = J.n_features;
    d.B = J.n_bins;
    d.fb_off = lay.total_fb;
    d.perm_off = lay.total_perm;
    d.blk_off = lay.total_blocks;
    d.f_off = (uint32_t)lay.total_f;
    d.nblk = (uint32_t)((J.n_samples + he::kSampleBlock - 1) / he::kSampleBlock);
    d.n_bad = J.n_bad;
    d.s_off = samples;
    samples += d.n;
    lay.total_fb += (uint64_t)d.F * d.B;
    lay.total_f += d.F;
    lay.total_blocks += (uint64_t)d.F * d.nblk;
    lay.total_perm += (uint64_t)d.F * d.n;
    lay.items_cap += (uint64_t)d.F * ((d.n + chunk - 1) / chunk + std::min<uint64_t>(d.B, d.n));
    lay.contributions += 2ull * d.F * d.n;
  }
  if (lay.items_cap >= (1ull << 32)) return fail(HE_ERR_ARG, "too many work items; use a larger chunk");
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = align_up(off + bytes);
    return o;
  };
  lay.o_jobs = take(n_jobs * sizeof(he::DJob));
  lay.o_counts = take((lay.total_fb + he::kHistClasses + 1) * 4);
  lay.o_offs = take(lay.total_fb * 4);
  lay.o_cursor = take(lay.total_fb * 4);
  lay.o_fch = take(lay.total_fb * 4);
  lay.o_fitem = take(lay.total_fb * 4);
  lay.o_border = take(lay.total_fb * 4);
  lay.o_nitems = take(8);  // item count, then the product kernel's work counter
  lay.o_items = take(std::max<uint64_t>(lay.items_cap, 1) * sizeof(he::HistItem));
  lay.o_perm = take(std::max<uint64_t>(lay.total_perm, 1) * 4);
  // partial products and the ciphertexts in two digits of 29-bit limbs: every
  // resident row, or where the jobs hold fewer samples those one by one
  const uint64_t row = 2 * (uint64_t)he29::limbs_for_group((int)S, he::kHistGroup) * 4;
  lay.o_part = take(std::max<uint64_t>(lay.items_cap, 1) * row);
  lay.direct = direct;
  if (!direct) {
    lay.gather = samples < rows;
    lay.pairs = lay.gather ? samples : rows;
    lay.o_pairs = take(std::max<uint64_t>(lay.pairs, 1) * row);
  }
  lay.bytes = off;
  return HE_OK;
}

he::HistWs bind_layout(const HistLayout &lay, const uint32_t *ct, char *base) {
  he::HistWs ws{};
  ws.jobs = (he::DJob *)(base + lay.o_jobs);
  ws.n_jobs = (uint32_t)lay.dj.size();
  ws.counts = (uint32_t *)(base + lay.o_counts);
  ws.cls = ws.counts + lay.total_fb;
  ws.scanned = ws.cls + he::kHistClasses;
  ws.offs = (uint32_t *)(base + lay.o_offs);
  ws.cursor = (uint32_t *)(base + lay.o_cursor);
  ws.fch = (uint32_t *)(base + lay.o_fch);
  ws.fitem = (uint32_t *)(base + lay.o_fitem);
  ws.border = (uint32_t *)(base + lay.o_border);
  ws.n_items = (uint32_t *)(base + lay.o_nitems);
  ws.next = ws.n_items + 1;
  ws.items = (he::HistItem *)(base + lay.o_items);
  ws.perm = (uint32_t *)(base + lay.o_perm);
  ws.partials = (uint32_t *)(base + lay.o_part);
  ws.pairs = lay.direct ? nullptr : (uint32_t *)(base + lay.o_pairs);
  ws.ct = ct;
  ws.mont = lay.mont ? 1u : 0u;
  ws.total_fb = lay.total_fb;
  ws.total_f = lay.total_f;
  ws.total_blocks = lay.total_blocks;
  ws.items_cap = lay.items_cap;
  ws.rows = lay.rows;
  ws.chunk = lay.chunk;
  ws.runs = lay.runs;
  ws.stretch = lay.stretch ? 1u : 0u;
  ws.gather = lay.gather ? 1u : 0u;
  return ws;
}

// Enqueues every kernel of one batch on `stream` (no allocation, no
// memset: safe to capture into a graph).
int enqueue_hist(const he_key *key, const uint32_t *ct, const HistLayout &lay, char *base, hipStream_t stream,
                 uint64_t *mm_count = nullptr) {
  he::HistWs ws = bind_layout(lay, ct, base);
  ws.mm_count = (unsigned long long *)mm_count;
  const int KP = kp_of(key);
  he::HistLaunch hl{0, he::hist_dyn_lds(KP, lay.direct, lay.waves)};
  // a wave takes 8 / runs items at a time
  const uint64_t waves = (lay.items_cap * lay.runs + 7) / 8;
  hl.grid = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(he::hist_resident_blocks(KP, lay.direct, hl.dyn),
                                                                     (waves + 3) / 4));
  HE_TRY_HIP(he::launch_hist(KP, key->dk, lay.pairs, lay.dj.data(), ws, hl, stream));
  return HE_OK;
}

int hist_run(const he_key *key, const uint32_t *ct, uint64_t rows, int ct_form, const he_hist_job *jobs,
             uint32_t n_jobs, uint32_t chunk, uint32_t split, hipStream_t stream, uint64_t *mm_count = nullptr,
             int G = he::kHistGroup, int waves = 0, bool stretch = false) {
  if (n_jobs == 0) return key ? HE_OK : fail(HE_ERR_ARG, "null key");
  HistLayout lay;
  int rc = plan_layout(key, ct, rows, ct_form, jobs, n_jobs, chunk, split, G, lay);
  if (rc) return rc;
  Workspace *w = workspace(stream);
  rc = ensure(w->hist, lay.bytes, stream);
  if (rc == HE_ERR_OOM && lay.pairs) {
    // no memory for the ciphertexts in two digits beside the caller's
    rc = plan_layout(key, ct, rows, ct_form, jobs, n_jobs, chunk, split, G, lay, true);
    if (!rc) rc = ensure(w->hist, lay.bytes, stream);
  }
  if (rc) return rc;
  lay.waves = waves;
  lay.stretch = stretch;
  return enqueue_hist(key, ct, lay, (char *)w->hist.p, stream, mm_count);
}

// Autotuner cache: best (chunk, split) per shape class.
struct TuneKey {
  uint32_t bits, log2_contrib, log2_jobs, max_bins;
  bool operator<(const TuneKey &o) const {
    return std::tie(bits, log2_contrib, log2_jobs, max_bins) < std::tie(o.bits, o.log2_contrib, o.log2_jobs, o.max_bins);
  }
};
struct TuneVal {
  uint32_t chunk, split;
  float ms;
  int G = he::kHistGroup, waves = 0;
  bool stretch = false;  // longer items for full bins: the default shape only
};
std::mutex g_tune_mu;
std::map<TuneKey, TuneVal> g_tune;

uint32_t ilog2(uint64_t x) {
  uint32_t r = 0;
  while (x > 1) {
    x >>= 1;
    ++r;
  }
  return r;
}

TuneKey tune_key(const he_key *key, const he_hist_job *jobs, uint32_t n_jobs) {
  uint64_t contrib = 0;
  uint32_t mb = 0;
  for (uint32_t j = 0; j < n_jobs; ++j) {
    contrib += 2ull * jobs[j].n_features * jobs[j].n_samples;
    mb = std::max(mb, jobs[j].n_bins);
  }
  return TuneKey{key->n_bits, ilog2(contrib + 1), ilog2(n_jobs), mb};
}

// Work shape of an untuned batch (chunk 0, no autotuner entry for its class):
// two runs per (item, slot), joined in the wave, of at most `len` samples each.
// A wave per SIMD holds 8,192 runs of both slots, so W samples x features make
// W / (8192 len) rounds of them; about two to four rounds even out the ends
// (the last round is the shortest items), longer runs save joins.  Below 8
// samples the joins of the partials cost more than the rounds save, except
// for the smallest batches, where nothing else fills the device.  Measured at
// 2048 bits (ms at half, this and twice the length): W = 8,000 0.20 / 0.20 /
// 0.24; 36,000 0.33 / 0.29 / 0.39; 168,000 0.73 / 0.62 / 0.74; 480,000 1.32 /
// 1.13 / 1.14; 3,200,000 6.35 / 6.18 / 6.31; 14.7 M 46.2 / 45.4 / -.  At 1024 bits
// the best lengths are the same to one doubling, the rule's within 8% of them: W =
// 8,000 0.124 / 0.112 / 0.124; 36,000 0.21 / 0.18 / 0.20; 165,000 0.44 / 0.38 / 0.36;
// 480,000 0.93 / 0.83 / 0.92; 1,280,000 1.33 / 1.43 / 1.74; 3,200,000 2.55 / 2.50 /
// 2.69; 12.8 M 9.42 / 9.33 / 9.47.
// The bins' counts are known on the device only: there a full bin's items are
// longer (item_chunk).  100,000 samples of one feature at 2048 bits, all in one
// bin 5.33 -> 1.88 ms, in two 2.92 -> 1.36; 32 features x 256 Zipf bins as before.
TuneVal default_hist_shape(const he_hist_job *jobs, uint32_t n_jobs) {
  uint64_t w = 0;
  for (uint32_t j = 0; j < n_jobs; ++j) w += (uint64_t)jobs[j].n_features * jobs[j].n_samples;
  const uint32_t lo = w < 16000 ? 4 : 8, hi = w < 6000000 ? 64 : 128;
  uint32_t len = lo;
  while (len < hi && (uint64_t)len * 2 * 20000 <= w) len *= 2;
  return TuneVal{2 * len, 2, 0.f, 8, 0, true};
}

}  // namespace

extern "C" int he_hist_aggregate_ex(const he_key *key, const uint32_t *ct, uint64_t rows, int ct_form,
                                    const he_hist_job *jobs, uint32_t n_jobs, uint32_t chunk,
                                    hipStream_t stream) {
  uint32_t split = 2;
  int G = he::kHistGroup, waves = 0;
  bool stretch = false;
  if (chunk == 0 && key && jobs && n_jobs) {
    TuneVal v = default_hist_shape(jobs, n_jobs);
    {
      std::lock_guard<std::mutex> lk(g_tune_mu);
      auto it = g_tune.find(tune_key(key, jobs, n_jobs));
      if (it != g_tune.end()) v = it->second;
    }
    chunk = v.chunk;
    split = v.split;
    G = v.G;
    waves = v.waves;
    stretch = v.stretch;
  }
  return hist_run(key, ct, rows, ct_form, jobs, n_jobs, chunk, split, stream, nullptr, G, waves, stretch);
}

extern "C" int he_hist_aggregate_counted(const he_key *key, const uint32_t *ct, uint64_t rows, int ct_form,
                                         const he_hist_job *jobs, uint32_t n_jobs, uint32_t chunk, uint32_t split,
                                         uint32_t lanes, uint32_t waves, uint64_t *mm_count, hipStream_t stream) {
  if (!mm_count) return fail(HE_ERR_ARG, "null mm_count");
  if (split != 1 && split != 2) return fail(HE_ERR_ARG, "split must be 1 or 2");
  if (!key) return fail(HE_ERR_ARG, "null key");
  if (lanes == 0) lanes = he::kHistGroup;
  if (!hist_shape_valid(kp_of(key), (int)lanes))
    return fail(HE_ERR_ARG, "lanes must be 16, or 8 at 2048-bit keys");
  if (waves > 8) return fail(HE_ERR_ARG, "waves must be 0 (own occupancy) to 8");
  return hist_run(key, ct, rows, ct_form, jobs, n_jobs, chunk, split, stream, mm_count, (int)lanes, (int)waves);
}

extern "C" int he_hist_autotune(const he_key *key, const uint32_t *ct, uint64_t rows, int ct_form,
                                const he_hist_job *jobs, uint32_t n_jobs, uint32_t *chunk_out,
                                uint32_t *split_out, uint32_t *lanes_out, uint32_t *waves_out, float *ms_out,
                                hipStream_t stream) {
  if (!key || !jobs || n_jobs == 0) return fail(HE_ERR_ARG, "need a key and at least one job");
  static const uint32_t chunks[] = {16, 32, 64, 128, 256, 512};
  hipEvent_t e0, e1;
  HE_TRY_HIP(hipEventCreate(&e0));
  HE_TRY_HIP(hipEventCreate(&e1));
  TuneVal best{64, 2, 1e30f};
  TuneVal best_g[2] = {{64, 2, 1e30f}, {64, 2, 1e30f}};  // per lanes per ciphertext: [0] 16, [1] 8
  int rc = HE_OK;
  auto trial = [&](uint32_t c, uint32_t split, int G, int waves) -> int {
    int r = hist_run(key, ct, rows, ct_form, jobs, n_jobs, c, split, stream, nullptr, G, waves);  // warm-up
    if (r) return r;
    HE_TRY_HIP(hipEventRecord(e0, stream));
    for (int k = 0; k < 2 && !r; ++k) r = hist_run(key, ct, rows, ct_form, jobs, n_jobs, c, split, stream, nullptr, G, waves);
    if (r) return r;
    HE_TRY_HIP(hipEventRecord(e1, stream));
    HE_TRY_HIP(hipEventSynchronize(e1));
    float ms = 0;
    HE_TRY_HIP(hipEventElapsedTime(&ms, e0, e1));
    ms /= 2;
    const TuneVal v{c, split, ms, G, waves};
    if (ms < best.ms) best = v;
    TuneVal &bg = best_g[G == he::kHistGroup ? 0 : 1];
    if (ms < bg.ms) bg = v;
    return HE_OK;
  };
  // work items (chunk, groups per item) for each lane count at the kernel's
  // own occupancy (the 8-lane waves take two or four items at once, so their
  // best items differ), then waves per SIMD at the best items of each
  const int KP = kp_of(key);
  for (int G : {he::kHistGroup, 8}) {
    if (rc || !hist_shape_valid(KP, G)) continue;
    for (uint32_t split : {2u, 1u}) {
      for (uint32_t c : chunks) {
        if (G != he::kHistGroup && (c < 32 || c > 256)) continue;  // 8 lanes: the middle lengths only
        if ((rc = trial(c, split, G, 0))) break;
      }
      if (rc) break;
    }
  }
  for (int G : {he::kHistGroup, 8}) {
    if (rc || !hist_shape_valid(KP, G)) continue;
    const TuneVal bg = best_g[G == he::kHistGroup ? 0 : 1];
    for (int waves : {4, 3, 2}) {
      if (he::hist_dyn_lds(KP, false, waves) == 0) continue;  // no cap needed: same as its own occupancy
      if ((rc = trial(bg.chunk, bg.split, G, waves))) break;
    }
  }
  hipEventDestroy(e0);
  hipEventDestroy(e1);
  if (rc) return rc;
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tune[tune_key(key, jobs, n_jobs)] = best;
  }
  if (chunk_out) *chunk_out = best.chunk;
  if (split_out) *split_out = best.split;
  if (lanes_out) *lanes_out = (uint32_t)best.G;
  if (waves_out) *waves_out = (uint32_t)best.waves;
  if (ms_out) *ms_out = best.ms;
  return HE_OK;
}

// ------------------------------------------- exponentiation shape autotuner
namespace {
struct DevBuf {
  void *p = nullptr;
  ~DevBuf() {
    if (p) hipFree(p);
  }
};

// Times `launch` (two runs after one warm-up) on `stream`; ms per run.
template <typename F>
int time_ms(F launch, hipStream_t stream, hipEvent_t e0, hipEvent_t e1, float *ms) {
  HE_TRY_HIP(launch());
  HE_TRY_HIP(hipEventRecord(e0, stream));
  for (int r = 0; r < 2; ++r) HE_TRY_HIP(launch());
  HE_TRY_HIP(hipEventRecord(e1, stream));
  HE_TRY_HIP(hipEventSynchronize(e1));
  HE_TRY_HIP(hipEventElapsedTime(ms, e0, e1));
  *ms /= 2;
  return HE_OK;
}
}  // namespace

extern "C" int he_crt_autotune(const he_key *key, uint64_t enc_count, uint64_t dec_count, uint32_t *choice,
                               float *ms_out, hipStream_t stream) {
  if (!key) return fail(HE_ERR_ARG, "null key");
  if (!key->priv) return fail(HE_ERR_NOPRIV, "the CRT exponentiations need p and q");
  if (enc_count == 0 || dec_count == 0) return fail(HE_ERR_ARG, "need enc_count >= 1 and dec_count >= 1");
  const int KP = kp_of(key);
  const size_t L = key->n_bits / 32;
  const uint64_t n_ct = std::max(enc_count, dec_count);
  int dev = 0;
  HE_TRY_HIP(hipGetDevice(&dev));
  // trial buffers: r mod P / t, omega, ciphertexts, their powers, window
  // tables, work counters
  DevBuf tq, cpq, ct, xpq, tab, ctr;
  size_t tab_bytes = 0;
  // mod P, the lift (with public digits: both powers at once), decryption
  const int kinds[3] = {4, he::pow_lift_kind(key->dk), he::pow_dec_kind(key->dk)};
  for (int kind : kinds)
    for (int G : {1, 2, 4, 8, 16})
      if (he::pow_shape_valid(KP, kind, G))
        tab_bytes = std::max<size_t>(tab_bytes, (size_t)he::pow_resident_blocks(KP, kind, G, 0) *
                                                   he::table_bytes_per_block(KP, kind, G));
  const size_t sizes[5] = {n_ct * L * 4, n_ct * 2 * L * 4, n_ct * 2 * L * 4, n_ct * 2 * L * 4, 256};
  DevBuf *bufs[5] = {&tq, &cpq, &ct, &xpq, &ctr};
  for (int b = 0; b < 5; ++b)
    if (hipMalloc(&bufs[b]->p, sizes[b]) != hipSuccess) {
      hipGetLastError();
      return fail(HE_ERR_OOM, "autotuner trial buffers");
    }
  uint32_t *tq_p = (uint32_t *)tq.p, *cpq_p = (uint32_t *)cpq.p, *ct_p = (uint32_t *)ct.p,
           *xpq_p = (uint32_t *)xpq.p;
  // real operands: r mod P, one encryption (default shapes)
  HE_TRY_HIP(he::launch_enc_r(KP, key->dk, enc_count, nullptr, 1, 0, tq_p, stream));
  int rc = encrypt_impl(key, nullptr, n_ct, nullptr, 1, 0, ct_p, stream, false);
  if (rc) return rc;
  // the window tables, or what there is room for: shapes that need more are not tried
  while (hipMalloc(&tab.p, tab_bytes) != hipSuccess) {
    hipGetLastError();
    tab.p = nullptr;
    tab_bytes /= 2;
    if (tab_bytes < (1u << 20)) return fail(HE_ERR_OOM, "autotuner window tables");
  }
  uint32_t *tab_p = (uint32_t *)tab.p;
  hipEvent_t e0, e1;
  HE_TRY_HIP(hipEventCreate(&e0));
  HE_TRY_HIP(hipEventCreate(&e1));
  PowShape best[3];
  float best_ms[3] = {1e30f, 1e30f, 1e30f};
  for (int t = 0; t < 3 && !rc; ++t) {
    const int kind = kinds[t];
    const uint64_t count = t == 2 ? dec_count : enc_count;
    auto trial = [&](const PowShape &sh, he::PowPlan p) -> int {
      if (plan_table_bytes(KP, kind, p) > tab_bytes) return HE_OK;
      p.ctr = (uint32_t *)ctr.p;
      auto run = [&]() -> hipError_t {
        return he::launch_pow_kind(KP, key->dk, kind, t == 2 ? ct_p : tq_p, t == 0 ? tq_p : (t == 2 ? xpq_p : cpq_p), count,
                                   tab_p, p, stream);
      };
      float ms = 0;
      const int r = time_ms(run, stream, e0, e1, &ms);
      if (r) return r;
      if (ms < best_ms[t]) {
        best_ms[t] = ms;
        best[t] = sh;
      }
      return HE_OK;
    };
    // Ordinary keys have no step mod P: its present plan is timed for the report
    // and nothing remembered (a sweep took 15 times three launches of up to 140 ms
    // each at 200,000 encryptions).
    if (t == 0 && !key->dk.ct) {
      rc = trial(pow_pin(KP, kind, count), pow_plan(KP, kind, count));
      continue;
    }
    // lanes per integer and waves per SIMD in one launch, then, at the best
    // of those, a separate launch for the last partial round at each wider
    // group
    for (int G : {1, 2, 4, 8, 16}) {
      if (!pow_shape_named(KP, kind, G)) continue;
      for (int waves : {0, 3, 2}) {
        const PowShape sh{G, waves, 0};
        const he::PowPlan p = pow_plan_at(KP, kind, count, sh);
        if (waves && p.main.dyn == 0) continue;  // the kernel's own occupancy is already at most `waves`
        if ((rc = trial(sh, p))) break;
      }
      if (rc) break;
    }
    // the default plan, kept as such (its split follows the count), unless it is
    // one of the launches above
    const PowShape one = best[t];
    const he::PowPlan dp = default_pow_plan(KP, kind, count);
    if (!rc && (dp.tail.G || !pow_shape_named(KP, kind, dp.main.G))) rc = trial(PowShape{}, dp);
    for (int tg : {4, 8, 16}) {
      if (rc || one.G == 0 || tg <= one.G || !he::pow_shape_valid(KP, kind, tg)) continue;
      const PowShape sh{one.G, one.waves, tg};
      const he::PowPlan p = pow_plan_at(KP, kind, count, sh);
      if (p.tail.G == 0) break;  // whole rounds only, or less than one: nothing to split
      rc = trial(sh, p);
    }
  }
  hipEventDestroy(e0);
  hipEventDestroy(e1);
  HE_TRY_HIP(hipStreamSynchronize(stream));
  if (rc) return rc;
  {
    std::lock_guard<std::mutex> lk(g_pow_mu);
    for (int t = key->dk.ct ? 0 : 1; t < 3; ++t)
      g_pow_tuned[{dev, KP, kinds[t], count_class(t == 2 ? dec_count : enc_count)}] = best[t];
  }
  for (int t = 0; t < 3; ++t) {
    if (choice) {
      choice[3 * t] = (uint32_t)best[t].G;
      choice[3 * t + 1] = (uint32_t)best[t].waves;
      choice[3 * t + 2] = (uint32_t)best[t].tailG;
    }
    if (ms_out) ms_out[t] = best_ms[t] < 1e30f ? best_ms[t] : 0.f;
  }
  return HE_OK;
}

extern "C" int he_crt_set_shape(const he_key *key, uint32_t kind, uint64_t count, uint32_t lanes, uint32_t waves,
                                uint32_t tail_lanes) {
  if (!key) return fail(HE_ERR_ARG, "null key");
  if (kind > 3)
    return fail(HE_ERR_ARG, "kind must be 0 (mod p), 1 (lift), 2 (decryption) or 3 (public-key encryption)");
  if (count == 0) return fail(HE_ERR_ARG, "count must be at least 1");
  const int KP = kp_of(key), k = kind == 0 ? 4 : (kind == 1 ? 0 : (kind == 2 ? 2 : 1));
  // public-key encryption plans its exponentiation over unit pairs of two ciphertexts
  const uint64_t units = kind == 3 ? (count + 1) / 2 : count;
  if (lanes != 0 && !pow_shape_named(KP, k, (int)lanes))
    return fail(HE_ERR_ARG, "lanes " + std::to_string(lanes) + " not a shape of this kind and key size");
  if (lanes == 0 && (waves != 0 || tail_lanes != 0))
    return fail(HE_ERR_ARG, "the default plan (lanes 0) has no waves or tail_lanes");
  if (waves != 0 && waves != 2 && waves != 3) return fail(HE_ERR_ARG, "waves must be 0 (own occupancy), 2 or 3");
  if (tail_lanes != 0 && (tail_lanes <= lanes || !pow_shape_named(KP, k, (int)tail_lanes)))
    return fail(HE_ERR_ARG, "tail_lanes must be 0 or a built width above lanes");
  int dev = 0;
  HE_TRY_HIP(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lk(g_pow_mu);
  // a pin holds for every key of this size: the lift and decryption with secret
  // digits and without
  const int both[2] = {k, k == 0 ? 3 : (k == 2 ? 5 : k)};
  for (int kk : both)
    g_pow_tuned[{dev, KP, kk, count_class(units)}] = PowShape{(int)lanes, (int)waves, (int)tail_lanes};
  return HE_OK;
}

// ------------------------------------------------------------ captured plans
struct he_hist_plan {
  const he_key *key = nullptr;
  HistLayout lay;
  void *ws = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

extern "C" void he_hist_plan_free(he_hist_plan *plan) {
  if (!plan) return;
  if (plan->exec) hipGraphExecDestroy(plan->exec);
  if (plan->graph) hipGraphDestroy(plan->graph);
  if (plan->ws) hipFree(plan->ws);
  delete plan;
}

extern "C" int he_hist_plan_create(const he_key *key, const uint32_t *ct, uint64_t rows, int ct_form,
                                   const he_hist_job *jobs, uint32_t n_jobs, uint32_t chunk, uint32_t split,
                                   he_hist_plan **out) {
  if (!out) return fail(HE_ERR_ARG, "null out");
  if (!key || !jobs || n_jobs == 0) return fail(HE_ERR_ARG, "need a key and at least one job");
  int G = he::kHistGroup, waves = 0;
  bool stretch = false;
  if (chunk == 0) {
    TuneVal v = default_hist_shape(jobs, n_jobs);
    {
      std::lock_guard<std::mutex> lk(g_tune_mu);
      auto it = g_tune.find(tune_key(key, jobs, n_jobs));
      if (it != g_tune.end()) v = it->second;
    }
    chunk = v.chunk;
    if (split == 0) split = v.split;
    G = v.G;
    waves = v.waves;
    stretch = v.stretch;
  }
  if (split == 0) split = 2;
  he_hist_plan *p = new (std::nothrow) he_hist_plan();
  if (!p) return fail(HE_ERR_OOM, "out of host memory");
  p->key = key;
  int rc = plan_layout(key, ct, rows, ct_form, jobs, n_jobs, chunk, split, G, p->lay);
  if (rc) {
    delete p;
    return rc;
  }
  if (hipMalloc(&p->ws, std::max<size_t>(p->lay.bytes, 256)) != hipSuccess) {
    hipGetLastError();
    p->ws = nullptr;
    // no memory for the ciphertexts in two digits beside the caller's
    if (p->lay.pairs) rc = plan_layout(key, ct, rows, ct_form, jobs, n_jobs, chunk, split, G, p->lay, true);
    if (rc || !p->lay.direct || hipMalloc(&p->ws, std::max<size_t>(p->lay.bytes, 256)) != hipSuccess) {
      hipGetLastError();
      const size_t bytes = p->lay.bytes;
      delete p;
      return rc ? rc : fail(HE_ERR_OOM, "plan workspace allocation of " + std::to_string(bytes) + " bytes failed");
    }
  }
  p->lay.waves = waves;
  p->lay.stretch = stretch;
  // resident block counts and LDS caps are queried before capture
  // (occupancy calls are not stream work, but keep capture free of anything
  // but launches)
  (void)he::hist_resident_blocks(kp_of(key), p->lay.direct, he::hist_dyn_lds(kp_of(key), p->lay.direct, waves));
  hipStream_t cs;
  if (hipStreamCreateWithFlags(&cs, hipStreamNonBlocking) != hipSuccess) {
    he_hist_plan_free(p);
    return fail(HE_ERR_DEVICE, "stream creation failed");
  }
  hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
  if (e == hipSuccess) {
    rc = enqueue_hist(key, ct, p->lay, (char *)p->ws, cs);
    hipError_t e2 = hipStreamEndCapture(cs, &p->graph);
    if (rc == HE_OK && e2 != hipSuccess) rc = fail(HE_ERR_DEVICE, std::string("capture: ") + hipGetErrorString(e2));
  } else {
    rc = fail(HE_ERR_DEVICE, std::string("begin capture: ") + hipGetErrorString(e));
  }
  hipStreamDestroy(cs);
  if (rc == HE_OK) {
    e = hipGraphInstantiate(&p->exec, p->graph, nullptr, nullptr, 0);
    if (e != hipSuccess) rc = fail(HE_ERR_DEVICE, std::string("instantiate: ") + hipGetErrorString(e));
  }
  if (rc != HE_OK) {
    he_hist_plan_free(p);
    return rc;
  }
  *out = p;
  return HE_OK;
}

extern "C" int he_hist_plan_launch(he_hist_plan *plan, hipStream_t stream) {
  if (!plan || !plan->exec) return fail(HE_ERR_ARG, "null plan");
  HE_TRY_HIP(hipGraphLaunch(plan->exec, stream));
  return HE_OK;
}

extern "C" int he_probe_int_mul(uint64_t iters, uint32_t blocks, uint64_t *products, hipStream_t stream) {
  if (!blocks || !iters) return fail(HE_ERR_ARG, "iters and blocks must be > 0");
  Workspace *w = workspace(stream);
  int rc = ensure(w->tmp, 256, stream);
  if (rc) return rc;
  HE_TRY_HIP(he::launch_probe_mul(iters, blocks, (uint32_t *)w->tmp.p, stream));
  if (products) *products = (uint64_t)blocks * 256 * iters * 8;
  return HE_OK;
}
