// Internal interfaces between the host runtime (he_api.cpp) and the kernels
// (he_kernels.hip).  Not part of the public ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "radix29.hpp"

namespace he {

// One Montgomery modulus N of S limbs (R = 2^(32 S)); device pointers into
// the key's constant blob, each S limbs.  The radix-2^29 form (R' =
// 2^(29 S29), one set per limb-count variant) serves the exponentiations.
struct DMod {
  const uint32_t *N, *R1, *R2, *R3;       // N, R^k mod N
  uint32_t ninv;                          // -N^-1 mod 2^32
  // radix 2^29, null for a variant that no kernel reads
  const uint32_t *N29[he29::kVariants];   // N in S29 limbs of 29 bits
  const uint32_t *R1_29[he29::kVariants]; // R' mod N
  const uint32_t *R2_29[he29::kVariants]; // R'^2 mod N
};

// Exponent as limbs with one zero limb of padding and its fixed-window
// count, and its sliding-window schedule (keysetup.hpp, sliding_schedule).
struct DExp {
  const uint32_t *e;
  int nwin;
  const uint32_t *ops;
  int nops;
};

// Constants of the two-digit form of residues mod N^2 (radix29.hpp), per
// limb-count variant.
struct DPair {
  const uint32_t *c[he29::kPairVariants];
  uint32_t ninv;  // -N^-1 mod 2^32
};

// Arguments of an exponentiation on the engines of pair29.hpp: unit (i, w)
// reads its pieces at in + i in_i + w in_w and writes its digits at
// out + i out_i + w out_w.
struct PairPowArgs {
  const uint32_t *consts[2];
  uint32_t ninv[2];
  DExp exp[2];
  const uint32_t *in;
  uint32_t *out;
  uint32_t in_i, in_w, out_i, out_w;
  int pieces;
  uint64_t count;
  uint32_t *tabs;
  uint32_t *next;
};
// Exponentiation schedules: sliding windows, fixed windows with masked table
// reads (secret digits), or two exponents that share their squarings.
enum class PairPow { kSliding, kMasked, kJoint };
// The kernel for a base of SN 32-bit limbs at L lanes per integer (0: one
// residue mod N per lane, masked only), null if not built.
const void *pow_pair_kernel(int SN, int L, PairPow which);

// Per-prime constants for the CRT paths; P is this prime, Q the other one.
// S_P = L/2 limbs for P, S_P2 = L limbs for P^2 (L = limbs of n).
struct DPrime {
  DMod P, P2;
  DPair pair;
  DExp e_enc;        // Q mod (P - 1): r^Q mod P = r^(Q mod (P-1)) mod P
  DExp e_lift;       // P: x -> x^P mod P^2 depends only on x mod P
  DExp e_dec;        // P - 1: decryption exponent
  DExp joint;        // schedule of the powers P - 1 and e_enc mod P^2 of one base (ops only)
  const uint32_t *QR2_P;  // Q R^2 mod P        (S_P limbs)
  const uint32_t *PR_P2;  // P R' mod P^2       (S_P2 limbs)
  const uint32_t *Pinv;   // P^-1 mod 2^(32 S_P)
  const uint32_t *hR_P;   // h_P R mod P, h_P = L_P(g^(P-1) mod P^2)^-1 mod P
};

struct DKey {
  uint32_t n_bits;
  int has_priv;
  DMod n, n2;              // S_N = L, S_N2 = 2L limbs
  DPair pair_n;
  DExp e_n;                // n as an exponent (public encryption)
  const uint32_t *nR_n2;   // n R'' mod n^2
  const uint32_t *half;    // (n + 1) / 2 (L limbs) for the signed decode
  DPrime pr[2];            // [0]: P = p, Q = q; [1]: P = q, Q = p
  const uint32_t *Cq;      // (q^2)^-1 R' mod p^2
  const uint32_t *q2R_n2;  // q^2 R'' mod n^2
  const uint32_t *qinv_p;  // q^-1 mod p (canonical)
  const uint32_t *qR_n;    // q R_n mod n
  int ct;                  // private-key exponentiations read their window tables in full (secret digits)
};

// Histogram job as the kernels see it (host fills offsets).
struct DJob {
  const uint32_t *idx;
  const uint8_t *bins;
  uint32_t *hist;
  uint64_t n;          // samples in the node
  uint64_t ld;         // bins leading dimension
  uint32_t F, B;       // features, bins
  uint64_t fb_off;     // first (feature, bin) entry of this job in the flat lists
  uint64_t perm_off;   // first perm slot of this job (F * n slots)
  uint64_t blk_off;    // first sample block of this job (F * nblk blocks)
  uint32_t f_off;      // first (job, feature) entry
  uint32_t nblk;       // sample blocks per feature
  uint32_t *n_bad;     // optional: skipped (sample, feature) pairs, device counter
  uint64_t s_off;      // first of this job's samples among the batch's (gathered pairs)
};

struct HistItem {      // one chunk of one (feature, bin): perm[start .. start+len)
  uint64_t start;
  uint32_t len;
  uint32_t pad;
};

// Flat device workspace of one histogram batch.
constexpr int kHistClasses = 1024;  // item lengths told apart in the items' order
struct HistWs {
  DJob *jobs;
  uint32_t n_jobs;
  uint32_t *counts;                                // [total_fb], then the classes and the scan's block count
  uint32_t *cls;                                   // [kHistClasses] items per length, then each length's next item
  uint32_t *scanned;                               // (job, feature) pairs scanned
  uint32_t *offs, *cursor, *fch, *fitem;           // [total_fb]
  uint32_t *border;                                // [total_fb]: per (job, feature), its bins by decreasing count
  uint32_t *n_items;                               // device scalar
  uint32_t *next;                                  // device scalar: the product kernel's next wave unit
  HistItem *items;                                 // [items_cap]
  uint32_t *perm;                                  // [total_perm]: index into pairs
  uint32_t *pairs;                                 // [rows or samples][2][2 S29]: the ciphertexts in two digits,
                                                   // null: read from ct (mont: HE_FORM_MONT)
  const uint32_t *ct;
  uint32_t mont;
  uint32_t *partials;                              // [items_cap][2][2 S29]
  uint64_t total_fb, total_f, total_blocks, items_cap;
  uint64_t rows;                                   // resident ciphertext rows
  uint32_t chunk;                                  // most samples per item
  uint32_t stretch;                                // longer items for full bins (item_chunk)
  uint32_t runs;                                   // groups per (item, slot): 1, 2 or 4
  uint32_t gather;                                 // pairs holds the jobs' samples, not every row
  unsigned long long *mm_count;                    // optional debug counters [3], else null
};

constexpr int kWindowBits = 5;     // exponent window width (see mont.hpp)
constexpr int kSampleBlock = 4096;   // samples per bucketing block
constexpr int kBlockThreads = 256;   // 4 waves
constexpr int kHistGroup = 16;      // lanes per integer of the Montgomery form the histograms take (its R')
constexpr int kHistLanes = 4;       // lanes per ciphertext in the histogram products

// ---- launchers (he_kernels.hip) ------------------------------------------------
// KP = limbs per lane of a prime: 1 for 1024-bit keys, 2 for 2048-bit keys.
hipError_t launch_encode(const double *x, uint64_t count, uint32_t frac_bits, int64_t *m,
                         uint32_t *n_bad, hipStream_t s);
// Launch shape of a private-key exponentiation (k_pow): lanes per integer,
// grid, and dynamic LDS reserved only to cap the blocks per compute unit.
struct PowLaunch {
  int G;
  uint32_t grid;
  uint32_t dyn;
};
// A private-key exponentiation over `count` ciphertexts in up to two
// launches: the first main_count ciphertexts at `main`, whose resident waves
// then all take the same number of work units, and the rest (what would be
// a last, partly filled round) at `tail`, a narrower group per integer so
// that it spreads over more waves.  tail.G == 0: one launch of everything
// at `main` (main_count unused).  ctr: two device words for the launches'
// work counters (cleared by the launcher), or null for static units.
struct PowPlan {
  PowLaunch main;
  uint64_t main_count;
  PowLaunch tail;
  uint32_t *ctr;
};
// tq: [count][2][S_P] (r mod P, then t in place), cpq: [count][2][S_P2] (omega
// as two digits base P).
hipError_t launch_enc_crt(int KP, const DKey &k, const int64_t *m, uint64_t count, const uint32_t *r, uint64_t seed,
                          uint64_t roff, uint32_t *tq, uint32_t *cpq, uint32_t *ct, uint32_t *tab,
                          const PowPlan &p1, const PowPlan &p2, hipStream_t s);
// Public-key encryption: x holds count + (count & 1) rows of 3 S_N limbs (all
// rows of r mod n, then all of r^n mod n^2 as two digits base n); p plans the exponentiation over (count + 1) / 2
// unit pairs (kind 1).
hipError_t launch_enc_pub(int KP, const DKey &k, const int64_t *m, uint64_t count, const uint32_t *r, uint64_t seed,
                          uint64_t roff, uint32_t *x, uint32_t *ct, uint32_t *tab, const PowPlan &p, hipStream_t s);
// m null: 2^63 for every ciphertext.
hipError_t launch_enc_obf(int KP, const DKey &k, const int64_t *m, uint64_t count, const uint32_t *rho,
                          uint32_t *ct, hipStream_t s);
uint32_t ct_div_batch(uint64_t count);
hipError_t launch_ct_div(int KP, const DKey &k, const uint32_t *num, const uint32_t *den, uint64_t count,
                         uint32_t batch, uint32_t *out, uint32_t *n_bad, hipStream_t s);
hipError_t launch_split(const int64_t *hist, const int64_t *minus, uint32_t nodes, uint32_t F, uint32_t B,
                        double scale, double lam, double gamma, double mcw, int64_t *derived, void *out_feat,
                        void *out_node, hipStream_t s);
hipError_t launch_ct_mul(int KP, const DKey &k, const uint32_t *a, const uint32_t *b, uint64_t count,
                         uint32_t *out, hipStream_t s);
hipError_t launch_pack(int KP, const DKey &k, const uint32_t *ct, uint64_t count, uint32_t slots,
                       uint32_t *packed, hipStream_t s);
hipError_t launch_unpack(const uint32_t *raw, uint64_t count, uint32_t slots, uint32_t L, int64_t *m,
                         uint32_t *n_overflow, hipStream_t s);
uint32_t pack_slots(int n_bits, uint64_t count);
hipError_t launch_mont_convert(int KP, const DKey &k, const uint32_t *in, uint64_t count,
                               uint32_t *out, bool to_mont, hipStream_t s);
// The pieces, for the autotuner: r mod P into tq; one private-key
// exponentiation of `kind` (4 mod P: tq in place, 0 lift, 3 both powers: tq into out, 2
// and 5 decryption: ciphertexts into out).
hipError_t launch_enc_r(int KP, const DKey &k, uint64_t count, const uint32_t *r, uint64_t seed, uint64_t roff,
                        uint32_t *tq, hipStream_t s);
hipError_t launch_pow_kind(int KP, const DKey &k, int kind, const uint32_t *in, uint32_t *out, uint64_t count,
                           uint32_t *tab, const PowPlan &p, hipStream_t s);
// xpq: [count][2][S_P2] (c^(P-1) mod P^2 as two digits base P).
hipError_t launch_dec(int KP, const DKey &k, const uint32_t *ct, uint64_t count,
                      uint32_t *xpq, int64_t *m, uint32_t *raw, uint32_t *n_overflow,
                      uint32_t *tab, const PowPlan &p, hipStream_t s);
// Launch shape of the histogram product kernel: grid, and dynamic LDS reserved
// only to cap its blocks per compute unit.
struct HistLaunch {
  uint32_t grid;
  uint32_t dyn;
};
uint32_t hist_resident_blocks(int KP, bool direct, uint32_t dyn);
uint32_t hist_dyn_lds(int KP, bool direct, int waves);
// pairs: how many of the resident ciphertext pairs (or of the jobs' samples)
// ws.pairs holds.
hipError_t launch_hist(int KP, const DKey &k, uint64_t pairs, const DJob *host_jobs, const HistWs &ws,
                       const HistLaunch &l, hipStream_t s);
hipError_t launch_fill(uint32_t *p, uint64_t n, uint32_t v, hipStream_t s);
hipError_t launch_probe_mul(uint64_t iters, uint32_t grid, uint32_t *sink, hipStream_t s);

// The exponentiations by kind -- 4 mod P and 0 (lift) of an encryption with secret
// digits, 3 (both powers at once) of the others, 2 (decryption) mod P^2 and 5
// the same with secret digits, 1 (public key) mod n^2 -- at G lanes per integer:
// whether that shape is built, its resident blocks with `dyn` bytes of dynamic
// LDS, and the dynamic LDS that caps it at `waves` blocks per compute unit (0:
// no cap).
inline int pow_lift_kind(const DKey &k) { return k.ct ? 0 : 3; }
inline int pow_dec_kind(const DKey &k) { return k.ct ? 5 : 2; }
bool pow_shape_valid(int KP, int kind, int G);
int device_cus();
uint32_t pow_resident_blocks(int KP, int kind, int G, uint32_t dyn);
uint32_t pow_dyn_lds(int KP, int kind, int G, int waves);
// Window-table scratch bytes per resident block.
uint64_t table_bytes_per_block(int KP, int kind, int G);

}  // namespace he
