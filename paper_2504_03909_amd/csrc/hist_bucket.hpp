// Index logic of the histogram bucketing kernels (counting sort of a node's
// samples by bin, per feature), shared by the gfx950 kernels and the CPU
// harness that checks it under AddressSanitizer.
//
// A node lists row indices of the resident ciphertext array; bins[f][row] is
// the bin of that row for feature f.  Both come from device memory the caller
// fills, so a row at or past the number of resident rows, or a bin at or past
// the job's bin count, must not index anything: such a sample is skipped by
// every kernel (the count, the scatter and therefore the products) and
// counted as bad.  The count and the scatter take the same decision for a
// sample, so every per-bin run of the permutation holds exactly the samples
// counted for it.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__)
#define HE_HD __host__ __device__
#else
#define HE_HD
#endif

namespace he {

// Row and bin of sample s of a node for one feature; false when the sample
// is skipped (row >= rows or bin >= n_bins).  `bins_f` is the feature's row
// of the bin table (at least `rows` entries); it is read only for a row
// below `rows`.
HE_HD inline bool bucket_sample(const uint32_t *idx, const uint8_t *bins_f, uint64_t rows, uint32_t n_bins,
                                uint64_t s, uint32_t &row, uint32_t &bin) {
  row = idx[s];
  if ((uint64_t)row >= rows) return false;
  bin = bins_f[row];
  return bin < n_bins;
}

// The job that entry x of a batch's flat arrays belongs to: the last one whose
// offset `off` (ascending over the jobs; a job without entries shares the next
// one's) is at most x.  A search by halves: job by job, a batch of 4,000 jobs spent
// 230 ms in the look-ups of its kernels.
template <class Job, class T>
HE_HD inline uint32_t find_job(const Job *jobs, uint32_t n_jobs, T Job::*off, uint64_t x) {
  uint32_t lo = 0, hi = n_jobs;
  while (hi - lo > 1) {
    const uint32_t mid = lo + (hi - lo) / 2;
    if (jobs[mid].*off <= x) lo = mid;
    else hi = mid;
  }
  return lo;
}

// Feature and sample range [s0, s1) of bucketing block `local` of a job with
// n samples and nblk blocks of `block` samples per feature.
HE_HD inline void bucket_block(uint64_t local, uint32_t nblk, uint64_t n, uint32_t block, uint32_t &f,
                               uint64_t &s0, uint64_t &s1) {
  f = (uint32_t)(local / nblk);
  s0 = (local % nblk) * block;
  s1 = s0 + block < n ? s0 + block : n;
}

// Ranks (within a feature, by decreasing bin count) that k_hist_final takes one
// per block, their partials in up to eight runs; higher ranks go one per wave, in
// two runs.
constexpr uint32_t kFinalSolo = 8;

// Most samples per item of a feature's bin of `cnt` samples, the rank-th fullest,
// in an untuned batch of items of up to `chunk`: longer items where the bin's
// partials would otherwise chain for longer than its items do.  With c samples per
// item these are c / 2 products in k_hist_chunk (two runs) and cnt / (8 c) or
// cnt / (2 c) in k_hist_final, which take half the time each, so 2 c beats c from cnt =
// 16 c^2 or 4 c^2 on.
HE_HD inline uint32_t item_chunk(uint32_t cnt, uint32_t rank, uint32_t chunk) {
  const uint64_t k = rank < kFinalSolo ? 16 : 4;
  uint64_t c = chunk;
  while (k * c * c < cnt) c *= 2;
  return (uint32_t)c;
}

// Slot of a sample in the feature's permutation row: the start of its bin's
// run reserved by its block (`block_base`, taken from the bin's cursor, which
// starts at the bin's offset) plus its rank among the block's samples of
// that bin.  Below offset + count of the bin when the count and the scatter
// skip the same samples.
HE_HD inline uint64_t bucket_slot(uint32_t block_base, uint32_t rank) { return (uint64_t)block_base + rank; }

}  // namespace he
