// Which batched attention a call of the draft layer takes, and the LDS of the one on the matrix cores.
#pragma once
#include "body_kernels.hpp"

namespace ddd {

constexpr int kSeqRows = 16;                 // most rows per sequence (k) of a workgroup that handles a whole sequence
constexpr int kMfThreads = 256;
constexpr int kMfLeast = 32;                 // shortest prompt (fewer keys leave most of the waves without a step of 32)
constexpr int kMfWaves = kMfThreads / 64;
constexpr int kMfOutPitch = kHeadDim + 4;    // floats of a row in a wave's outputs

struct MfLds {              // offsets in bytes, 16-byte aligned
  int spitch, ppitch;       // floats of a row of scores, bf16 of a row of weights
  size_t rsum, anc, ks, vs, aw, sct, ph, pl, total;
};
__host__ __device__ inline MfLds mf_lds(int L, int step) {
  MfLds m;
  m.spitch = ((L + 3) & ~3) + 4;
  m.ppitch = ((L + 31) & ~31) + 8;
  m.rsum = (size_t)kSeqRows * kHeadDim * 4;            // behind the rotated queries
  m.anc = m.rsum + kSeqRows * 4;
  m.ks = m.anc + kSeqRows * 32 * 4;
  m.vs = m.ks + kSeqRows * kHeadDim * 2;
  m.aw = m.vs + kSeqRows * kHeadDim * 2;               // [kSeqRows][step + 1] scores, then weights, past the prompt
  m.sct = (m.aw + (size_t)kSeqRows * (step + 1) * 4 + 15) & ~(size_t)15;
  m.ph = m.sct + (size_t)kSeqRows * m.spitch * 4;
  m.pl = m.ph + (size_t)kSeqRows * m.ppitch * 2;
  m.total = m.pl + (size_t)kSeqRows * m.ppitch * 2;
  const size_t outs = m.sct + (size_t)kMfWaves * kSeqRows * kMfOutPitch * 4;   // the waves' outputs take the place of sct, ph, pl
  if (outs > m.total) m.total = outs;
  return m;
}

// Scores and weights of the whole prompt sit in LDS: three workgroups share a CU up to 256 positions, two up to 480, one
// beyond.  151 KB holds prompts of 1024 positions in every call of a round and up to 1056 in its first three; longer ones (up to
// DDD_BODY_LMAX) leave the matrix cores.
constexpr int kMfLdsMost = 151 * 1024;
inline bool attention_on_matrix_cores(int R, int k, int L, int step) {
  return R > kBodyRows && k <= kSeqRows && L >= kMfLeast && mf_lds(L, step).total <= kMfLdsMost;
}

}  // namespace ddd
