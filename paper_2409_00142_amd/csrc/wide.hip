// Wide beams (DDD_KMAX < k <= DDD_KWIDE_MAX): beam update, stop test and final tree of one
// sequence by one workgroup (Appendix, Table 2: draft speed against beam width).
//
// With up to 128 x 128 candidates per draft call and tens of thousands of pool nodes one workgroup must not do what many
// can: inside a draft call the candidates' pool entries and beam keys (score desc, token asc, flat index asc) are written
// by the row reduction, one workgroup per row, and this launch only reads the keys, sixteen per thread.  The beam: a lower
// bound from the rows' first few candidates, the keys above it ranked by counting; many equal scores: a radix select
// (8-bit digits from the top: histogram in LDS, the digit holding the wanted rank narrows the prefix).  The final rerank
// selects the m best pool nodes the same way from the scores in global memory.  At k = 100, V = 32000, B = 1: 31 -> 16 us
// a call, 73 -> 32 us for the call that builds the final tree (with the candidates formed here and the 64-bit radix
// select and counting over 512 keys), 14 and 28 with the bound found by one wave, the sample taken from the rows' keys and
// the keys requested before the sequence's flag is known.  Everything else (Eq. 1 in fp64 in index order, parents, ancestor rows, mask) is as
// for narrow beams.
#include "bookkeep_device.hpp"
#include "tree_device.hpp"

namespace ddd {

constexpr int kKW = DDD_KWIDE_MAX;
constexpr int kWideThreads = 1024;
constexpr int kGlobalChunk = 8;                    // loads in flight per thread when the keys come from global memory
// final tree of a large pool: sample, candidates and their ranks (tree_finalize_wide_block)
constexpr int kWSub = 512, kWCand = 1024;
constexpr int kBeamSample = 320;                   // most candidates that bound a new beam
constexpr int kWideWorkBytes = kWSub * 8 + kWCand * 8 + kWCand * 4;
static_assert(kWSub >= DDD_MMAX && kWSub <= kWCand, "the sample holds m keys and lies in the candidate list");
static_assert(kBeamSample >= kKW && kBeamSample <= kKthMost && kBeamSample <= kWSub, "one of each row at least, ranked by one wave");
// LDS in front of WideSmem in the step kernel: the k*k candidate keys of a call, later the work area of the final tree
__host__ __device__ inline size_t wide_front_bytes(int k) {
  const size_t keys = ((size_t)k * k * 8 + 15) & ~(size_t)15;
  return keys > (size_t)kWideWorkBytes ? keys : (size_t)kWideWorkBytes;
}

struct WideSmem {
  unsigned hist[256];
  int digit, rem, alone, cnt, stopped;
  unsigned or_lo, or_hi, and_lo, and_hi, found_lo, found_hi;
  float lps_old[kKW];
  int node_old[kKW];
  uint64_t sel[kKW];
  uint32_t red[1];
  TreeEmitSmem te;
};

// One count for this lane's digit into the histogram.  Scores cluster (a handful of exponents), so
// most lanes of a wave often hit the same bin, which an LDS atomic serialises lane by lane: up to
// eight distinct digits per wave are therefore counted with a ballot and added once by a leader
// (`clustered`: the first digit examined, where the keys still share their leading bits); whatever
// is left, and every later digit, goes through plain atomics (spread digits rarely collide).
__device__ __forceinline__ void hist_add(unsigned* hist, unsigned digit, bool valid, int lane, bool clustered) {
  unsigned long long remaining = __ballot(valid);
  for (int it = 0; clustered && it < 8 && remaining != 0ull; ++it) {
    const int leader = __ffsll((long long)remaining) - 1;
    const unsigned d = (unsigned)__shfl((int)digit, leader, 64);
    const unsigned long long same = __ballot(valid && digit == d) & remaining;
    if (lane == leader) atomicAdd(&hist[d], (unsigned)__popcll(same));
    remaining &= ~same;
  }
  if ((remaining >> lane) & 1ull) atomicAdd(&hist[digit], 1u);
}

// The key of rank `want` (0-based, descending) among n distinct keys key_of(0..n-1), n > want.
// Every thread of the block calls it with the same arguments; the result is uniform.
// Radix select, 8-bit digits from the top; the bytes above the first one in which any two keys
// differ are skipped, and the search ends as soon as the wanted key is alone in its bin.
// One pass over keys 0..n-1 by the whole block (1024 threads): element i = tid + j * 1024.  CH
// keys are fetched before any is used, so a pass over keys that come from global memory pays one
// memory latency per CH elements.  fn(key, in) is called for every slot of a chunk that holds
// at least one element, by all threads (in == false past the end): it may use wave-wide operations.
template <int CH, class KeyFn, class Fn>
__device__ __forceinline__ void sweep_keys(int n, int tid, KeyFn key_of, Fn fn) {
  for (int j0 = 0; j0 * kWideThreads < n; j0 += CH) {
    uint64_t kk[CH];
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int i = tid + (j0 + u) * kWideThreads;
      kk[u] = (i < n) ? key_of(i) : 0ull;
    }
#pragma unroll
    for (int u = 0; u < CH; ++u) {
      const int i0 = (j0 + u) * kWideThreads;
      if (i0 < n) fn(kk[u], tid + i0 < n);
    }
  }
}

// The key of rank `want` (0-based, descending) among the n distinct keys key_of(0..n-1), n > want.
// Every thread of the block calls it with the same arguments; the result is uniform.  Radix
// select, 8-bit digits from the top; the bytes above the first one in which any two keys differ
// are skipped, and the search ends as soon as the wanted key is alone in its bin.
template <int CH, class KeyFn>
__device__ __forceinline__ uint64_t block_select_kth(int n, int want, KeyFn key_of, WideSmem& sm, int tid) {
  const int lane = tid & 63;
  // bits in which the keys differ: OR of all keys against AND of all keys
  uint64_t vor = 0ull, vand = ~0ull;
  sweep_keys<CH>(n, tid, key_of, [&](uint64_t key, bool in) {
    if (in) {
      vor |= key;
      vand &= key;
    }
  });
  uint32_t olo = (uint32_t)vor, ohi = (uint32_t)(vor >> 32), alo = (uint32_t)vand, ahi = (uint32_t)(vand >> 32);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    olo |= (uint32_t)__shfl_xor((int)olo, off, 64);
    ohi |= (uint32_t)__shfl_xor((int)ohi, off, 64);
    alo &= (uint32_t)__shfl_xor((int)alo, off, 64);
    ahi &= (uint32_t)__shfl_xor((int)ahi, off, 64);
  }
  if (tid == 0) {
    sm.or_lo = 0u;
    sm.or_hi = 0u;
    sm.and_lo = ~0u;
    sm.and_hi = ~0u;
  }
  __syncthreads();
  if (lane == 0) {
    atomicOr(&sm.or_lo, olo);
    atomicOr(&sm.or_hi, ohi);
    atomicAnd(&sm.and_lo, alo);
    atomicAnd(&sm.and_hi, ahi);
  }
  __syncthreads();
  const uint64_t all_or = ((uint64_t)sm.or_hi << 32) | sm.or_lo, all_and = ((uint64_t)sm.and_hi << 32) | sm.and_lo;
  const uint64_t diff = all_or ^ all_and;
  if (diff == 0ull) return all_or;                    // a single key
  const int top_byte = (63 - __clzll((long long)diff)) >> 3;
  uint64_t prefix = (top_byte == 7) ? 0ull : (all_and & (~0ull << (8 * (top_byte + 1))));
  int rem = want;
  for (int shift = 8 * top_byte; shift >= 0; shift -= 8) {
    for (int i = tid; i < 256; i += kWideThreads) sm.hist[i] = 0u;
    __syncthreads();
    const uint64_t hi_mask = (shift == 56) ? 0ull : (~0ull << (shift + 8));
    sweep_keys<CH>(n, tid, key_of, [&](uint64_t key, bool in) {
      hist_add(sm.hist, (unsigned)(key >> shift) & 255u, in && (key & hi_mask) == prefix, lane, shift == 8 * top_byte);
    });
    __syncthreads();
    if (tid < 64) {   // wave 0: lane l owns digits 255-4l .. 252-4l; running count from the top digit down
      unsigned h[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) h[q] = sm.hist[255 - 4 * lane - q];
      const unsigned s = h[0] + h[1] + h[2] + h[3];
      unsigned incl = s;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const unsigned t = __shfl_up(incl, off, 64);
        if (lane >= off) incl += t;
      }
      const unsigned excl = incl - s;
      if ((unsigned)rem >= excl && (unsigned)rem < incl) {   // exactly one lane
        unsigned c = excl;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if ((unsigned)rem >= c && (unsigned)rem < c + h[q]) {
            sm.digit = 255 - 4 * lane - q;
            sm.rem = (int)((unsigned)rem - c);
            sm.alone = (h[q] == 1u) ? 1 : 0;
          }
          c += h[q];
        }
      }
    }
    __syncthreads();
    prefix |= (uint64_t)(unsigned)sm.digit << shift;
    rem = sm.rem;
    if (sm.alone && shift > 0) {                      // uniform: the wanted key is the only one with this prefix
      const uint64_t pm = ~0ull << shift;
      sweep_keys<CH>(n, tid, key_of, [&](uint64_t key, bool in) {
        if (in && (key & pm) == prefix) {
          sm.found_lo = (uint32_t)key;
          sm.found_hi = (uint32_t)(key >> 32);
        }
      });
      __syncthreads();
      return ((uint64_t)sm.found_hi << 32) | sm.found_lo;
    }
  }
  return prefix;
}

// Descending bitonic sort of sm.sel[0..127] (unused slots hold 0) by one wave (all 64 lanes): each
// stage is one compare-exchange per lane, ordered by wave barriers instead of block barriers.
__device__ __forceinline__ void sort_sel_desc_wave(WideSmem& sm, int lane) {
  for (int size = 2; size <= kKW; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      const int pos = 2 * stride * (lane / stride) + (lane % stride);
      const int partner = pos + stride;
      const bool desc = ((pos & size) == 0);
      const uint64_t x = sm.sel[pos], y = sm.sel[partner];
      if ((x < y) == desc) {
        sm.sel[pos] = y;
        sm.sel[partner] = x;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
}

// Final tree for a pool of any size.  The m best rerank keys are found as for narrow beams (tree_device.hpp): the m-th
// best score of the first 256 nodes is a lower bound of the tree's scores (summed logprobs fall with depth), one sweep over
// the pool collects the nodes at or above it (up to kWCand), and they are ranked by counting.  If more pass the bound, the
// same with whole keys, the first kWSub nodes and then kWSub of the candidates as the sample (three attempts); after that the
// radix select takes over.  work: kWideWorkBytes of LDS.
__device__ __forceinline__ void tree_finalize_wide_block(const ddd_state& st, const ddd_tree& tree, int b, int m, int nmax,
                                                         int tid, int nthr, WideSmem& sm, unsigned char* work) {
  const int N = st.n_nodes[b] - 1;
  const int m_eff = min(m, N);
  const float* psc = st.pool_score + (size_t)b * nmax;
  auto key_of = [&](int i) { return rerank_key(psc[i + 1], i + 1); };
  uint64_t* sample = reinterpret_cast<uint64_t*>(work);            // [kWSub]
  uint64_t* cand = sample + kWSub;                                   // [kWCand]
  int* rank = reinterpret_cast<int*>(cand + kWCand);                // [kWCand]
  bool ranked = false;
  // First with 32-bit scores: the m-th best of the first 256 nodes, and one plain sweep over the scores.
  if (m_eff < N && nthr == kWideThreads) {                           // uniform
    constexpr int kFirst = 256;
    static_assert(kFirst >= DDD_MMAX && kFirst <= kKthMost && kFirst <= 2 * kWSub, "the sample holds m scores and lies in front of the candidates");
    uint32_t* first = reinterpret_cast<uint32_t*>(work);             // [kFirst]
    const int n_first = min(N, kFirst);
    for (int i = tid; i < n_first; i += nthr) first[i] = ord32(psc[i + 1]);
    for (int i = tid; i < kWCand; i += nthr) rank[i] = 0;
    if (tid == 0) sm.cnt = 0;
    __syncthreads();
    // Compared as ordered bits, a total order: at least the m_eff scores of the sample that made the bound pass it, whatever
    // they are (a NaN, from a row whose largest logit is infinite, would fail every comparison of floats).
    const uint32_t bound = block_kth_largest_u32(first, n_first, m_eff, sm.red, tid);
    constexpr int kSweep = 16;
    for (int i0 = tid; i0 < N; i0 += kSweep * kWideThreads) {
      float x[kSweep];
#pragma unroll
      for (int u = 0; u < kSweep; ++u) x[u] = psc[min(i0 + u * kWideThreads, N - 1) + 1];   // no branch: all in flight
#pragma unroll
      for (int u = 0; u < kSweep; ++u)
        if (ord32(x[u]) >= bound && i0 + u * kWideThreads < N) {
          const int p = atomicAdd(&sm.cnt, 1);
          if (p < kWCand) cand[p] = rerank_key(x[u], i0 + u * kWideThreads + 1);
        }
    }
    __syncthreads();
    const int C = sm.cnt;
    if (__builtin_expect(C <= kWCand, 1)) {                          // uniform
      count_larger_keys(cand, C, rank, tid, nthr);
      __syncthreads();
      for (int c = tid; c < C; c += nthr)
        if (rank[c] < m_eff) sm.te.pick[rank[c]] = (int)(0xFFFFFFFFu - (uint32_t)cand[c]);
      ranked = true;
    }
    __syncthreads();
  }
  if (__builtin_expect(!ranked && m_eff < N && nthr == kWideThreads, 0)) {      // uniform
    int n_sample = min(N, kWSub);
    for (int i = tid; i < n_sample; i += nthr) sample[i] = key_of(i);
    for (int attempt = 0; attempt < 3; ++attempt) {
      for (int i = tid; i < kWCand; i += nthr) rank[i] = 0;
      if (tid == 0) sm.cnt = 0;
      __syncthreads();
      count_larger_keys(sample, n_sample, rank, tid, nthr);
      __syncthreads();
      for (int i = tid; i < n_sample; i += nthr)
        if (rank[i] == min(m_eff, n_sample) - 1) {                   // exactly one key has this rank
          sm.found_lo = (uint32_t)sample[i];
          sm.found_hi = (uint32_t)(sample[i] >> 32);
        }
      __syncthreads();
      const uint64_t bound = ((uint64_t)sm.found_hi << 32) | sm.found_lo;
      sweep_keys<kGlobalChunk>(N, tid, key_of, [&](uint64_t key, bool in) {
        if (in && key >= bound) {
          const int p = atomicAdd(&sm.cnt, 1);
          if (p < kWCand) cand[p] = key;
        }
      });
      __syncthreads();
      const int C = sm.cnt;
      if (C <= kWCand) {                                             // uniform
        for (int i = tid; i < kWCand; i += nthr) rank[i] = 0;
        __syncthreads();
        count_larger_keys(cand, C, rank, tid, nthr);
        __syncthreads();
        for (int c = tid; c < C; c += nthr)
          if (rank[c] < m_eff) sm.te.pick[rank[c]] = (int)(0xFFFFFFFFu - (uint32_t)cand[c]);
        ranked = true;
        break;
      }
      for (int i = tid; i < kWSub; i += nthr) sample[i] = cand[i];  // the first kWSub candidates: all above the old bound
      n_sample = kWSub;
      __syncthreads();
    }
  }
  if (__builtin_expect(!ranked, 0)) {
    uint64_t kth = 0ull;                       // every key is at least 1
    if (m_eff < N) kth = block_select_kth<kGlobalChunk>(N, m_eff - 1, key_of, sm, tid);
    if (tid == 0) sm.cnt = 0;
    __syncthreads();
    sweep_keys<kGlobalChunk>(N, tid, key_of, [&](uint64_t key, bool in) {
      if (in && key >= kth) {
        const int p = atomicAdd(&sm.cnt, 1);
        if (p < kTreeMax) sm.te.pick[p] = (int)(0xFFFFFFFFu - (uint32_t)key);   // exactly m_eff: keys are distinct
      }
    });
  }
  __syncthreads();
  tree_emit_block(st, tree, b, m, m_eff, nmax, tid, nthr, sm.te);
}

// One draft call of one sequence by one workgroup; returns whether the sequence is still active after it
// (the same value in every thread; true when no stop test is asked for).
// KEYS: the row reduction has formed the candidates' beam keys (a call of a round, which also selects and tests).
template <bool KEYS>
__device__ __forceinline__ bool step_wide_block(const WideStepArgs& a, unsigned char* wsm_raw) {
  const BeamArgs& g = a.beam;
  const int b = blockIdx.x, tid = threadIdx.x, nthr = blockDim.x;
  const int k = g.k, step = g.step;
  WideSmem& sm = *reinterpret_cast<WideSmem*>(wsm_raw + wide_front_bytes(k));
  constexpr bool from_keys = KEYS;
  const bool do_select = KEYS || a.do_select, do_stop = KEYS || a.do_stop;
  const size_t row0 = (step == 0) ? (size_t)b : (size_t)b * k;
  // The candidates' beam keys that the row reduction has formed, element f = tid + u * 1024, and the rows' first few of them (below):
  // on their way before the sequence's flag is looked at.
  constexpr int kPer = kKW * kKW / kWideThreads;
  uint64_t kv[kPer], mine = 0ull;
  uint32_t* sample = reinterpret_cast<uint32_t*>(wsm_raw);       // [kWSub]
  const int per_row = min(k, max(1, kBeamSample / k)), n_sample = k * per_row;
  const int on_flag = g.st.active[b];
  if (do_select && step > 0 && from_keys) {                    // uniform
    const int i = tid / per_row;                                 // n_sample <= kBeamSample
    if (tid < n_sample) mine = a.part_key[row0 * k + i * k + (tid - i * per_row)];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int f = u * kWideThreads + tid;
      kv[u] = (f < k * k) ? a.part_key[row0 * k + f] : 0ull;
    }
  }
  if (!on_flag) return false;                // uniform over the workgroup

  float* lps = g.st.logprobsum + (size_t)b * k;
  int32_t* bnode = g.st.beam_node + (size_t)b * k;
  int32_t* btok = g.st.beam_token + (size_t)b * k;
  int32_t* bslot = g.st.beam_parent_slot + (size_t)b * k;
  int32_t* ptok = g.st.pool_token + (size_t)b * g.nmax;
  int32_t* ppar = g.st.pool_parent + (size_t)b * g.nmax;
  int32_t* pdep = g.st.pool_depth + (size_t)b * g.nmax;
  float* psc = g.st.pool_score + (size_t)b * g.nmax;
  int steps_done = a.steps_done;

  if (do_select) {
    steps_done = step + 1;
    if (step == 0) {
      // the prompt call: nodes 1..k in rank order are the first beam
      for (int j = tid; j < k; j += nthr) {
        int t;
        float s;
        if (from_keys) {
          const uint64_t key = a.part_key[row0 * k + j];
          t = key_token(key);
          s = key_value(key) - a.part_lse[row0];
        } else {
          t = g.topk_token[row0 * k + j];
          s = g.topk_logprob[row0 * k + j];
        }
        const int nid = 1 + j;
        ptok[nid] = t;
        ppar[nid] = 0;
        pdep[nid] = 1;
        psc[nid] = s;
        bnode[j] = nid;
        btok[j] = t;
        bslot[j] = 0;
        lps[j] = s;
      }
      if (tid == 0) {
        g.st.n_nodes[b] = 1 + k;
        g.st.steps[b] = 1;
        if (a.lse_dbg != nullptr && from_keys) a.lse_dbg[row0] = a.part_lse[row0];
      }
    } else {
      const int base = 1 + k + (step - 1) * k * k, kk = k * k;
      if (a.lse_dbg != nullptr && from_keys)
        for (int i = tid; i < k; i += nthr) a.lse_dbg[row0 + i] = a.part_lse[row0 + i];
      // every candidate's beam key: formed by the row reduction, or here from the caller's rows
      if (from_keys) {
        if (tid < n_sample) sample[tid] = (uint32_t)(mine >> 32);
      } else {
        for (int i = tid; i < k; i += nthr) {
          sm.lps_old[i] = lps[i];
          sm.node_old[i] = bnode[i];
        }
        __syncthreads();
#pragma unroll
        for (int u0 = 0; u0 < kPer; u0 += 4) {            // four candidates per thread in flight
          int t[4];
          float lp[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int f = (u0 + u) * kWideThreads + tid;
            t[u] = (f < kk) ? g.topk_token[row0 * k + f] : 0;
            lp[u] = (f < kk) ? g.topk_logprob[row0 * k + f] : 0.f;
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int f = (u0 + u) * kWideThreads + tid;
            kv[u0 + u] = 0ull;
            if (f < kk) {
              const int i = f / k;
              const float sc = __fadd_rn(sm.lps_old[i], lp[u]);
              ptok[base + f] = t[u];
              ppar[base + f] = sm.node_old[i];
              pdep[base + f] = step + 1;
              psc[base + f] = sc;
              kv[u0 + u] = wide_beam_key(sc, t[u], f);
              if (f - i * k < per_row) sample[i * per_row + f - i * k] = (uint32_t)(kv[u0 + u] >> 32);
            }
          }
        }
      }
      // The new beam: the k-th best score of the rows' first few candidates is a lower bound of the beam's scores (a row's
      // logprobs fall), the keys at or above it - k and a few more - are ranked by counting.  Three per row at k = 100: a
      // size chosen when the bound was found by comparing all pairs, and not tuned again for the one wave that finds it now.
      uint64_t* cand = reinterpret_cast<uint64_t*>(sample + 2 * kWSub); // [kWCand]
      int* rank = reinterpret_cast<int*>(cand + kWCand);         // [kWCand]
      for (int i = tid; i < kWCand; i += nthr) rank[i] = 0;
      if (tid == 0) sm.cnt = 0;
      __syncthreads();
      const uint32_t bound = block_kth_largest_u32(sample, n_sample, k, sm.red, tid);
      auto passes = [&](int u) { return kv[u] != 0ull && (uint32_t)(kv[u] >> 32) >= bound; };
      int at = 0;                                                 // of this wave's candidates: one look at the counter
#pragma unroll
      for (int u = 0; u < kPer; ++u) at += __popcll(__ballot(passes(u)));
      if ((tid & 63) == 0 && at != 0) at = atomicAdd(&sm.cnt, at);
      at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const bool in = passes(u);
        const unsigned long long bal = __ballot(in);
        const int p = at + __popcll(bal & ((1ull << (tid & 63)) - 1ull));
        if (in && p < kWCand) cand[p] = kv[u];
        at += __popcll(bal);
      }
      __syncthreads();
      const int C = sm.cnt;
      if (__builtin_expect(C <= kWCand, 1)) {                     // uniform
        count_larger_keys(cand, C, rank, tid, nthr);
        __syncthreads();
        for (int i = tid; i < C; i += nthr)
          if (rank[i] < k) sm.sel[rank[i]] = cand[i];
      } else {
        // many equal or nearly equal scores: radix select over all keys
        __syncthreads();                                          // everybody has the count; the keys take the work area's place
        uint64_t* keys = reinterpret_cast<uint64_t*>(wsm_raw);
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
          const int f = u * kWideThreads + tid;
          if (f < kk) keys[f] = kv[u];
        }
        __syncthreads();
        const uint64_t kth = block_select_kth<8>(kk, k - 1, [&](int i) { return keys[i]; }, sm, tid);
        for (int i = tid; i < kKW; i += nthr) sm.sel[i] = 0ull;
        if (tid == 0) sm.cnt = 0;
        __syncthreads();
        for (int f = tid; f < kk; f += nthr)
          if (keys[f] >= kth) {
            const int p = atomicAdd(&sm.cnt, 1);
            if (p < kKW) sm.sel[p] = keys[f];     // exactly k of them: keys are distinct
          }
        __syncthreads();
        if (tid < 64) sort_sel_desc_wave(sm, tid);
      }
      __syncthreads();
      for (int r = tid; r < k; r += nthr) {
        const uint64_t key = sm.sel[r];
        const int f = wide_key_flat(key);
        bnode[r] = base + f;
        btok[r] = wide_key_token(key);
        bslot[r] = f / k;
        lps[r] = key_value(key);
      }
      if (tid == 0) {
        g.st.n_nodes[b] = base + k * k;
        g.st.steps[b] = step + 1;
      }
    }
    __syncthreads();   // the new beam is visible to the block
  }

  if (tid == 0) sm.stopped = 0;
  if (do_stop) {
    if (tid < 64) {                              // wave 0: lane l holds beam slots l and l + 64
      const double e0 = (tid < k) ? exp((double)lps[tid]) : 0.0, e1 = (tid + 64 < k) ? exp((double)lps[tid + 64]) : 0.0;
      const uint64_t b0 = (uint64_t)__double_as_longlong(e0), b1 = (uint64_t)__double_as_longlong(e1);
      double P = 0.0;
      auto add8 = [&](uint64_t bits, int i0) {   // slots i0 .. i0 + 7 of 64 (those past k hold 0)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)bits, i0 + i);
          const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(bits >> 32), i0 + i);
          P += __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
        }
      };
      for (int i = 0; i < min(k, 64); i += 8) add8(b0, i);        // index order
      for (int i = 0; i < k - 64; i += 8) add8(b1, i);
      bool cont = steps_done < g.D;
      if (cont && ((g.check_mask >> steps_done) & 1u) && P < (double)g.threshold) cont = false;
      if (tid == 0) {
        g.st.conf[b] = P;
        g.st.active[b] = cont ? 1 : 0;
        sm.stopped = cont ? 0 : 1;
      }
    }
    __syncthreads();
    const uint8_t on = sm.stopped ? 0 : 1;
    for (int i = tid; i < k; i += nthr) g.st.row_active[(size_t)b * k + i] = on;
  }
  __syncthreads();   // also orders the pool writes before the reads below
  const bool stopped = sm.stopped != 0;
  if (__builtin_expect(a.tree.mask != nullptr && stopped, 0))   // the candidate keys of the beam update are no longer needed: their LDS is the work area
    tree_finalize_wide_block(g.st, a.tree, b, a.m, g.nmax, tid, nthr, sm, wsm_raw);
  return !stopped;
}

template <bool KEYS>
__global__ __launch_bounds__(kWideThreads) void step_wide_kernel(WideStepArgs a) {
  extern __shared__ __align__(16) unsigned char wsm_raw[];
  const bool active = step_wide_block<KEYS>(a, wsm_raw);
  report_call(a.report, active, blockIdx.x, a.beam.k, threadIdx.x, blockDim.x);
}

__global__ __launch_bounds__(kWideThreads) void tree_finalize_wide_kernel(FinalizeArgs a) {
  __shared__ WideSmem sm;
  __shared__ __align__(16) unsigned char work[kWideWorkBytes];
  tree_finalize_wide_block(a.st, a.tree, blockIdx.x, a.m, a.nmax, threadIdx.x, blockDim.x, sm, work);
}

static size_t wide_lds_bytes(int k) { return wide_front_bytes(k) + sizeof(WideSmem); }

hipError_t prepare_wide() {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&step_wide_kernel<true>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)wide_lds_bytes(kKW));
  if (e == hipSuccess)
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&step_wide_kernel<false>), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)wide_lds_bytes(kKW));
  return e;
}

hipError_t launch_step_wide(const WideStepArgs& a, hipStream_t stream) {
  if (a.part_key != nullptr && a.do_select && a.do_stop)
    hipLaunchKernelGGL(step_wide_kernel<true>, dim3(a.beam.B), dim3(kWideThreads), wide_lds_bytes(a.beam.k), stream, a);
  else
    hipLaunchKernelGGL(step_wide_kernel<false>, dim3(a.beam.B), dim3(kWideThreads), wide_lds_bytes(a.beam.k), stream, a);
  return hipGetLastError();
}

hipError_t launch_tree_finalize_wide(const FinalizeArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL(tree_finalize_wide_kernel, dim3(a.B), dim3(kWideThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace ddd
