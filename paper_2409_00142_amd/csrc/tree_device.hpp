// Final draft tree of one sequence, built by one workgroup (device functions shared by the
// stand-alone finalize kernels and the per-call bookkeeping kernels).
//
// Section 1: the m best nodes of the draft tree by summed logprob go to the target model in
// one pass; a node may attend to itself and its ancestors only.  Rerank key: (score desc,
// node id asc); tree order: ascending node id.
#pragma once
#include "ddd_device.hpp"
#include "ddd_kernels.hpp"

namespace ddd {

constexpr int kPoolMax = DDD_POOL_MAX;
constexpr int kTreeMax = DDD_MMAX + 1;
constexpr int kMaskWords = (kTreeMax + 31) / 32;

// Working set of the part that follows the selection (at most m + 1 nodes).
struct TreeEmitSmem {
  int pick[kTreeMax];                   // pool ids of the m_eff best nodes, any order
  int sel[kTreeMax];                    // pool ids of tree indices 0..m_eff (0 = root), ascending
  int par[kTreeMax];                    // tree index of the parent
  uint32_t bits[kTreeMax][kMaskWords];  // ancestor bit rows
};

struct TreeSmem {
  uint64_t keys[kPoolMax + 2];          // rerank keys of pool nodes 1..N (+ padding)
  TreeEmitSmem e;
};

__device__ __forceinline__ uint64_t rerank_key(float score, int node) {
  return ((uint64_t)ord32(score) << 32) | (uint32_t)(0xFFFFFFFFu - (uint32_t)node);
}

// From the m_eff chosen pool ids in sm.pick (any order, already visible to the block): order
// them by id, find parents, ancestor rows, and write the tree.  Every thread of the block calls it.
__device__ __forceinline__ void tree_emit_block(const ddd_state& st, const ddd_tree& tree, int b, int m, int m_eff,
                                                int nmax, int tid, int nthr, TreeEmitSmem& sm) {
  const int T = m + 1;
  const int32_t* ppar = st.pool_parent + (size_t)b * nmax;
  const int32_t* pdep = st.pool_depth + (size_t)b * nmax;
  const int32_t* ptok = st.pool_token + (size_t)b * nmax;
  // chosen ids in ascending order: rank by counting
  if (tid == 0) sm.sel[0] = 0;
  for (int i = tid; i < m_eff; i += nthr) {
    const int id = sm.pick[i];
    int rank = 0;
    for (int j = 0; j < m_eff; ++j) rank += (sm.pick[j] < id) ? 1 : 0;
    sm.sel[1 + rank] = id;
  }
  __syncthreads();
  // parents as tree indices (a parent has a smaller id, hence a smaller tree index); the node's
  // token and depth are requested in the same round trip as its parent's id and kept until the
  // tree is written (tree index tid; a block narrower than the tree takes the rest in a plain loop)
  const bool mine = tid <= m_eff;
  const int my_node = mine ? sm.sel[tid] : 0;
  const int my_pn = (mine && tid > 0) ? ppar[my_node] : -1;
  const int my_tok = mine ? ptok[my_node] : -1;
  const int my_dep = mine ? pdep[my_node] : 0;
  if (mine) {
    int par = -1;
    for (int j = 0; j < tid; ++j)
      if (sm.sel[j] == my_pn) par = j;
    sm.par[tid] = par;
  }
  for (int i = tid + nthr; i <= m_eff; i += nthr) {
    const int pn = ppar[sm.sel[i]];
    int par = -1;
    for (int j = 0; j < i; ++j)
      if (sm.sel[j] == pn) par = j;
    sm.par[i] = par;
  }
  __syncthreads();
  for (int i = tid; i < T; i += nthr) {
#pragma unroll
    for (int w = 0; w < kMaskWords; ++w) sm.bits[i][w] = 0u;
    if (i <= m_eff) {
      int c = i;
      while (c >= 0) {
        sm.bits[i][c >> 5] |= (1u << (c & 31));
        c = sm.par[c];
      }
    }
  }
  __syncthreads();
  if (tid == 0) tree.n_sel[b] = m_eff;
  for (int i = tid; i < m; i += nthr) tree.sel_node[(size_t)b * m + i] = (i < m_eff) ? sm.sel[1 + i] : -1;
  if (tid < T) {
    tree.tree_token[(size_t)b * T + tid] = my_tok;
    tree.pos[(size_t)b * T + tid] = my_dep;
    tree.parent_idx[(size_t)b * T + tid] = mine ? sm.par[tid] : -1;
  }
  for (int i = tid + nthr; i < T; i += nthr) {
    const bool ok = (i <= m_eff);
    const int node = ok ? sm.sel[i] : 0;
    tree.tree_token[(size_t)b * T + i] = ok ? ptok[node] : -1;
    tree.pos[(size_t)b * T + i] = ok ? pdep[node] : 0;
    tree.parent_idx[(size_t)b * T + i] = ok ? sm.par[i] : -1;
  }
  uint8_t* mask = tree.mask + (size_t)b * T * T;
  for (int e = tid; e < T * T; e += nthr) {
    const int i = e / T, j = e - i * T;
    mask[e] = (uint8_t)((sm.bits[i][j >> 5] >> (j & 31)) & 1u);
  }
}

// One compare-exchange of a bitonic network on keys in LDS: pair p of the stage with distance j
// inside sorted runs of length kk (descending overall).
__device__ __forceinline__ void bitonic_exchange(uint64_t* keys, int p, int j, int kk) {
  const int lo = ((p & ~(j - 1)) << 1) | (p & (j - 1)), hi = lo | j;
  const uint64_t x = keys[lo], y = keys[hi];
  const bool desc = (lo & kk) == 0;
  if ((x < y) == desc) {
    keys[lo] = y;
    keys[hi] = x;
  }
}

// Sorts keys[0 .. n2) (n2 a power of two >= 2) in descending order.  Every thread of the block
// calls it; nthr is a multiple of 64.  Pairs are dealt to the waves in blocks of 64 consecutive
// pairs; a stage with distance j <= 32 stays inside the 128 keys of such a block, so those stages
// need only the wave's own ordering, and only the stages with j >= 64 end in a block barrier.
__device__ __forceinline__ void bitonic_sort_desc(uint64_t* keys, int n2, int tid, int nthr) {
  const int lane = tid & 63, wave = tid >> 6, nwaves = nthr >> 6;
  const int npairs = n2 >> 1;
  for (int kk = 2; kk <= n2; kk <<= 1) {
    int j = kk >> 1;
    for (; j >= 64; j >>= 1) {
      for (int p = tid; p < npairs; p += nthr) bitonic_exchange(keys, p, j, kk);
      __syncthreads();
    }
    for (int pb = wave * 64; pb < npairs; pb += nwaves * 64) {
      const int p = pb + lane;
      for (int jj = j; jj >= 1; jj >>= 1) {
        if (p < npairs) bitonic_exchange(keys, p, jj, kk);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
    }
    if (kk >= 64) __syncthreads();     // the next run length starts with a stage across blocks
  }
  if (n2 < 128) __syncthreads();
}

// rank[i] = number of keys[0..n) larger than keys[i] (keys distinct, rank zeroed beforehand), by every thread of the block:
// with fewer keys than threads the comparisons of a key are shared by nthr / n threads.  No barrier inside.
__device__ __forceinline__ void count_larger_keys(const uint64_t* keys, int n, int* rank, int tid, int nthr) {
  if (n <= 0) return;                                            // uniform: nothing to rank (and nothing to divide by)
  if (n <= nthr) {                                               // uniform
    const int P = nthr / n, part = tid / n, i = tid - part * n;
    if (part < P) {
      const int chunk = ((n + P - 1) / P + 1) & ~1;              // even, so a pair never straddles two parts
      const int lo = part * chunk, hi = min(n, lo + chunk);
      const uint64_t mine = keys[i];
      int cnt = 0;
      for (int j = lo; j < hi; j += 2) {
        const uint64_t x = keys[j], y = (j + 1 < hi) ? keys[j + 1] : 0ull;
        cnt += (x > mine ? 1 : 0) + (y > mine ? 1 : 0);
      }
      if (cnt != 0) atomicAdd(&rank[i], cnt);
    }
  } else {
    for (int i = tid; i < n; i += nthr) {
      const uint64_t mine = keys[i];
      int cnt = 0;
      for (int j = 0; j < n; j += 2) {
        const uint64_t x = keys[j], y = (j + 1 < n) ? keys[j + 1] : 0ull;
        cnt += (x > mine ? 1 : 0) + (y > mine ? 1 : 0);
      }
      rank[i] = cnt;
    }
  }
}

// Sums over the lanes from this one up to lane 63.
__device__ __forceinline__ int suffix64_i32(int x, int lane) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x101, 0xf, 0xf, true);                  // row_shl:1, 2, 4, 8
  x += __builtin_amdgcn_update_dpp(0, x, 0x102, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x104, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x108, 0xf, 0xf, true);
  const int r1 = __builtin_amdgcn_readlane(x, 16), r2 = __builtin_amdgcn_readlane(x, 32), r3 = __builtin_amdgcn_readlane(x, 48);
  return x + (lane < 16 ? r1 + r2 + r3 : lane < 32 ? r2 + r3 : lane < 48 ? r3 : 0);
}

// The k-th largest of n values (1 <= k <= n <= kKthMost), ties counted: the smallest with fewer than k larger ones.  vals: LDS; red:
// LDS [1].
// By wave 0 alone; the block barriers also order the caller's writes of vals before and its reuse of them after.  Six bits at a time from
// the highest one in which any two values differ: the digits are counted in LDS, a lane looks after one of the 64, and the search ends at a
// prefix that exactly k values reach, after two or three passes.  (Bit by bit, a compare and a popcount per 64 values and bit: row reduction
// and beam update of a call of 100 beams 10.4 and 14.0 us, now 9.0 and 12.5; the row reduction of 170 rows 5.9, now 5.5; counting by the
// whole block, 32-bit compares against values that a wave reads from one address: 500 values 3.3 us on a CU.)
constexpr int kKthMost = 64 * 8;           // eight values per lane
template <int S>
__device__ __forceinline__ uint32_t wave_kth_largest(const uint32_t* vals, int n, int k, int lane) {
  __shared__ int hist[64];
  uint32_t key[S], lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
  for (int q = 0; q < S; ++q) {
    const bool real = 64 * q + lane < n;
    key[q] = real ? vals[64 * q + lane] : 0u;
    hi = umax32(hi, key[q]);
    lo = real ? min(lo, key[q]) : lo;
  }
  hi = wave_max_u32(hi);
  lo = ~wave_max_u32(~lo);
  if (hi == lo) return hi;                                        // uniform, as everything below
  int end = 32 - __clz((int)(hi ^ lo)), above = 0;                // bits below `end` are open; values beyond the prefix
  uint32_t T = end == 32 ? 0u : hi >> end << end;
  while (end > 0) {
    const int width = min(end, 6), shift = end - width;
    hist[lane] = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < S; ++q) {
      const uint32_t rest = (key[q] - T) >> shift;                // a value of the prefix has a digit here, one beyond it more
      if (64 * q + lane < n && key[q] >= T && (rest >> width) == 0u) atomicAdd(&hist[rest], 1);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int from = above + suffix64_i32(hist[lane], lane);      // values that reach this lane's digit: falling, lane 0 all
    const int d = 63 - __clzll((long long)__ballot(from >= k)), reach = __builtin_amdgcn_readlane(from, d);
    if (d < 63) above = __builtin_amdgcn_readlane(from, d + 1);
    T |= (uint32_t)d << shift;
    end = reach == k ? 0 : shift;
  }
  uint32_t least = 0xFFFFFFFFu;            // of the values at or above the prefix
#pragma unroll
  for (int q = 0; q < S; ++q) least = (64 * q + lane < n && key[q] >= T) ? min(least, key[q]) : least;
  return ~wave_max_u32(~least);
}
__device__ __forceinline__ uint32_t block_kth_largest_u32(const uint32_t* vals, int n, int k, uint32_t* red, int tid) {
  __syncthreads();
  if (tid < 64) {
    const uint32_t least = n <= 256 ? wave_kth_largest<4>(vals, n, k, tid) : wave_kth_largest<kKthMost / 64>(vals, n, k, tid);
    if (tid == 0) red[0] = least;
  }
  __syncthreads();
  return red[0];
}

// Orders LDS alone: global loads stay in flight.
__device__ __forceinline__ void tree_lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Inclusive prefix sums over the first 32 lanes.
__device__ __forceinline__ uint32_t scan32_u32(uint32_t x, int lane) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true);   // row_shr:1, 2, 4, 8 (0 comes in)
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true);
  const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)x, 15);
  return lane >= 16 ? x + first : x;
}
// By one wave: the tree indices of the `want` best of nodes 1 .. n (n <= 64 S, sc[h] the score of node 64 h + lane + 1), i.e. 1 + the number
// of taken nodes with a smaller id, to tidx, and their ids to sel.  The prefix is found bit by bit, a compare and a scalar popcount per 64
// nodes, and no further than one that exactly `want` reach; of equal scores the lowest ids are taken.
template <int S>
__device__ __forceinline__ void wave_take(const float* sc, int n, int want, int lane, int* tidx, int* sel) {
  uint32_t key[S], thr = 0u;
  bool real[S];
#pragma unroll
  for (int h = 0; h < S; ++h) {
    real[h] = 64 * h + lane < n;
    key[h] = real[h] ? ord32(sc[h]) : 0u;
  }
  if (want < n)                                                   // uniform
    for (uint32_t bit = 0x80000000u; bit != 0u; bit >>= 1) {
      const uint32_t cand = thr | bit;
      int cnt = 0;
#pragma unroll
      for (int h = 0; h < S; ++h) cnt += __popcll(__ballot(key[h] >= cand));
      if (cnt >= want) thr = cand;
      if (cnt == want) break;
    }
  int left = want;                                                // places for scores equal to thr
#pragma unroll
  for (int h = 0; h < S; ++h) left -= __popcll(__ballot(real[h] && key[h] > thr));
  const unsigned long long below = (1ull << lane) - 1ull;
  int over = 0, same = 0;                                         // of smaller ids
#pragma unroll
  for (int h = 0; h < S; ++h) {
    const unsigned long long gt = __ballot(real[h] && key[h] > thr), eq = __ballot(real[h] && key[h] == thr);
    const int o = over + __popcll(gt & below), e = same + __popcll(eq & below);
    const bool in = real[h] && (key[h] > thr || (key[h] == thr && e < left));
    const int t = 1 + o + min(e, left), id = 64 * h + lane + 1;
    if (real[h]) tidx[id] = in ? t : -1;
    if (in) sel[t] = id;
    over += __popcll(gt);
    same += __popcll(eq);
  }
}
// Pools of up to Q nodes per thread of the block: thread t looks after pool nodes t + 1, t + 1 + nthr, ... from their scores to their
// lines of the tree, so nothing is searched for and nothing is fetched twice.  One round trip brings the pool's size and every node's
// score, parent, token and depth.  Selection: the m-th largest score (ordered bits) is found six bits at a time by the whole block -
// the 64 digits are counted in LDS, one barrier, and every wave draws the same conclusion, lane d for the digit d - and no further than a
// prefix that exactly m nodes reach, three passes as a rule; of equal scores the lowest ids are taken.  FEW: pools of up to 256 nodes are
// left to one wave (wave_take; 37 nodes and m = 16 4.2 -> 3.6 us, 131 and m = 48 5.1 -> 4.2, 211 and m = 60 5.2 -> 5.0; a wave that selects
// for itself in every wave: 4.1, 4.9); not in the bookkeeping, of whose calls most make no tree: the code alone takes each call 0.15 us (ten
// calls with the tree of 911 nodes 7.87 and 7.69 us a call, three with one of 211 7.92 and 7.83).  The tree index of a selected node
// is 1 + the number of selected nodes with a smaller id (ballots, and the waves' totals through LDS).  A parent's tree index is read from
// the node -> index table (a selected node's parent is selected: its score is no smaller and its id is smaller).
// A launch is latency alone, and small code: behind a stream of weights its instructions come from memory.  ddd_tree_finalize of one
// sequence with 211 / 511 / 811 / 1809 / 3857 nodes, m = 60: 5.0 / 5.3 / 5.3 / 6.4 / 8.3 us on the GPU; with one wave that found the score bit
// by bit up to 1024 nodes, a ranking of candidates up to 2048 and a sort beyond 5.0 / 6.3 / 7.7 / 10.3 / 36.5.
constexpr int kTreeMost = kPoolMax;        // nodes of the largest pool
constexpr int kTreeFew = 256;              // nodes up to which one wave selects
constexpr int kTreeDigit = 6, kTreePasses = (32 + kTreeDigit - 1) / kTreeDigit;
template <int Q, bool FEW>
__device__ __forceinline__ void tree_select_block(const ddd_state& st, const ddd_tree& tree, int b, int m, int nmax,
                                                  int tid, int nthr, TreeSmem& sm, int n_nodes) {
  const int T = m + 1;
  int* tidx = reinterpret_cast<int*>(sm.keys);                    // [kTreeMost + 2]  tree index of a pool node; -1: not in the tree
  int* hist = tidx + kTreeMost + 2;                               // [kTreePasses][64] nodes per digit
  uint32_t* wtot = reinterpret_cast<uint32_t*>(hist + kTreePasses * 64);   // [Q][16]  a wave's larger (low half) and equal scores
  static_assert((kTreeMost + 2 + kTreePasses * 64 + Q * 16) * 4 <= (kPoolMax + 2) * 8, "working set");
  static_assert(Q == 2 || Q == 4, "totals are scanned 32 at a time");
  const int32_t* ppar = st.pool_parent + (size_t)b * nmax;
  const int32_t* pdep = st.pool_depth + (size_t)b * nmax;
  const int32_t* ptok = st.pool_token + (size_t)b * nmax;
  const float* psc = st.pool_score + (size_t)b * nmax;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwaves = nthr >> 6;
  int my_pn[Q], my_tok[Q], my_dep[Q], root_tok = -1, root_dep = 0;
  float my_sc[Q];
  const int most = (n_nodes >= 0 ? n_nodes : nmax) - 1;           // the pool's size, if the caller has it not at hand, in the same trip
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int n = tid + q * nthr;                                 // pool node n + 1
    my_sc[q] = 0.f;
    my_pn[q] = 0;
    my_tok[q] = -1;
    my_dep[q] = 0;
    if (n < most) {
      my_sc[q] = psc[n + 1];
      my_pn[q] = ppar[n + 1];
      my_tok[q] = ptok[n + 1];
      my_dep[q] = pdep[n + 1];
    }
  }
  const bool few = FEW && most <= kTreeFew;                     // uniform
  float few_sc[kTreeFew / 64] = {};
  if (few && wave == 0) {
#pragma unroll
    for (int h = 0; h < kTreeFew / 64; ++h)
      if (64 * h + lane < most) few_sc[h] = psc[64 * h + lane + 1];
  }
  if (tid == 0) {
    root_tok = ptok[0];
    root_dep = pdep[0];
  }
  const int N = (n_nodes >= 0 ? n_nodes : min(st.n_nodes[b], nmax)) - 1, m_eff = min(m, N);
  if (tid == 0) {
    tidx[0] = 0;
    sm.e.sel[0] = 0;
    sm.e.par[0] = -1;
  }
  uint32_t key[Q];
  bool real[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    real[q] = tid + q * nthr < N;
    key[q] = ord32(my_sc[q]);
  }
  int ti[Q];
  const unsigned long long below = (1ull << lane) - 1ull;
  if (few) {
    if (wave == 0) {
      if (most <= 128)                                            // uniform
        wave_take<2>(few_sc, N, m_eff, lane, tidx, sm.e.sel);
      else
        wave_take<4>(few_sc, N, m_eff, lane, tidx, sm.e.sel);
    }
  } else {
    for (int i = tid; i < kTreePasses * 64; i += nthr) hist[i] = 0;
    for (int i = tid; i < Q * 16; i += nthr) wtot[i] = 0u;          // of waves that are not there
    tree_lds_barrier();
    // ---- thr: the m_eff-th largest score, or a prefix that exactly m_eff reach ---------------------------------------
    uint32_t thr = 0u;
    if (m_eff < N) {                                                // uniform
      int above = 0;                                                // scores beyond the prefix
#pragma unroll 1
      for (int pass = 0; pass < kTreePasses; ++pass) {
        const int shift = max(32 - kTreeDigit * (pass + 1), 0);
        const uint32_t known = pass == 0 ? 0u : ~0u << (32 - kTreeDigit * pass);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
          const bool in = real[q] && ((key[q] ^ thr) & known) == 0u;
          const int digit = (int)((key[q] & ~known) >> shift);
          const unsigned long long who = __ballot(in);
          if (who == 0ull) continue;                                // wave-uniform
          // One addition for all lanes with the digit of the first: the scores' highest digits are alike, and additions to one address
          // wait for each other.  1809 nodes 7.5 -> 6.4 us, 511 5.45 -> 5.27; all scores equal 14.5 -> 7.5, 511 nodes 7.7 -> 6.1.
          const int first = __ffsll(who) - 1, common = __builtin_amdgcn_readlane(digit, first);
          const unsigned long long same = __ballot(in && digit == common);
          if (lane == first || (in && digit != common)) atomicAdd(&hist[pass * 64 + digit], lane == first ? (int)__popcll(same) : 1);
        }
        __syncthreads();
        const int from = above + suffix64_i32(hist[pass * 64 + lane], lane);   // scores that reach this lane's digit: falling, lane 0 all
        const int d = 63 - __clzll((long long)__ballot(from >= m_eff));
        const int reach = __builtin_amdgcn_readlane(from, d);
        if (d < 63) above = __builtin_amdgcn_readlane(from, d + 1);
        thr |= (uint32_t)d << shift;
        if (reach == m_eff) break;                                  // uniform
      }
    }
    // ---- tree indices --------------------------------------------------------------------------------------------------
    unsigned long long larger[Q], equal[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      larger[q] = __ballot(real[q] && key[q] > thr);
      equal[q] = __ballot(real[q] && key[q] == thr);
      if (lane == 0) wtot[q * 16 + wave] = (uint32_t)__popcll(larger[q]) | (uint32_t)__popcll(equal[q]) << 16;
    }
    __syncthreads();
    {
      uint32_t own[Q / 2], before[Q / 2], all = 0u;                 // totals of nodes with smaller ids
#pragma unroll
      for (int h = 0; h < Q / 2; ++h) {
        own[h] = lane < 32 ? wtot[h * 32 + lane] : 0u;
        const uint32_t incl = scan32_u32(own[h], lane);
        before[h] = all + incl - own[h];
        all += (uint32_t)__builtin_amdgcn_readlane((int)incl, 31);
      }
      const int left = m_eff - (int)(all & 0xFFFFu);                // places for scores equal to thr
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const uint32_t pre = (uint32_t)__builtin_amdgcn_readlane((int)before[q / 2], (q & 1) * 16 + wave);
        const int gt = (int)(pre & 0xFFFFu) + __popcll(larger[q] & below), eq = (int)(pre >> 16) + __popcll(equal[q] & below);
        const bool in = real[q] && (key[q] > thr || (key[q] == thr && eq < left));
        ti[q] = in ? 1 + gt + min(eq, left) : -1;
        if (real[q]) tidx[tid + q * nthr + 1] = ti[q];
        if (in) sm.e.sel[ti[q]] = tid + q * nthr + 1;
      }
    }
  }
  __syncthreads();
  if (few) {
#pragma unroll
    for (int q = 0; q < Q; ++q) ti[q] = real[q] ? tidx[tid + q * nthr + 1] : -1;
  }
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (ti[q] >= 0) {
      const int p = tidx[my_pn[q]];
      sm.e.par[ti[q]] = p < ti[q] ? p : -1;   // a pool whose parents do not come first must not send the walk below in a circle
    }
  __syncthreads();
  for (int i = tid; i < T; i += nthr) {                           // ancestor rows
    uint32_t w[kMaskWords] = {};
    for (int c = i <= m_eff ? i : -1; c >= 0; c = sm.e.par[c]) {
      const uint32_t bit = 1u << (c & 31);
#pragma unroll
      for (int x = 0; x < kMaskWords; ++x) w[x] |= (c >> 5) == x ? bit : 0u;
    }
#pragma unroll
    for (int x = 0; x < kMaskWords; ++x) sm.e.bits[i][x] = w[x];
  }
  if (tid == 0) {
    tree.n_sel[b] = m_eff;
    tree.tree_token[(size_t)b * T] = root_tok;
    tree.pos[(size_t)b * T] = root_dep;
    tree.parent_idx[(size_t)b * T] = -1;
  }
  for (int i = tid; i < m; i += nthr) tree.sel_node[(size_t)b * m + i] = (i < m_eff) ? sm.e.sel[1 + i] : -1;
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (ti[q] >= 0) {
      tree.tree_token[(size_t)b * T + ti[q]] = my_tok[q];
      tree.pos[(size_t)b * T + ti[q]] = my_dep[q];
      tree.parent_idx[(size_t)b * T + ti[q]] = sm.e.par[ti[q]];
    }
  for (int i = m_eff + 1 + tid; i < T; i += nthr) {     // padding
    tree.tree_token[(size_t)b * T + i] = -1;
    tree.pos[(size_t)b * T + i] = 0;
    tree.parent_idx[(size_t)b * T + i] = -1;
  }
  tree_lds_barrier();
  uint8_t* mask = tree.mask + (size_t)b * T * T;
  if (T <= 52) {                                                  // rows would leave lanes idle: 17 rows 0.2 us
    for (int e = tid; e < T * T; e += nthr) {
      const int i = e / T, j = e - i * T;
      mask[e] = (uint8_t)((sm.e.bits[i][j >> 5] >> (j & 31)) & 1u);
    }
  } else {
    for (int i = wave; i < T; i += nwaves)                        // a row per wave
      for (int j = lane; j < T; j += 64) mask[i * T + j] = (uint8_t)((sm.e.bits[i][j >> 5] >> (j & 31)) & 1u);
  }
}

// The final tree of a pool of at most DDD_POOL_MAX nodes.  Must be called by every thread of the block, at most 1024.
// n_nodes: the sequence's pool size (st.n_nodes[b]) if the caller has it at hand, else -1.
// QMOST = 4: the block has a thread for every four nodes.  QMOST = 2: a block of 64 k threads inside the bookkeeping, where pools beyond two
// nodes a thread (k = 16 from nine calls on, k = 10 from fourteen) have their rerank keys sorted in LDS (they are distinct: the id is part of
// the key).
template <int QMOST>
__device__ __forceinline__ void tree_finalize_block(const ddd_state& st, const ddd_tree& tree, int b, int m, int nmax,
                                                    int tid, int nthr, TreeSmem& sm, int n_nodes = -1) {
  static_assert(QMOST == 2 || QMOST == 4, "nodes per thread");
  if (n_nodes < 0 && nmax - 1 > 2 * nthr) n_nodes = min(st.n_nodes[b], nmax);
  const int most = (n_nodes >= 0 ? n_nodes : nmax) - 1;
  if (most <= 2 * nthr) {                                         // uniform
    tree_select_block<2, QMOST == 4>(st, tree, b, m, nmax, tid, nthr, sm, n_nodes);
  } else if constexpr (QMOST == 4) {
    tree_select_block<4, false>(st, tree, b, m, nmax, tid, nthr, sm, n_nodes);
  } else {
    const int N = most, m_eff = min(m, N);
    const float* psc = st.pool_score + (size_t)b * nmax;
    int n2 = 2;
    while (n2 < N) n2 <<= 1;
    for (int i = tid; i < n2; i += nthr) sm.keys[i] = (i < N) ? rerank_key(psc[i + 1], i + 1) : 0ull;   // 0: below every key
    __syncthreads();
    bitonic_sort_desc(sm.keys, n2, tid, nthr);
    for (int i = tid; i < m_eff; i += nthr) sm.e.pick[i] = (int)(0xFFFFFFFFu - (uint32_t)sm.keys[i]);
    __syncthreads();
    tree_emit_block(st, tree, b, m, m_eff, nmax, tid, nthr, sm.e);
  }
}

}  // namespace ddd
