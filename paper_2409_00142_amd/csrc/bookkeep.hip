// Stand-alone kernels of the per-call bookkeeping (device code in bookkeep_device.hpp) and the
// row reduction of materialised logits.
#include "bookkeep_device.hpp"

namespace ddd {

// ---- standalone merge: one wave per row ------------------------------------------------------
__global__ __launch_bounds__(256) void merge_kernel(MergeArgs a) {
  __shared__ uint64_t s_mrg[4][kMergeWords];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + wave;
  if (row >= a.n_rows) return;                                 // wave-uniform
  if (a.row_active != nullptr && !a.row_active[row]) return;   // wave-uniform
  uint64_t key;
  float lse;
  {
    RowHeads heads;
    const uint64_t* pk = a.part_key + (size_t)row * a.nslice * a.k;
    merge_load_heads(pk, a.part_sum + (size_t)row * a.nslice, a.nslice, a.k, lane, heads);
    merge_row_dispatch(pk, heads, a.nslice, a.k, lane, key, lse, s_mrg[wave]);
  }
  if (lane < a.k) {
    a.topk_token[(size_t)row * a.k + lane] = key_token(key);
    a.topk_logprob[(size_t)row * a.k + lane] = key_value(key) - lse;
  }
  if (lane == 0) a.lse[row] = lse;
}

hipError_t launch_merge(const MergeArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL(merge_kernel, dim3((a.n_rows + 3) / 4), dim3(256), 0, stream, a);
  return hipGetLastError();
}

// ---- row reduction of materialised logits (GEMM path) ------------------------------------------
// One workgroup per row.  The GEMM left, for every group of 64 consecutive vocabulary rows, the
// group's max and sum of exponentials.  lse follows from those alone.  The k-th largest of the threads' maxima (of one to eight
// groups each) is a lower bound T of the row's k-th largest logit (k distinct elements are >= T), and only the
// groups whose max reaches T - k of them, or a few more - can hold an element >= T: those groups'
// logits are read (64 values each), the candidates >= T collected, and the exact top-k by (logit
// desc, token asc) taken among them (a candidate's rank is the number of larger keys).  Massive ties (e.g. constant logits) overflow
// the lists: with too many candidate groups the whole row is scanned instead, and with too many candidates an
// exact but slow path takes over: k passes over the row, each finding the largest key below the
// previous winner.
constexpr int kCandMax = 2048;
constexpr int kGrpListMax = 256;   // groups that may hold a candidate; more than that: the row is scanned

// The rank-j key of a row of logits, in the form the launch's caller wants it.  For a wide beam inside a draft call the row
// also forms its candidates of the beam update (Algorithm 1's next summed logprobs) - with k * k of them per sequence that is
// 160 KB of pool entries, which one workgroup per sequence spent most of its launch on - and leaves their keys.  WIDE: whether the
// kernel serves such beams.
template <bool WIDE>
struct RowEmit {
  const RowTopkArgs& a;
  int row;
  float lse;
  float parent_lps;    // of this row's beam slot (a.form)
  int parent_node;

  __device__ __forceinline__ RowEmit(const RowTopkArgs& args, int r) : a(args), row(r), lse(0.f), parent_lps(0.f), parent_node(0) {
    if (WIDE && a.form) {
      parent_lps = a.beam.st.logprobsum[row];            // row b * k + i is slot i of sequence b
      parent_node = a.beam.st.beam_node[row];
    }
  }
  __device__ __forceinline__ void operator()(int j, uint64_t key) const {
    if (a.topk_token != nullptr) {
      // the results of a single LM-head call (a separate launch that turned keys into tokens and logprobs cost 5 us)
      a.topk_token[(size_t)row * a.k + j] = key_token(key);
      a.topk_logprob[(size_t)row * a.k + j] = key_value(key) - lse;
    } else if (WIDE && a.form) {
      const int k = a.k, b = row / k, f = (row - b * k) * k + j, t = key_token(key);
      const float sc = __fadd_rn(parent_lps, key_value(key) - lse);   // logprob = logit - lse, then one fp32 add
      const size_t pn = (size_t)b * a.beam.nmax + 1 + k + (size_t)(a.beam.step - 1) * k * k + f;
      a.beam.st.pool_token[pn] = t;
      a.beam.st.pool_parent[pn] = parent_node;
      a.beam.st.pool_depth[pn] = a.beam.step + 1;
      a.beam.st.pool_score[pn] = sc;
      a.part_key[(size_t)row * k + j] = wide_beam_key(sc, t, f);
    } else {
      a.part_key[(size_t)row * a.k + j] = key;
    }
  }
  __device__ __forceinline__ void row_lse() const {       // by one thread
    if (a.topk_token != nullptr)
      a.lse[row] = lse;
    else
      a.part_sum[row] = lse;
  }
};

// S: groups per thread (V <= 64 * 256 * S).  Their statistics are asked for once, all together, and stay in registers: five loops over
// the groups in memory were five chains of round trips (V = 128256, 128 rows, k = 16: 22.7 us a launch, now 9; V = 32000: 7.5, now 5.8).
template <int S>
__global__ __launch_bounds__(256) void row_topk_kernel(RowTopkArgs a) {
  __shared__ uint64_t s_cand[kCandMax];
  __shared__ float s_red[8];
  __shared__ int s_cnt, s_ng;
  __shared__ int s_glist[kGrpListMax];
  __shared__ uint32_t s_max[256], s_least[1];
  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // The compiler waits for the flag in front of the row's loads all the same (its load hangs on the null test), but the kernel's
  // arguments arrive beside it: 0.6 us a launch less than with the return here.
  const int on = a.row_active != nullptr ? a.row_active[row] : 1;
  RowEmit<false> emit(a, row);
  const int ngrp_valid = (a.V + 63) >> 6;
  const float* gmax = a.grp_max + (size_t)row * a.ngrp;
  const float* gsum = a.grp_sum + (size_t)row * a.ngrp;
  float gm[S], gs[S];                                          // of groups tid + 256 i; past the last: -inf, 0
#pragma unroll
  for (int i = 0; i < S; ++i) {
    const int g = tid + 256 * i;
    gm[i] = g < ngrp_valid ? gmax[g] : -INFINITY;
    gs[i] = g < ngrp_valid ? gsum[g] : 0.f;
  }
  if (on == 0) return;                                         // uniform

  // ---- row max, lse ---------------------------------------------------------------------------
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < S; ++i) m = fmaxf(m, gm[i]);
  m = wave_max_f32(m);
  if (lane == 0) s_red[wave] = m;
  __syncthreads();
  const float M = fmaxf(fmaxf(s_red[0], s_red[1]), fmaxf(s_red[2], s_red[3]));
  float acc = 0.f;
#pragma unroll
  for (int i = 0; i < S; ++i)
    if (tid + 256 * i < ngrp_valid) acc += gs[i] * __expf(gm[i] - M);
  acc = wave_sum_f32(acc);
  if (lane == 0) s_red[4 + wave] = acc;
  // ---- T: the k-th largest of the threads' maxima (or -inf if there are fewer than k), reached by k groups at least ----
  uint32_t tm = 0u;
#pragma unroll
  for (int i = 0; i < S; ++i)
    if (tid + 256 * i < ngrp_valid) tm = umax32(tm, ord32(gm[i]));
  s_max[tid] = tm;
  if (tid == 0) {
    s_cnt = 0;
    s_ng = 0;
  }
  const int nval = min(ngrp_valid, 256);
  const uint32_t least = block_kth_largest_u32(s_max, nval, min(a.k, nval), s_least, tid);   // its barriers publish s_red
  const float T = nval < a.k ? -INFINITY : unord32(least);
  const float lse = M + __logf(s_red[4] + s_red[5] + s_red[6] + s_red[7]);
  emit.lse = lse;
  if (tid == 0) emit.row_lse();

  // ---- collect candidates >= T ------------------------------------------------------------------
  // Only groups whose max reaches T can hold one: usually k or a few more of them, so the row's
  // logits are read group by group (64 consecutive values, one per lane) rather than scanned.
  const float* x = a.logits + (size_t)row * a.ldl;
#pragma unroll
  for (int i = 0; i < S; ++i)
    if (tid + 256 * i < ngrp_valid && gm[i] >= T) {
      const int p = atomicAdd(&s_ng, 1);
      if (p < kGrpListMax) s_glist[p] = tid + 256 * i;
    }
  __syncthreads();
  const int ng = s_ng;
  if (__builtin_expect(ng <= kGrpListMax, 1)) {                // uniform
    for (int i0 = wave; i0 < ng; i0 += 16) {
      float xv[4];
      int vv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {                            // four independent loads in flight
        const int i = i0 + 4 * u;
        vv[u] = (i < ng) ? s_glist[i] * 64 + lane : a.V;
        xv[u] = (vv[u] < a.V) ? x[vv[u]] : -INFINITY;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (vv[u] < a.V && xv[u] >= T) {
          const int p = atomicAdd(&s_cnt, 1);
          if (p < kCandMax) s_cand[p] = row_key(xv[u], vv[u]);
        }
    }
  } else if ((a.ldl & 3) == 0) {                               // too many groups tie at T: scan the row
    const int nchunk = (a.V + 3) >> 2;                         // the last piece may reach into the row's padding
    for (int c0 = tid; c0 < nchunk; c0 += 8 * 256) {
      float4 q[8];   // eight independent 16-byte loads in flight before any is consumed
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int c = c0 + u * 256;
        q[u] = (c < nchunk) ? *reinterpret_cast<const float4*>(x + 4 * c)
                            : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int c = c0 + u * 256;
        const float xq[4] = {q[u].x, q[u].y, q[u].z, q[u].w};
        if (c < nchunk && fmaxf(fmaxf(xq[0], xq[1]), fmaxf(xq[2], xq[3])) >= T) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (xq[e] >= T && 4 * c + e < a.V) {
              const int p = atomicAdd(&s_cnt, 1);
              if (p < kCandMax) s_cand[p] = row_key(xq[e], 4 * c + e);
            }
        }
      }
    }
  } else {
    for (int v = tid; v < a.V; v += 256) {
      const float xs = x[v];
      if (xs >= T) {
        const int p = atomicAdd(&s_cnt, 1);
        if (p < kCandMax) s_cand[p] = row_key(xs, v);
      }
    }
  }
  __syncthreads();
  const int cnt = s_cnt;

  if (__builtin_expect(cnt <= 256, 1)) {                       // uniform: the usual case, a few more than k candidates
    // ---- exact top-k among the candidates: a candidate's rank is the number of larger keys (keys are distinct) ---
    if (tid < cnt) {
      const uint64_t mine = s_cand[tid];
      int rank = 0;
      for (int j = 0; j < cnt; ++j) rank += (s_cand[j] > mine) ? 1 : 0;
      if (rank < a.k) emit(rank, mine);
    } else if (tid < a.k) {
      emit(tid, 0ull);                                         // fewer candidates than beams (V < k cannot happen; kept total)
    }
  } else if (cnt <= kCandMax) {                                // uniform
    // ---- many candidates (ties at the threshold): wave 0, k rounds of wave max over its strided share ---
    if (wave == 0) {
      uint64_t mine = 0ull;
      for (int round = 0; round < a.k; ++round) {
        uint64_t loc = 0ull;
        for (int i = lane; i < cnt; i += 64) loc = umax64(loc, s_cand[i]);
        const uint64_t best = wave_max_u64(loc);
        if (lane == round) mine = best;
        for (int i = lane; i < cnt; i += 64)
          if (s_cand[i] == best) s_cand[i] = 0ull;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
      if (lane < a.k) emit(lane, mine);
    }
  } else {
    // ---- more than kCandMax elements tie at or above T (e.g. constant logits): exact but slow ------
    // k rounds; each finds the largest key below the previous winner by a pass over the whole row.
    uint64_t* s_best = s_cand;   // [4] per-wave maxima
    uint64_t prev = ~0ull, mine = 0ull;
    for (int round = 0; round < a.k; ++round) {
      uint64_t loc = 0ull;
      for (int v = tid; v < a.V; v += 256) {
        const uint64_t key = row_key(x[v], v);
        if (key < prev) loc = umax64(loc, key);
      }
      loc = wave_max_u64(loc);
      __syncthreads();
      if (lane == 0) s_best[wave] = loc;
      __syncthreads();
      prev = umax64(umax64(s_best[0], s_best[1]), umax64(s_best[2], s_best[3]));
      if (tid == round) mine = prev;
    }
    if (tid < a.k) emit(tid, mine);
  }
}

// The same for wide beams (DDD_KMAX < k <= DDD_KWIDE_MAX), where a bound from quad maxima no longer holds k keys: 1024
// threads find the k-th largest group maximum (one wave, bit by bit), and rank the candidates at or above it by counting.  More
// than 512 groups are folded to the maxima of up to four first: the
// k-th largest of those is reached by k groups too, only a few more groups pass it (counting all 2000 groups of V = 128000
// took 60 us).  (Bitonic sorts of both by 256 threads, a block barrier per stage, took 28 us a launch at k = 100,
// V = 32000, whatever the number of rows; 14 us with the counting, 11 with the k-th group maximum found by one wave.)
constexpr int kWideRowThreads = 1024;
constexpr int kWideGroups = 2048;   // V <= 2^17
constexpr int kWideFold = 512;      // most values that are ranked
static_assert(kWideGroups == 2 * kWideRowThreads && kWideFold == kWideRowThreads / 2, "a thread's two groups, and its neighbour's");
static_assert(kWideFold <= kKthMost, "one wave ranks them");

__global__ __launch_bounds__(kWideRowThreads) void row_topk_wide_kernel(RowTopkArgs a) {
  __shared__ __align__(16) uint32_t s_gm[kWideFold];         // (folded) group maxima as ordered keys
  __shared__ int s_num[kWideGroups];                         // the groups that hold candidates
  __shared__ uint64_t s_cand[kCandMax];
  __shared__ int s_rank[kCandMax];
  __shared__ float s_red[2][16];
  __shared__ uint32_t s_min[1];
  __shared__ int s_cnt, s_ng;
  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // The compiler waits for the flag in front of the row's loads all the same (its load hangs on the null test), but the kernel's
  // arguments arrive beside it: 0.6 us a launch less than with the return here.
  const int on = a.row_active != nullptr ? a.row_active[row] : 1;
  RowEmit<true> emit(a, row);
  const int ngrp = (a.V + 63) >> 6;
  uint32_t top = 0u;                                         // the larger of the thread's groups
  float m = -INFINITY, mine_max[2] = {-INFINITY, -INFINITY}, mine_sum[2] = {0.f, 0.f};
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int g = tid + u * kWideRowThreads;
    if (g < ngrp) {
      mine_max[u] = a.grp_max[(size_t)row * a.ngrp + g];
      mine_sum[u] = a.grp_sum[(size_t)row * a.ngrp + g];
      top = umax32(top, ord32(mine_max[u]));
    }
    m = fmaxf(m, mine_max[u]);
  }
  if (on == 0) return;                                       // uniform
  const bool fold = ngrp > kWideFold;                        // uniform
  if (fold) {
    top = umax32(top, dpp_move_u32<0xB1>(top));              // lane ^ 1
    if ((tid & 1) == 0) s_gm[tid >> 1] = top;
  } else if (tid < kWideFold) {
    s_gm[tid] = top;
  }
  const int nval = fold ? (min(ngrp, kWideRowThreads) + 1) >> 1 : ngrp;   // more than k if folded
  if (tid == 0) s_cnt = s_ng = 0;
  for (int i = tid; i < kCandMax; i += kWideRowThreads) s_rank[i] = 0;
  m = wave_max_f32(m);
  if (lane == 0) s_red[0][wave] = m;
  __syncthreads();
  float M = s_red[0][0];
#pragma unroll
  for (int w = 1; w < 16; ++w) M = fmaxf(M, s_red[0][w]);
  float acc = 0.f;
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (tid + u * kWideRowThreads < ngrp) acc += mine_sum[u] * __expf(mine_max[u] - M);
  acc = wave_sum_f32(acc);
  if (lane == 0) s_red[1][wave] = acc;
  // ---- T = k-th largest (folded) group max --------------------------------------------------------------------------
  const uint32_t least = block_kth_largest_u32(s_gm, nval, min(a.k, nval), s_min, tid);   // its barriers publish s_red
  const float T = (ngrp < a.k) ? -INFINITY : unord32(least);
  float total = 0.f;
#pragma unroll
  for (int w = 0; w < 16; ++w) total += s_red[1][w];            // fixed order
  emit.lse = M + __logf(total);
  if (tid == 0) emit.row_lse();
  // ---- the groups that can hold a candidate, and the candidates >= T -------------------------------------------------
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int g = tid + u * kWideRowThreads;
    if (g < ngrp && mine_max[u] >= T) s_num[atomicAdd(&s_ng, 1)] = g;
  }
  __syncthreads();
  const float* x = a.logits + (size_t)row * a.ldl;
  const int ng = s_ng;
  for (int i0 = wave; i0 < ng; i0 += 16 * 8) {
    float xv[8];
    int vv[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {                               // eight groups' loads in flight
      const int i = i0 + 16 * u;
      vv[u] = (i < ng) ? s_num[i] * 64 + lane : a.V;
      xv[u] = (vv[u] < a.V) ? x[vv[u]] : -INFINITY;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const bool in = vv[u] < a.V && xv[u] >= T;
      const unsigned long long bal = __ballot(in);
      if (bal == 0ull) continue;                                // wave-uniform
      int base = 0;
      if (lane == 0) base = atomicAdd(&s_cnt, __popcll(bal));
      const int p = __builtin_amdgcn_readfirstlane(base) + __popcll(bal & ((1ull << lane) - 1ull));
      if (in && p < kCandMax) s_cand[p] = row_key(xv[u], vv[u]);
    }
  }
  __syncthreads();
  const int cnt = s_cnt;
  if (__builtin_expect(cnt <= kCandMax, 1)) {                   // uniform
    count_larger_keys(s_cand, cnt, s_rank, tid, kWideRowThreads);
    __syncthreads();
    for (int i = tid; i < cnt; i += kWideRowThreads)
      if (s_rank[i] < a.k) emit(s_rank[i], s_cand[i]);
    for (int j = cnt + tid; j < a.k; j += kWideRowThreads) emit(j, 0ull);   // fewer candidates than beams: no number in the row
    return;
  }
  // ---- more than kCandMax elements tie at or above T (e.g. constant logits): exact but slow ---------------------------
  uint64_t prev = ~0ull, mine = 0ull;
  for (int round = 0; round < a.k; ++round) {
    uint64_t loc = 0ull;
    for (int v = tid; v < a.V; v += kWideRowThreads) {
      const uint64_t key = row_key(x[v], v);
      if (key < prev) loc = umax64(loc, key);
    }
    loc = wave_max_u64(loc);
    __syncthreads();
    if (lane == 0) s_cand[wave] = loc;
    __syncthreads();
    prev = s_cand[0];
#pragma unroll
    for (int w = 1; w < 16; ++w) prev = umax64(prev, s_cand[w]);
    if (tid == round) mine = prev;
  }
  if (tid < a.k) emit(tid, mine);
}

hipError_t launch_row_topk(const RowTopkArgs& a, hipStream_t stream) {
  if (a.k > DDD_KMAX)
    hipLaunchKernelGGL(row_topk_wide_kernel, dim3(a.n_rows), dim3(kWideRowThreads), 0, stream, a);
  else if (a.V <= 64 * 256 * 2)
    hipLaunchKernelGGL(row_topk_kernel<2>, dim3(a.n_rows), dim3(256), 0, stream, a);
  else if (a.V <= 64 * 256 * 4)
    hipLaunchKernelGGL(row_topk_kernel<4>, dim3(a.n_rows), dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL(row_topk_kernel<8>, dim3(a.n_rows), dim3(256), 0, stream, a);
  return hipGetLastError();
}

__global__ __launch_bounds__(64) void beam_select_kernel(BeamArgs a) {
  const int b = blockIdx.x, lane = threadIdx.x;
  if (!a.st.active[b]) return;
  const size_t row0 = (a.step == 0) ? (size_t)b : (size_t)b * a.k;
  const int li = min(lane, a.k - 1);
  const float old_lps = a.st.logprobsum[(size_t)b * a.k + li];
  const int old_node = a.st.beam_node[(size_t)b * a.k + li];
  beam_update(a, b, lane, a.topk_token + row0 * a.k, a.topk_logprob + row0 * a.k, a.k, old_lps, old_node);
}

__global__ __launch_bounds__(64) void depth_continue_kernel(BeamArgs a, int steps_done) {
  const int b = blockIdx.x, lane = threadIdx.x;
  if (!a.st.active[b]) return;
  const float v = (lane < a.k) ? a.st.logprobsum[(size_t)b * a.k + lane] : 0.f;
  stop_test(a, b, lane, v, steps_done);
}

hipError_t launch_beam_select(const BeamArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL(beam_select_kernel, dim3(a.B), dim3(64), 0, stream, a);
  return hipGetLastError();
}
hipError_t launch_depth_continue(const BeamArgs& a, int steps_done, hipStream_t stream) {
  hipLaunchKernelGGL(depth_continue_kernel, dim3(a.B), dim3(64), 0, stream, a, steps_done);
  return hipGetLastError();
}

// ---- one launch per draft call (rows that came through the GEMM path, or a caller that runs
// the weight stream separately): one workgroup per sequence ---------------------------------------
template <bool DENSE>
__global__ __launch_bounds__(1024) void step_bookkeep_kernel(StepArgs a) {
  __shared__ StepSmem sm;
  const int b = blockIdx.x, tid = threadIdx.x;
  if (a.trace != nullptr && b == 0 && tid == 0) a.trace[0] = (uint64_t)wall_clock64();
  const bool active = step_bookkeep_block<DENSE>(a, b, tid, blockDim.x, sm);
  if (a.trace != nullptr && b == 0 && tid == 0) a.trace[5] = (uint64_t)wall_clock64();
  report_call(a.report, active, b, a.beam.k, tid, blockDim.x);
}

hipError_t launch_step_bookkeep(const StepArgs& a, hipStream_t stream) {
  if (a.nslice == 0)
    hipLaunchKernelGGL(step_bookkeep_kernel<true>, dim3(a.beam.B), dim3(64 * a.beam.k), 0, stream, a);
  else
    hipLaunchKernelGGL(step_bookkeep_kernel<false>, dim3(a.beam.B), dim3(64 * a.beam.k), 0, stream, a);
  return hipGetLastError();
}

// ---- poison fill of the scratch (debugging aid) -------------------------------------------------
__global__ __launch_bounds__(256) void poison_kernel(uint32_t* p, size_t n_words) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_words; i += (size_t)gridDim.x * blockDim.x)
    p[i] = 0xFFFFFFFFu;
}

hipError_t launch_poison(void* p, size_t bytes, hipStream_t stream) {
  const size_t n = bytes / 4;
  if (n == 0) return hipSuccess;
  const size_t want = (n + 255) / 256;
  hipLaunchKernelGGL(poison_kernel, dim3((unsigned)(want < 2048 ? want : 2048)), dim3(256), 0, stream,
                     static_cast<uint32_t*>(p), n);
  return hipGetLastError();
}

// ---- start of a round ------------------------------------------------------------------------
__global__ __launch_bounds__(64) void round_reset_kernel(ResetArgs a) {
  const int b = blockIdx.x, lane = threadIdx.x;
  if (lane == 0) {
    a.st.pool_token[(size_t)b * a.nmax] = a.root_token ? a.root_token[b] : -1;
    a.st.pool_parent[(size_t)b * a.nmax] = -1;
    a.st.pool_depth[(size_t)b * a.nmax] = 0;
    a.st.pool_score[(size_t)b * a.nmax] = 0.f;
    a.st.n_nodes[b] = 1;
    a.st.steps[b] = 0;
    a.st.active[b] = 1;
    a.st.conf[b] = 1.0;
  }
  if (lane < a.k) a.st.row_active[(size_t)b * a.k + lane] = 1;
}

hipError_t launch_round_reset(const ResetArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL(round_reset_kernel, dim3(a.B), dim3(64), 0, stream, a);
  return hipGetLastError();
}

}  // namespace ddd
