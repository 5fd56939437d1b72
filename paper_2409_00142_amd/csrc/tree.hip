// Final draft tree (top-m rerank, order, parents, positions, attention mask), the greedy accept
// walk and sampled acceptance.  One workgroup per sequence; everything is integer work on at most
// DDD_POOL_MAX nodes, so it lives in LDS.
#include "tree_device.hpp"

namespace ddd {

__global__ __launch_bounds__(1024) void tree_finalize_kernel(FinalizeArgs a) {
  __shared__ TreeSmem sm;
  tree_finalize_block<4>(a.st, a.tree, blockIdx.x, a.m, a.nmax, threadIdx.x, blockDim.x, sm);
}

hipError_t launch_tree_finalize(const FinalizeArgs& a, hipStream_t stream) {
  // Half the waves, two nodes a thread, where neither the pool nor the mask keeps them busy: barriers and the conclusions that every wave
  // draws cost less.  512 against 1024 threads, m = 60: one sequence with 511 / 811 nodes 5.27 and 5.57 us, 5.26 and 5.41; eight
  // 5.7 and 6.2, 5.99 and 6.09; 64 5.9 and 6.3, 6.3 and 6.6.  A wider mask keeps sixteen waves busy: 511
  // nodes and m = 64 5.72 and 5.81, m = 80 5.88 and 5.85.
  const int threads = a.nmax <= 1025 && a.m <= 64 ? 512 : 1024;
  static_assert(DDD_POOL_MAX <= 4 * 1024 + 1, "a thread for every four nodes");
  hipLaunchKernelGGL(tree_finalize_kernel, dim3(a.B), dim3(threads), 0, stream, a);
  return hipGetLastError();
}

// Round statistics (Section 3.3 / Table 1: accepted length per round; Section 2: draft calls per round), added by
// the one thread per sequence that has the sequence's accepted length.  That thread calls stats_begin before its
// walk: the sequence's depth is read and goes into the round's running maximum while the walk runs, so that the end
// of the walk waits for nothing.  The sequence that arrives last closes the round: every sequence's depth has gone
// into the maximum before its arrival (the arrival's operand depends on the value the maximum returned, so the
// two atomics cannot pass each other), and the two words are zero again when the launch ends.  A batch of one has
// nothing to agree on.  Every update is an integer atomic without a returned value where none is needed.
struct StatsPre {
  int d;
  unsigned before;
};
__device__ __forceinline__ StatsPre stats_begin(const StatsArgs& s, int b, int B) {
  StatsPre p{0, 0u};
  if (s.sync == nullptr) return p;
  if (s.steps != nullptr) p.d = min(max(s.steps[b], 0), 31);
  if (B > 1) p.before = atomicMax(s.sync + 1, (unsigned)p.d);
  return p;
}
__device__ __forceinline__ void stats_end(const StatsArgs& s, const StatsPre& p, int B, int len) {
  if (s.sync == nullptr) return;
  typedef unsigned long long u64;
  if (s.accept_hist != nullptr) atomicAdd(reinterpret_cast<u64*>(s.accept_hist + min(max(len, 0), 31)), 1ull);
  if (s.depth_hist != nullptr && s.steps != nullptr) atomicAdd(reinterpret_cast<u64*>(s.depth_hist + p.d), 1ull);
  unsigned deepest = (unsigned)p.d;
  if (B > 1) {
    unsigned one = 1u;
    asm volatile("" : "+v"(one) : "v"(p.before));
    if (atomicAdd(s.sync, one) != (unsigned)(B - 1)) return;
    deepest = atomicExch(s.sync + 1, 0u);
    atomicExch(s.sync, 0u);
  }
  if (s.batch_depth_hist != nullptr && s.steps != nullptr) atomicAdd(reinterpret_cast<u64*>(s.batch_depth_hist + deepest), 1ull);
  if (s.rounds != nullptr) atomicAdd(reinterpret_cast<u64*>(s.rounds), 1ull);
}

// Section 1 / Section 3.1 (temperature 0): follow the child whose token equals the target's
// argmax at the current node until there is none; the argmax there is the bonus token.  One wave, one round trip: the whole tree and
// the target's tokens are in registers (three tree indices per lane) before the walk, whose steps are ballots and one lane read (a
// load per step: 3.9 us a launch of one sequence, now 2.4; 64 of them 5.7, now 3.9).
constexpr int kVaSlots = (DDD_MMAX + 1 + 63) / 64;
__global__ __launch_bounds__(64) void verify_accept_kernel(VerifyArgs a) {
  const int b = blockIdx.x, lane = threadIdx.x;
  const int T = a.m + 1;
  const int32_t* tok = a.tree.tree_token + (size_t)b * T;
  const int32_t* par = a.tree.parent_idx + (size_t)b * T;
  const int32_t* tgt = a.target_argmax + (size_t)b * T;
  int32_t* path = a.accept_path + (size_t)b * (a.D + 1);
  int tk[kVaSlots], pr[kVaSlots], tg[kVaSlots];
#pragma unroll
  for (int q = 0; q < kVaSlots; ++q) {
    const int c = min(64 * q + lane, T - 1);
    tk[q] = tok[c];
    pr[q] = par[c];
    tg[q] = tgt[c];
  }
  const int n = a.tree.n_sel[b] + 1;
  int cur = 0, len = 0;
  StatsPre sp{0, 0u};
  if (lane == 0) {
    path[0] = 0;
    sp = stats_begin(a.stats, b, a.B);
  }
  auto target_of = [&](int c) {            // c is wave-uniform
    int t = 0;
#pragma unroll
    for (int q = 0; q < kVaSlots; ++q) t = (c >> 6) == q ? __builtin_amdgcn_readlane(tg[q], c & 63) : t;
    return t;
  };
  int want = target_of(0);
  for (int it = 0; it < a.D; ++it) {
    int found = -1;
#pragma unroll
    for (int q = kVaSlots - 1; q >= 0; --q) {
      const int c = 64 * q + lane;
      const unsigned long long hit = __ballot(c >= 1 && c < n && pr[q] == cur && tk[q] == want);
      if (hit != 0ull) found = 64 * q + __ffsll(hit) - 1;
    }
    if (found < 0) break;                  // uniform
    cur = found;
    want = target_of(cur);
    ++len;
    if (lane == 0) path[len] = cur;
  }
  if (lane == 0) {
    for (int i = len + 1; i <= a.D; ++i) path[i] = -1;
    a.accept_len[b] = len;
    a.bonus_token[b] = want;
    stats_end(a.stats, sp, a.B, len);
  }
}

hipError_t launch_verify_accept(const VerifyArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL(verify_accept_kernel, dim3(a.B), dim3(64), 0, stream, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Sampled acceptance at temperature T > 0.  The paper measures at temperature 0 (Section 3.1) and
// fixes only that the emitted tokens follow the target model's distribution (Section 1).  The
// drafted children of a node are a deterministic function of the context, i.e. point-mass
// proposals: child x is accepted with probability p(x); after a rejection p continues without x,
// renormalised.  With w_j = exp((x_j - max x) / T) kept unnormalised and rem = sum of the
// weights not yet rejected:   accept child c  iff  u_accept[c] * rem < w[token_c];  when no child is
// accepted the bonus token is the first j whose prefix sum of the remaining weights exceeds
// u_bonus[node] * rem.  Every decision is taken in fp64.
//
// A row is cut into 128 blocks of consecutive tokens (coalesced loads, fixed summation order) whose sums of weights are
// kept, so the bonus draw only has to look inside the one block in which the prefix sum passes the threshold.
//
// The walk is a chain - which row is next depends on the decision at this one - and a row of 32 000 fp64 exponentials
// keeps one CU busy for about 8 us, so the two ways of doing it differ in where the rows' sums are made:
//  * small batches (verify_sample_from_sums): a first launch makes the sums of the rows of every tree with the whole chip, and the walk
//    that follows looks numbers up.  It is bound by the rows it reads (62 MB take the memory 12 us, the fp64 instructions 9), so the
//    rows of leaves, half of a tree's nodes, are left out: a walk tests no children there, and few end there.  Where one does, the
//    workgroups of the walk's launch make that row's sums between them (4 to 5 us).  With and without the leaves' rows, 61 nodes:
//    B = 8, V = 32000 24.7 and 18.9 to 21.3 us a call, B = 16 40.4 and 29.2, B = 6 21.5 and 18.9, B = 1 11.9 and 12.3; B = 30, V = 4001,
//    49 nodes 17.4 and 18.4: what is left out must be worth the leaf of the walk (sums_of_leaves).  (Workgroups of twice and four times
//    the blocks, which issue a tenth less per token: 31 and 36 us, because all of the loads then come before all of the arithmetic.)
//    Above 128 MiB of logits the rows are still more than a walk needs if it ends early, so a launch in front makes the roots' sums and
//    decides there, and only rows below the accepted child are summed up (roots_first).
//  * beyond that (verify_sample_kernel): one workgroup of 16 waves per sequence makes the sums of the rows it visits.
// The line lies where the extra rows would cost what they save (rows_from_sums).
constexpr int kVsWaves = 16;
constexpr int kVsThreads = kVsWaves * kWave;
constexpr int kVsSubPerWave = 8;
constexpr int kVsSub = kVsWaves * kVsSubPerWave;     // 128 = two per lane of the wave that draws the bonus
constexpr int kVsMaxRemoved = 128;                   // children of one node <= beam width <= 128
constexpr int kVsChunk = 4 * kWave;                  // tokens one wave loads per instruction

// exp(d / T) for d = x - max <= 0 as 2^(d * beta2), beta2 = log2(e) / T: n = the nearest integer of the exponent, f the
// exact rest, and a polynomial of degree 10 through the Chebyshev nodes of [-1/2, 1/2] (3e-16).  The difference from
// the row maximum is taken first (exact for the logits that matter), so the weight of the maximum is 1 and the error of
// the others 2e-15 at T = 1, that of a row's sum 1e-16 (a Taylor polynomial of degree 11 around exp(x / T - max / T), as before:
// 9e-15 and 5e-16).  19 fp64 instructions per token.  Exactly 0 for -inf.
__device__ __forceinline__ double weight_of(double d, double beta2) {
  const double t = fmax(d * beta2, -1200.0);
  const double n = __builtin_rint(t);
  const double f = t - n;
  double p = 7.072585949269223e-09;
  p = fma(p, f, 1.0208690299958306e-07);
  p = fma(p, f, 1.321544258792169e-06);
  p = fma(p, f, 1.5252657260200837e-05);
  p = fma(p, f, 0.0001540353044173605);
  p = fma(p, f, 0.0013333558230164974);
  p = fma(p, f, 0.009618129107606888);
  p = fma(p, f, 0.05550410866444772);
  p = fma(p, f, 0.24022650695910097);
  p = fma(p, f, 0.69314718055995);
  p = fma(p, f, 1.0);
  return ldexp(p, (int)n);
}
// The same for the rows' sums, in 10 fp64 instructions instead of 19, by a table (the usual table-driven exponential; Tang, "Table-driven
// implementation of the exponential function in IEEE floating-point arithmetic", ACM TOMS 15, 1989): 2^t = 2^(n/128) 2^f with
// |f| <= 1/256, where adding 1.5 * 2^45 leaves n in the low word, the 128 values of 2^(j/128), rounded to nearest, sit in LDS and
// 2^f - 1 is f times a cubic through the Chebyshev nodes (1.5e-16 with the rounding of its coefficients).  f takes one rounding (t is
// never rounded), so a weight is closer to the exact one than above.  B = 8, V = 32000, 61 nodes: 29.5 -> 26.8 us a call with the
// constants of T made by the host; B = 16 48.2 -> 43.2.  The high words of the table are less by j << 13, so that adding n << 13 puts
// the integer part of n / 128 into the exponent field.  For t in (-1021, 0].
constexpr int kVsExpSize = 128;
__device__ const unsigned long long kVsExp[kVsExpSize] = {
    0x3ff0000000000000ull, 0x3feff63da9fb3335ull, 0x3fefec9a3e778061ull, 0x3fefe315e86e7f85ull,
    0x3fefd9b0d3158574ull, 0x3fefd06b29ddf6deull, 0x3fefc74518759bc8ull, 0x3fefbe3ecac6f383ull,
    0x3fefb5586cf9890full, 0x3fefac922b7247f7ull, 0x3fefa3ec32d3d1a2ull, 0x3fef9b66affed31bull,
    0x3fef9301d0125b51ull, 0x3fef8abdc06c31ccull, 0x3fef829aaea92de0ull, 0x3fef7a98c8a58e51ull,
    0x3fef72b83c7d517bull, 0x3fef6af9388c8deaull, 0x3fef635beb6fcb75ull, 0x3fef5be084045cd4ull,
    0x3fef54873168b9aaull, 0x3fef4d5022fcd91dull, 0x3fef463b88628cd6ull, 0x3fef3f49917ddc96ull,
    0x3fef387a6e756238ull, 0x3fef31ce4fb2a63full, 0x3fef2b4565e27cddull, 0x3fef24dfe1f56381ull,
    0x3fef1e9df51fdee1ull, 0x3fef187fd0dad990ull, 0x3fef1285a6e4030bull, 0x3fef0cafa93e2f56ull,
    0x3fef06fe0a31b715ull, 0x3fef0170fc4cd831ull, 0x3feefc08b26416ffull, 0x3feef6c55f929ff1ull,
    0x3feef1a7373aa9cbull, 0x3feeecae6d05d866ull, 0x3feee7db34e59ff7ull, 0x3feee32dc313a8e5ull,
    0x3feedea64c123422ull, 0x3feeda4504ac801cull, 0x3feed60a21f72e2aull, 0x3feed1f5d950a897ull,
    0x3feece086061892dull, 0x3feeca41ed1d0057ull, 0x3feec6a2b5c13cd0ull, 0x3feec32af0d7d3deull,
    0x3feebfdad5362a27ull, 0x3feebcb299fddd0dull, 0x3feeb9b2769d2ca7ull, 0x3feeb6daa2cf6642ull,
    0x3feeb42b569d4f82ull, 0x3feeb1a4ca5d920full, 0x3feeaf4736b527daull, 0x3feead12d497c7fdull,
    0x3feeab07dd485429ull, 0x3feea9268a5946b7ull, 0x3feea76f15ad2148ull, 0x3feea5e1b976dc09ull,
    0x3feea47eb03a5585ull, 0x3feea34634ccc320ull, 0x3feea23882552225ull, 0x3feea155d44ca973ull,
    0x3feea09e667f3bcdull, 0x3feea012750bdabfull, 0x3fee9fb23c651a2full, 0x3fee9f7df9519484ull,
    0x3fee9f75e8ec5f74ull, 0x3fee9f9a48a58174ull, 0x3fee9feb564267c9ull, 0x3feea0694fde5d3full,
    0x3feea11473eb0187ull, 0x3feea1ed0130c132ull, 0x3feea2f336cf4e62ull, 0x3feea427543e1a12ull,
    0x3feea589994cce13ull, 0x3feea71a4623c7adull, 0x3feea8d99b4492edull, 0x3feeaac7d98a6699ull,
    0x3feeace5422aa0dbull, 0x3feeaf3216b5448cull, 0x3feeb1ae99157736ull, 0x3feeb45b0b91ffc6ull,
    0x3feeb737b0cdc5e5ull, 0x3feeba44cbc8520full, 0x3feebd829fde4e50ull, 0x3feec0f170ca07baull,
    0x3feec49182a3f090ull, 0x3feec86319e32323ull, 0x3feecc667b5de565ull, 0x3feed09bec4a2d33ull,
    0x3feed503b23e255dull, 0x3feed99e1330b358ull, 0x3feede6b5579fdbfull, 0x3feee36bbfd3f37aull,
    0x3feee89f995ad3adull, 0x3feeee07298db666ull, 0x3feef3a2b84f15fbull, 0x3feef9728de5593aull,
    0x3feeff76f2fb5e47ull, 0x3fef05b030a1064aull, 0x3fef0c1e904bc1d2ull, 0x3fef12c25bd71e09ull,
    0x3fef199bdd85529cull, 0x3fef20ab5fffd07aull, 0x3fef27f12e57d14bull, 0x3fef2f6d9406e7b5ull,
    0x3fef3720dcef9069ull, 0x3fef3f0b555dc3faull, 0x3fef472d4a07897cull, 0x3fef4f87080d89f2ull,
    0x3fef5818dcfba487ull, 0x3fef60e316c98398ull, 0x3fef69e603db3285ull, 0x3fef7321f301b460ull,
    0x3fef7c97337b9b5full, 0x3fef864614f5a129ull, 0x3fef902ee78b3ff6ull, 0x3fef9a51fbc74c83ull,
    0x3fefa4afa2a490daull, 0x3fefaf482d8e67f1ull, 0x3fefba1bee615a27ull, 0x3fefc52b376bba97ull,
    0x3fefd0765b6e4540ull, 0x3fefdbfdad9cbe14ull, 0x3fefe7c1819e90d8ull, 0x3feff3c22b8f71f1ull,
};
__device__ __forceinline__ void load_exp_table(double* table, int tid) {
  if (tid < kVsExpSize) table[tid] = __longlong_as_double((long long)kVsExp[tid]);
}
__device__ __forceinline__ double add_weight(double acc, double d, double beta2, const double* table) {
  constexpr double kMagic = 52776558133248.0;   // 1.5 * 2^45: one unit in the last place is 1/128
  const double s = fma(d, beta2, kMagic);
  const int n = __double2loint(s);
  const double base = table[n & (kVsExpSize - 1)];
  const double f = fma(d, beta2, -(s - kMagic));
  double p = 0.009618131458021427;
  p = fma(p, f, 0.05550412901022388);
  p = fma(p, f, 0.24022650695909623);
  p = fma(p, f, 0.6931471805599065);
  p = fma(p, f, 1.0);
  return fma(__hiloint2double(__double2hiint(base) + (n << 13), __double2loint(base)), p, acc);
}
// Logits from which on the short form holds (weights of 2^-1000 and more); NaN, which no logit reaches, below an infinite maximum.
__device__ __forceinline__ float short_from(double Md, double span) {
  const double lo = fmax(Md - span, -3.4028234663852886e38);
  float f = (float)lo;
  if ((double)f < lo) f = nextafterf(f, __builtin_inff());
  return f + (float)(Md - Md);
}
// acc and the weights of four tokens; by whole waves.
__device__ __forceinline__ double add_weight4(double acc, const float4& v, double Md, double beta2, float from, const double* table) {
  if (__ballot(!(v.x >= from && v.y >= from && v.z >= from && v.w >= from)) == 0ull) {
    acc = add_weight(acc, (double)v.x - Md, beta2, table);
    acc = add_weight(acc, (double)v.y - Md, beta2, table);
    acc = add_weight(acc, (double)v.z - Md, beta2, table);
    return add_weight(acc, (double)v.w - Md, beta2, table);
  }
  const float ninf = -__builtin_inff();
  if (__ballot(v.x != ninf || v.y != ninf || v.z != ninf || v.w != ninf) == 0ull) return acc;   // past the vocabulary
  const double e0 = weight_of((double)v.x - Md, beta2), e1 = weight_of((double)v.y - Md, beta2);
  const double e2 = weight_of((double)v.z - Md, beta2), e3 = weight_of((double)v.w - Md, beta2);
  return acc + ((e0 + e1) + (e2 + e3));
}

__device__ __forceinline__ double wave_scan_f64(double x, int lane) {   // inclusive prefix over the lanes
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const double t = __shfl_up(x, off, 64);
    if (lane >= off) x += t;
  }
  return x;
}
__device__ __forceinline__ double wave_sum_f64(double x) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}
// Sums over the wave of N values per lane at once (N = 4 or 8; N + 6 - log2 N - 1 exchanges instead of 6 N): the sum of
// value i ends up in the lanes whose top log2 N lane bits are i.
template <int N>
__device__ __forceinline__ double wave_sums_f64(double (&v)[N], int lane) {
  int off = 32;
#pragma unroll
  for (int n = N / 2; n >= 1; n >>= 1, off >>= 1) {
    const bool up = (lane & off) != 0;
#pragma unroll
    for (int i = 0; i < n; ++i) {
      const double keep = up ? v[i + n] : v[i], send = up ? v[i] : v[i + n];
      v[i] = keep + __shfl_xor(send, off, 64);
    }
  }
  double x = v[0];
#pragma unroll
  for (int o = 64 / N / 2; o >= 1; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef f32x4 f32x4_of_floats __attribute__((aligned(4)));   // a row of an odd vocabulary starts on any float

// Four consecutive logits starting at token j (a multiple of 4 past the row start); tokens at or
// beyond lim read as -inf, i.e. weight 0.  vec: the row is 16-byte aligned and V a multiple of 4.
__device__ __forceinline__ float4 load_logits4(const float* x, int j, int lim, bool vec) {
  const float ninf = -__builtin_inff();
  if (vec) return j < lim ? *reinterpret_cast<const float4*>(x + j) : make_float4(ninf, ninf, ninf, ninf);
  float4 v;
  v.x = j < lim ? x[j] : ninf;
  v.y = j + 1 < lim ? x[j + 1] : ninf;
  v.z = j + 2 < lim ? x[j + 2] : ninf;
  v.w = j + 3 < lim ? x[j + 3] : ninf;
  return v;
}
__device__ __forceinline__ float max4(float m, const float4& v) { return fmaxf(fmaxf(m, v.x), fmaxf(v.y, fmaxf(v.z, v.w))); }
__device__ __forceinline__ int chunks_per_block(int V) { return (V + kVsSub * kVsChunk - 1) / (kVsSub * kVsChunk); }
__device__ __forceinline__ bool rows_aligned(const VerifySampleArgs& a) {
  return (a.V & 3) == 0 && (reinterpret_cast<uintptr_t>(a.logits) & 15) == 0;
}
__device__ __forceinline__ double beta2_of(const VerifySampleArgs& a) { return a.beta2; }

// The sequence's tree, read once, and the tokens rejected at the current node.
struct VsTree {
  int par[DDD_MMAX + 1], tok[DDD_MMAX + 1];
  double ua[DDD_MMAX + 1], ub[DDD_MMAX + 1];
  int rm_tok[kVsMaxRemoved];
  double rm_w[kVsMaxRemoved];
};
__device__ __forceinline__ void load_tree(const VerifySampleArgs& a, int b, int tid, VsTree& t) {
  const int T = a.m + 1;
  if (tid < T) {
    t.par[tid] = a.tree.parent_idx[(size_t)b * T + tid];
    t.tok[tid] = min(max(a.tree.tree_token[(size_t)b * T + tid], 0), a.V - 1);
    t.ua[tid] = a.u_accept[(size_t)b * T + tid];
    t.ub[tid] = a.u_bonus[(size_t)b * T + tid];
  }
}

// The children tests of node `cur` by one wave, in tree-index order: lane = tree index base + lane.  kid / kw: whether that
// index is a child and its token's weight, asked for 64 indices at a time.  Returns the accepted child or -1; rem and
// nrm: the weight not rejected and the number of rejected tokens (listed in t).
template <class KidFn>
__device__ __forceinline__ int test_children(VsTree& t, int n, int lane, double& rem, int& nrm, KidFn kids_of) {
  int nxt = -1;
  for (int base = 1; base < n && nxt < 0; base += kWave) {
    bool kid;
    double kw, ku;
    int ktok;
    kids_of(base, kid, kw, ku, ktok);
    uint64_t kids = __ballot(kid);
    while (kids) {
      const int l = __ffsll((unsigned long long)kids) - 1;
      kids &= kids - 1;
      const double w = __shfl(kw, l, 64);
      const int tk = __shfl(ktok, l, 64);
      if (__shfl(ku, l, 64) * rem < w) {
        nxt = base + l;
        break;
      }
      rem -= w;
      if (lane == 0 && nrm < kVsMaxRemoved) {
        t.rm_tok[nrm] = tk;
        t.rm_w[nrm] = w;
      }
      ++nrm;
    }
  }
  nrm = min(nrm, kVsMaxRemoved);
  return nxt;
}

// Bonus token of a row by one wave: the block in which the prefix sum of the remaining weights passes the threshold (v0,
// v1: the sums of blocks 2 lane and 2 lane + 1), then the token inside it; -1 if rounding leaves none.
__device__ __forceinline__ int draw_bonus(const VsTree& t, int nrm, const float* x, double Md, double beta2, double thr, double v0,
                                          double v1, int sb, int V, bool vec, int lane) {
  for (int r = 0; r < nrm; ++r) {
    const int blk = t.rm_tok[r] / sb;
    if (blk == 2 * lane) v0 -= t.rm_w[r];
    if (blk == 2 * lane + 1) v1 -= t.rm_w[r];
  }
  const double inc = wave_scan_f64(v0 + v1, lane);        // prefix up to and including block 2*lane+1
  const double before = inc - (v0 + v1);
  const uint64_t hit = __ballot(inc > thr);
  if (hit == 0) return -1;
  const int hl = __ffsll((unsigned long long)hit) - 1;
  const double bef = __shfl(before, hl, 64), first = __shfl(v0, hl, 64);
  const bool in_first = bef + first > thr;
  double run = in_first ? bef : bef + first;
  for (int jb = (2 * hl + (in_first ? 0 : 1)) * sb; jb < V; jb += kVsChunk) {   // ends inside the block but for rounding
    const int j = jb + 4 * lane;
    const float4 v = load_logits4(x, j, V, vec);
    double w[4] = {weight_of((double)v.x - Md, beta2), weight_of((double)v.y - Md, beta2),
                   weight_of((double)v.z - Md, beta2), weight_of((double)v.w - Md, beta2)};
    for (int r = 0; r < nrm; ++r) {
      const int d = t.rm_tok[r] - j;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (d == e) w[e] = 0.0;
    }
    const double c0 = w[0], c1 = c0 + w[1], c2 = c1 + w[2], c3 = c2 + w[3];
    const double pre = run + (wave_scan_f64(c3, lane) - c3);     // remaining weight before this lane's tokens
    const int e = pre + c0 > thr ? 0 : pre + c1 > thr ? 1 : pre + c2 > thr ? 2 : pre + c3 > thr ? 3 : 4;
    const uint64_t over = __ballot(e < 4 && j + e < V);
    if (over != 0) {
      const int ol = __ffsll((unsigned long long)over) - 1;
      return jb + 4 * ol + __shfl(e, ol, 64);
    }
    run = __shfl(pre + c3, 63, 64);
  }
  return -1;
}

// Rounding left no prefix above the threshold: the last token that still has weight, and if the children covered
// everything the target's most likely token.  By the whole block.
template <int WAVES>
__device__ __forceinline__ int last_resort(const VsTree& t, int nrm, const float* x, double Md, float temperature, int V, int tid) {
  __shared__ int s_last[WAVES];
  __shared__ uint64_t s_key[WAVES];
  const int lane = tid & 63, wv = tid >> 6;
  const double beta = 1.0 / (double)temperature;
  int last = -1;
  uint64_t key = 0;
  for (int j = tid; j < V; j += WAVES * kWave) {
    key = umax64(key, row_key(x[j], j));
    bool live = exp(((double)x[j] - Md) * beta) > 0.0;
    for (int r = 0; r < nrm; ++r)
      if (t.rm_tok[r] == j) live = false;
    if (live) last = max(last, j);
  }
  key = wave_max_u64(key);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) last = max(last, __shfl_xor(last, off, 64));
  if (lane == 0) {
    s_last[wv] = last;
    s_key[wv] = key;
  }
  __syncthreads();
  last = -1;
  key = 0;
#pragma unroll
  for (int i = 0; i < WAVES; ++i) {
    last = max(last, s_last[i]);
    key = umax64(key, s_key[i]);
  }
  return last >= 0 ? last : key_token(key);
}

// ---- one workgroup per sequence makes the sums of the rows it visits --------------------------------------------
__global__ __launch_bounds__(kVsThreads) void verify_sample_kernel(VerifySampleArgs a) {
  __shared__ float s_max[kVsWaves];
  __shared__ double s_sub[kVsSub], s_exp[kVsExpSize];
  __shared__ VsTree t;
  __shared__ int s_next, s_nrm, s_bonus;

  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int T = a.m + 1, V = a.V;
  load_tree(a, b, tid, t);
  load_exp_table(s_exp, tid);
  const int n = min(a.tree.n_sel[b], a.m) + 1;
  StatsPre sp{0, 0u};
  if (tid == 0) sp = stats_begin(a.stats, b, a.B);
  __syncthreads();
  int32_t* path = a.accept_path + (size_t)b * (a.D + 1);
  const int cpb = chunks_per_block(V);
  const int sb = cpb * kVsChunk;                                          // tokens per block
  const int j0 = wv * kVsSubPerWave * sb + 4 * lane;                      // may lie beyond V
  const bool vec = rows_aligned(a);
  const double beta2 = beta2_of(a);

  int cur = 0, len = 0, nrm = 0;
  double Md = 0.0, rem = 0.0;          // nrm, rem: meaningful in wave 0
  const float* x = a.logits;
  if (tid == 0) path[0] = 0;

  for (int it = 0; it <= a.D; ++it) {
    x = a.logits + ((size_t)b * T + cur) * V;
    // wave 0: what the children tests will need (tree indices 1..64; larger trees fetch the rest
    // when they get there), requested now so that it arrives behind the sums
    float kx = 0.0f;
    if (wv == 0 && 1 + lane < n) kx = x[t.tok[1 + lane]];
    // row maximum
    float mx = -__builtin_inff();
#pragma unroll 8
    for (int c = 0; c < kVsSubPerWave * cpb; ++c) mx = max4(mx, load_logits4(x, j0 + c * kVsChunk, V, vec));
    mx = wave_max_f32(mx);
    if (lane == 0) s_max[wv] = mx;
    __syncthreads();
    mx = s_max[0];
#pragma unroll
    for (int i = 1; i < kVsWaves; ++i) mx = fmaxf(mx, s_max[i]);
    Md = (double)mx;
    const float from = short_from(Md, a.span);
    // weights: one sum per block of sb consecutive tokens, in a fixed order
#pragma unroll 1
    for (int i0 = 0; i0 < kVsSubPerWave; i0 += 4) {
      double sums[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        double acc = 0.0;
        for (int c = 0; c < cpb; ++c)
          acc = add_weight4(acc, load_logits4(x, j0 + ((i0 + i) * cpb + c) * kVsChunk, V, vec), Md, beta2, from, s_exp);
        sums[i] = acc;
      }
      const double sum = wave_sums_f64<4>(sums, lane);
      if ((lane & 15) == 0) s_sub[wv * kVsSubPerWave + i0 + (lane >> 4)] = sum;
    }
    __syncthreads();
    if (wv == 0) {
      rem = wave_sum_f64(s_sub[2 * lane] + s_sub[2 * lane + 1]);
      nrm = 0;
      int nxt = -1;
      if (len < a.D)
        nxt = test_children(t, n, lane, rem, nrm, [&](int base, bool& kid, double& kw, double& ku, int& ktok) {
          const int c = base + lane;
          kid = c < n && t.par[c] == cur;
          ktok = c < n ? t.tok[c] : 0;
          if (base > 1) kx = x[ktok];
          ku = c < n ? t.ua[c] : 0.0;
          kw = weight_of((double)kx - Md, beta2);
        });
      if (lane == 0) s_next = nxt;
    }
    __syncthreads();
    const int nxt = s_next;
    if (nxt < 0) break;
    cur = nxt;
    ++len;
    if (tid == 0) path[len] = cur;
  }

  // Bonus token at `cur` (x, Md, s_sub, the rejected tokens describe that node)
  if (wv == 0) {
    const int bonus = draw_bonus(t, nrm, x, Md, beta2, t.ub[cur] * rem, s_sub[2 * lane], s_sub[2 * lane + 1], sb, V, vec, lane);
    if (lane == 0) {
      s_bonus = bonus;
      s_nrm = nrm;
    }
  }
  __syncthreads();
  int bonus = s_bonus;
  if (bonus < 0) bonus = last_resort<kVsWaves>(t, s_nrm, x, Md, a.temperature, V, tid);   // block-uniform branch
  if (tid == 0) {
    for (int i = len + 1; i <= a.D; ++i) path[i] = -1;
    a.accept_len[b] = len;
    a.bonus_token[b] = bonus;
    stats_end(a.stats, sp, a.B, len);
  }
}

// ---- small batches: the sums of the rows by the whole chip, then the walk -----------------------------------------
// A row's 128 blocks belong to kVsParts workgroups of 16 blocks; each takes its weights relative to its own maximum, and
// the walk scales them by exp((part's maximum - row's maximum) / T).
constexpr int kVsParts = 8, kVsPartSub = kVsSub / kVsParts, kVsPartWaves = 4, kVsPartPerWave = kVsPartSub / kVsPartWaves;
constexpr int kVsWalkThreads = 256, kVsWalkWaves = kVsWalkThreads / kWave;
struct VsRow {
  double sub[kVsSub];          // block sums, each relative to its part's maximum
  double psum[kVsParts];       // the parts' sums
  float pmax[kVsParts];        // and maxima
  // of a sequence's first row:
  uint64_t reach[3];           // bit i: row i's sums are needed if the walk leaves the root (verify_root_kernel)
  unsigned arrived;            // the workgroups that have left their part of a leaf's row
  unsigned pad;
};
static_assert(sizeof(VsRow) == 1152, "whole lines");
// Parts of a row that hold tokens (eight from 28 673 tokens up to 32 768, one up to 4096); only those are made and count.
static int vs_parts(int V) {
  const int cpb = (V + kVsSub * kVsChunk - 1) / (kVsSub * kVsChunk), part = kVsPartSub * cpb * kVsChunk;
  return (V + part - 1) / part;
}
static_assert(kVsWalkThreads >= DDD_MMAX + 1, "a thread per tree index");

size_t verify_sample_row_bytes() { return sizeof(VsRow); }

// The 16 block sums of one part of row x, relative to the part's maximum, by a workgroup of four waves.  Returns the maximum; s_sub (LDS)
// holds the sums, and behind the caller's barrier s_sub[] is complete.  CPB: chunks of 256 tokens per block, kept in registers between the
// maximum and the weights (1: V <= 32768, 2: V <= 65536 ...); 0: any V, the logits read twice.
template <int CPB>
__device__ __forceinline__ float part_sums(const VerifySampleArgs& a, const float* x, int part, int tid, float* s_max, double* s_sub,
                                           double* s_exp) {
  const int lane = tid & 63, wv = tid >> 6, V = a.V;
  const int cpb = CPB > 0 ? CPB : chunks_per_block(V);
  const int sb = cpb * kVsChunk;
  const int j0 = (part * kVsPartSub + wv * kVsPartPerWave) * sb + 4 * lane;   // may lie beyond V
  const bool vec = rows_aligned(a);
  const double beta2 = beta2_of(a);
  constexpr int kKeep = CPB > 0 ? CPB : 1;
  constexpr int kHeld = kVsPartPerWave * kKeep;
  float4 xv[kHeld];
  float mx = -__builtin_inff();
  if constexpr (CPB > 0) {
    // No branch at a load, so all of them are in flight together: 16 bytes wherever the row starts, past its end the row's last four.
    // What straddles the end, and what lies behind it, is put right afterwards.
    if (V >= 4) {                                                         // uniform
#pragma unroll
      for (int c = 0; c < kHeld; ++c) {
        const f32x4 v = *reinterpret_cast<const f32x4_of_floats*>(x + min(j0 + c * kVsChunk, V - 4));
        xv[c] = make_float4(v[0], v[1], v[2], v[3]);
      }
    }
#pragma unroll
    for (int c = 0; c < kHeld; ++c) {
      const int j = j0 + c * kVsChunk;
      if (j + 4 > V) xv[c] = load_logits4(x, j, V, false);
    }
#pragma unroll
    for (int c = 0; c < kHeld; ++c) mx = max4(mx, xv[c]);
  } else {
#pragma unroll 8
    for (int c = 0; c < kVsPartPerWave * cpb; ++c) mx = max4(mx, load_logits4(x, j0 + c * kVsChunk, V, vec));
  }
  mx = wave_max_f32(mx);
  if (lane == 0) s_max[wv] = mx;
  load_exp_table(s_exp, tid);
  __syncthreads();
  mx = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
  const bool none = mx == -__builtin_inff();                              // nothing but -inf, or past the vocabulary: no weight
  const double Md = none ? 0.0 : (double)mx;
  const float from = short_from(Md, a.span);
  auto block = [&](int q) {
    double acc = 0.0;
    if constexpr (CPB > 0) {
#pragma unroll
      for (int c = 0; c < kKeep; ++c) acc = add_weight4(acc, xv[q * kKeep + c], Md, beta2, from, s_exp);
    } else {
      for (int c = 0; c < cpb; ++c)
        acc = add_weight4(acc, load_logits4(x, j0 + (q * cpb + c) * kVsChunk, V, vec), Md, beta2, from, s_exp);
    }
    return acc;
  };
  static_assert(kVsPartPerWave == 4, "four blocks");
  // wave_sums_f64<4>, the values by name: an array of them goes to LDS for CPB > 2
  auto half = [&](double lo, double hi, int off) {
    const bool up = (lane & off) != 0;
    return (up ? hi : lo) + __shfl_xor(up ? lo : hi, off, 64);
  };
  const double b0 = block(0), b1 = block(1), b2 = block(2), b3 = block(3);
  const double h0 = half(b0, b2, 32), h1 = half(b1, b3, 32);
  double sum = half(h0, h1, 16);
#pragma unroll
  for (int o = 8; o >= 1; o >>= 1) sum += __shfl_xor(sum, o, 64);
  constexpr int kLanes = kWave / kVsPartPerWave;                          // lanes that hold the same block's sum
  if ((lane & (kLanes - 1)) == 0) s_sub[wv * kVsPartPerWave + lane / kLanes] = sum;
  return mx;
}
// By one thread, behind the barrier: the part's sum, in block order.
__device__ __forceinline__ double part_total(const double* s_sub) {
  double total = 0.0;
  for (int q = 0; q < kVsPartSub; ++q) total += s_sub[q];
  return total;
}

// What another workgroup of the launch left in a row: read past this XCD's L2.
__device__ __forceinline__ double left_f64(const double* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ float left_f32(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// The maximum of a row from its parts', and the row's sum relative to it; parts without tokens were never written.
__device__ __forceinline__ double row_total(float (&pm)[kVsParts], double (&ps)[kVsParts], int parts, double beta2, float& mx) {
#pragma unroll
  for (int p = 0; p < kVsParts; ++p) {
    pm[p] = p < parts ? pm[p] : -__builtin_inff();
    ps[p] = p < parts ? ps[p] : 0.0;
  }
  mx = -__builtin_inff();
#pragma unroll
  for (int p = 0; p < kVsParts; ++p) mx = fmaxf(mx, pm[p]);
  double rem = 0.0;
#pragma unroll
  for (int p = 0; p < kVsParts; ++p) rem = fma(ps[p], weight_of((double)pm[p] - (double)mx, beta2), rem);
  return rem;
}

// By one wave: a part's sums (LDS) and maximum are left to the other workgroups of the launch, then this one is counted; the number of
// those before it, in lane 0.  keep: what else has to be there when it is counted.
__device__ __forceinline__ unsigned leave_part(VsRow& r, int part, const double* s_sub, float mx, unsigned* count, unsigned& keep, int lane) {
  if (lane < kVsPartSub)
    __hip_atomic_store(&r.sub[part * kVsPartSub + lane], s_sub[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const double total = part_total(s_sub);
  if (lane == 0) {
    __hip_atomic_store(&r.psum[part], total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&r.pmax[part], mx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  asm volatile("s_waitcnt vmcnt(0)" : "+v"(keep) : : "memory");           // this wave's stores
  return lane == 0 ? __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
}
// By the workgroup that was counted last.
__device__ __forceinline__ double left_total(const VsRow& r, int parts, double beta2, float& mx) {
  float pm[kVsParts];
  double ps[kVsParts];
#pragma unroll
  for (int p = 0; p < kVsParts; ++p) {
    pm[p] = left_f32(&r.pmax[p]);
    ps[p] = left_f64(&r.psum[p]);
  }
  return row_total(pm, ps, parts, beta2, mx);
}

// The sums of the roots' rows alone, a workgroup per part; the one that is counted last tests the root's children and names the rows that
// the walk can ask for below the one it accepts, for the next launch.
template <int CPB>
__global__ __launch_bounds__(kVsPartWaves * kWave) void verify_root_kernel(VerifySampleArgs a) {
  __shared__ VsTree t;
  __shared__ float s_max[kVsPartWaves];
  __shared__ double s_sub[kVsPartSub], s_exp[kVsExpSize], s_kw[DDD_MMAX + 1];
  __shared__ int s_last, s_child;
  __shared__ bool s_kids[DDD_MMAX + 1];
  const int part = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int T = a.m + 1;
  const int n = min(a.tree.n_sel[b], a.m) + 1;
  const float* x = a.logits + (size_t)b * T * a.V;
  VsRow& r = static_cast<VsRow*>(a.rows)[(size_t)b * T];
  unsigned* const asked = static_cast<unsigned*>(a.rows) - a.B + b;
  const double beta2 = beta2_of(a);
  load_tree(a, b, tid, t);
  const float kx = tid < T ? x[t.tok[tid]] : 0.0f;                        // of the thread's own index: no barrier
  const float mx = part_sums<CPB>(a, x, part, tid, s_max, s_sub, s_exp);
  __syncthreads();
  if (wv == 0) {
    unsigned none = 0u;
    const unsigned before = leave_part(r, part, s_sub, mx, asked, none, lane);
    if (lane == 0) s_last = before == (unsigned)(a.parts - 1);
  }
  __syncthreads();
  if (!s_last) return;                                                    // block-uniform
  float top;   // no line of the row's sums has been read before in this launch: no fence, which would cost 1 to 4 us while others stream
  double rem = left_total(r, a.parts, beta2, top);
  if (tid < T) {
    s_kw[tid] = weight_of((double)kx - (double)top, beta2);
    s_kids[tid] = n <= a.leaf_rows;                                       // then a leaf's sums are made too
  }
  __syncthreads();
  if (tid >= 1 && tid < n && t.par[tid] >= 0 && t.par[tid] < n) s_kids[t.par[tid]] = true;
  if (wv == 0) {
    int nrm = 0;
    const int child = test_children(t, n, lane, rem, nrm, [&](int base, bool& kid, double& kw, double& ku, int& ktok) {
      const int c = base + lane;
      kid = c < n && t.par[c] == 0;
      ktok = c < n ? t.tok[c] : 0;
      ku = c < n ? t.ua[c] : 0.0;
      kw = c < n ? s_kw[c] : 0.0;
    });
    if (lane == 0) s_child = child;
  }
  __syncthreads();
  const int child = s_child;
  bool on = false;                                                        // a node is that child, or below it by no more than the walk goes
  for (int c = tid < n ? tid : -1, d = 0; child > 0 && c > 0 && c < n && d < a.D; c = t.par[c], ++d) on |= c == child;
  const uint64_t bits = __ballot(on && s_kids[tid]);
  if (lane == 0 && wv < 3) r.reach[wv] = bits;
  if (tid == 0) {
    r.arrived = 0u;
    *asked = 0u;
  }
}

template <int CPB>
__global__ __launch_bounds__(kVsPartWaves * kWave) void verify_row_sums_kernel(VerifySampleArgs a) {
  __shared__ float s_max[kVsPartWaves];
  __shared__ double s_sub[kVsPartSub], s_exp[kVsExpSize];
  const int part = blockIdx.x, i = blockIdx.y, b = blockIdx.z, tid = threadIdx.x, lane = tid & 63;
  const int T = a.m + 1, V = a.V;
  // In front of the row's loads: a pool with fewer nodes than m (a round that stopped early) has rows that nobody asks for.  B = 8,
  // V = 32000, m = 60: 10 nodes 15.1 us a call, 36 nodes 16.0, all of 60 21.4; the look itself costs 0.2 (0.4 with the row's address
  // fetched behind it).  So has a leaf of a larger tree, unless the walk ends there (verify_sample_from_sums).
  const int32_t* par = a.tree.parent_idx + (size_t)b * T;
  int p0 = 0, p1 = 0, p2 = 0;
  if (a.leaf_rows < T) {                                                  // uniform
    p0 = par[min(lane, T - 1)];
    p1 = par[min(64 + lane, T - 1)];
    p2 = par[min(128, T - 1)];
  }
  static_assert(DDD_MMAX + 1 <= 129, "three parents per lane");
  const int n = min(a.tree.n_sel[b], a.m) + 1;
  const float* x = a.logits + ((size_t)b * T + i) * V;
  VsRow* out = static_cast<VsRow*>(a.rows) + (size_t)b * T + i;
  asm volatile("" ::"s"(x), "s"(out));                                    // the arguments arrive beside the size, not behind it
  if (i >= n) return;                                                     // uniform: not a node of the tree
  if (n > a.leaf_rows) {                                                  // uniform
    if (i == 0 && part == 0 && tid == 0) out->arrived = 0u;
    const bool kid = (lane >= 1 && lane < n && p0 == i) || (64 + lane < n && p1 == i) || (128 < n && p2 == i);
    if (__ballot(kid) == 0ull) return;                                    // uniform: a leaf
  }
  const float mx = part_sums<CPB>(a, x, part, tid, s_max, s_sub, s_exp);
  __syncthreads();
  if (tid < kVsPartSub) out->sub[part * kVsPartSub + tid] = s_sub[tid];
  if (tid == 0) {
    out->psum[part] = part_total(s_sub);
    out->pmax[part] = mx;
  }
}

// The same for the rows that verify_root_kernel has named, dealt to gridDim.y workgroups per part.  Most rows of a tree are not named, and a
// workgroup for each costs as much where nothing is: 37 sequences, V = 32000, m = 60, nothing / all that 0.65 of the nodes ask for 27.1 and
// 36.4 us a call with 61 workgroups per part, 22.1 and 34.9 with 16; 8 20.1 and 36.1, and 8 sequences with V = 128256 37.9 with 16 and 49.5.
constexpr int kVsReached = 16;
template <int CPB>
__global__ __launch_bounds__(kVsPartWaves * kWave) void verify_reached_sums_kernel(VerifySampleArgs a) {
  __shared__ float s_max[kVsPartWaves];
  __shared__ double s_sub[kVsPartSub], s_exp[kVsExpSize];
  const int part = blockIdx.x, b = blockIdx.z, tid = threadIdx.x, T = a.m + 1;
  VsRow* rows = static_cast<VsRow*>(a.rows) + (size_t)b * T;
  const uint64_t reach[3] = {rows->reach[0], rows->reach[1], rows->reach[2]};
  int turn = blockIdx.y;                                                  // needed rows in front of this workgroup's next one
  // Three copies of the sums: one loop over all bits, half the code, took 0.3 to 1 us longer (32 sequences, V = 32000 33.7 and 34.7).
#pragma unroll
  for (int w = 0; w < 3; ++w)
    for (uint64_t left = reach[w]; left != 0ull; left &= left - 1ull) {   // uniform
      if (turn-- != 0) continue;
      turn = gridDim.y - 1;
      const int i = 64 * w + __ffsll((unsigned long long)left) - 1;
      const float mx = part_sums<CPB>(a, a.logits + ((size_t)b * T + i) * a.V, part, tid, s_max, s_sub, s_exp);
      __syncthreads();
      if (tid < kVsPartSub) rows[i].sub[part * kVsPartSub + tid] = s_sub[tid];
      if (tid == 0) {
        rows[i].psum[part] = part_total(s_sub);
        rows[i].pmax[part] = mx;
      }
    }
}

// The walk over the sums of the rows that have children, by as many workgroups per sequence as a row has parts: all take the same
// decisions, and where the walk ends at a leaf each makes its part of that row.  The one that arrives last draws the bonus token;
// nobody waits.  (Elsewhere the first does, and the others are done.)  CPB as above.
// LEAVES: the leaves' sums are there too, and one workgroup walks; otherwise they are in small trees.  ALL: every part of a row holds tokens.
template <int CPB, bool LEAVES, bool ALL>
__global__ __launch_bounds__(kVsWalkThreads) void verify_sample_from_sums_kernel(VerifySampleArgs a) {
  __shared__ VsTree t;
  __shared__ double s_rem[DDD_MMAX + 1], s_kw[DDD_MMAX + 1];
  __shared__ float s_max[DDD_MMAX + 1], s_pmax[kVsPartWaves];
  __shared__ double s_sub[kVsPartSub], s_exp[kVsExpSize];
  __shared__ int s_cur, s_len, s_leaf, s_nrm, s_bonus;
  const int part = LEAVES ? 0 : blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int T = a.m + 1, V = a.V;
  const int n = min(a.tree.n_sel[b], a.m) + 1;
  const bool missing = !LEAVES && n > a.leaf_rows;                        // the leaves' sums are: uniform
  VsRow* rows = static_cast<VsRow*>(a.rows) + (size_t)b * T;
  const int parts = ALL ? kVsParts : a.parts;
  const double beta2 = beta2_of(a);
  StatsPre sp{0, 0u};
  if (tid == 0 && part == 0) sp = stats_begin(a.stats, b, a.B);
  // thread i: the sums of tree index i's row, and its token's logit in its parent's row
  load_tree(a, b, tid, t);
  float kx = 0.0f;
  if (tid >= 1 && tid < n) kx = a.logits[((size_t)b * T + min(max(t.par[tid], 0), T - 1)) * V + t.tok[tid]];
  if (tid < n) {                                                          // a leaf's (or what is out of reach) were never written, and are not used
    float pm[kVsParts];
    double ps[kVsParts];
#pragma unroll
    for (int p = 0; p < kVsParts; ++p) {
      pm[p] = rows[tid].pmax[p];
      ps[p] = rows[tid].psum[p];
    }
    s_rem[tid] = row_total(pm, ps, parts, beta2, s_max[tid]);
  }
  __syncthreads();
  if (tid >= 1 && tid < n) s_kw[tid] = weight_of((double)kx - (double)s_max[min(max(t.par[tid], 0), T - 1)], beta2);
  __syncthreads();
  int32_t* path = a.accept_path + (size_t)b * (a.D + 1);
  int cur = 0, len = 0, nrm = 0;
  double rem = 0.0;
  if (wv == 0) {
    bool leaf = false;
    if (lane == 0 && part == 0) path[0] = 0;
    for (int it = 0; it <= a.D; ++it) {
      rem = s_rem[cur];
      nrm = 0;
      int nxt = -1;
      if (!LEAVES) {                                                      // as the first launch has seen it, at the depth limit too
        bool kids = false;
        for (int base = 0; base < n; base += kWave) {
          const int c = base + lane;
          kids |= __ballot(c >= 1 && c < n && t.par[c] == cur) != 0ull;
        }
        leaf = missing && !kids;
      }
      if (len < a.D && !leaf)
        nxt = test_children(t, n, lane, rem, nrm, [&](int base, bool& kid, double& kw, double& ku, int& ktok) {
          const int c = base + lane;
          kid = c < n && t.par[c] == cur;
          ktok = c < n ? t.tok[c] : 0;
          ku = c < n ? t.ua[c] : 0.0;
          kw = c < n ? s_kw[c] : 0.0;
        });
      if (nxt < 0) break;
      cur = nxt;
      ++len;
      if (lane == 0 && part == 0) path[len] = cur;
    }
    if (lane == 0) {
      s_cur = cur;
      s_len = len;
      s_leaf = leaf ? 1 : 0;
    }
  }
  __syncthreads();
  cur = s_cur;
  len = s_len;
  const bool leaf = s_leaf != 0;                                          // the same in every workgroup of the sequence
  if (part == 0)
    for (int i = len + 1 + tid; i <= a.D; i += kVsWalkThreads) path[i] = -1;
  const float* x = a.logits + ((size_t)b * T + cur) * V;
  VsRow& r = rows[cur];
  if (!leaf && part != 0) return;                                         // block-uniform
  if (!LEAVES && leaf) {
    const float mx = part_sums<CPB>(a, x, part, tid, s_pmax, s_sub, s_exp);
    __syncthreads();
    if (wv == 0) {
      // sp: the depth that stats_begin has put into the maximum
      const unsigned before = leave_part(r, part, s_sub, mx, &rows[0].arrived, sp.before, lane);
      if (lane == 0) s_leaf = before == (unsigned)(parts - 1) ? 2 : 1;
    }
    __syncthreads();
    if (s_leaf != 2) return;                                              // block-uniform
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");                    // lines of this row that this XCD has read before are old
    if (wv == 0) {
      float top;
      rem = left_total(r, parts, beta2, top);
      if (lane == 0) s_max[cur] = top;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    if (tid == 0 && part != 0 && a.stats.sync != nullptr && a.stats.steps != nullptr) sp.d = min(max(a.stats.steps[b], 0), 31);
  }
  if (wv == 0) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");                // lane 0's list of rejected tokens
    __builtin_amdgcn_wave_barrier();
    const bool held = 2 * lane < kVsPartSub * parts;
    const float pm = LEAVES ? r.pmax[(2 * lane) / kVsPartSub] : left_f32(&r.pmax[(2 * lane) / kVsPartSub]);
    const double scale = weight_of((double)pm - (double)s_max[cur], beta2);
    const double u0 = LEAVES ? r.sub[2 * lane] : left_f64(&r.sub[2 * lane]), u1 = LEAVES ? r.sub[2 * lane + 1] : left_f64(&r.sub[2 * lane + 1]);
    const int bonus = draw_bonus(t, nrm, x, (double)s_max[cur], beta2, t.ub[cur] * rem, held ? u0 * scale : 0.0, held ? u1 * scale : 0.0,
                                 chunks_per_block(V) * kVsChunk, V, rows_aligned(a), lane);
    if (lane == 0) {
      s_nrm = nrm;
      s_bonus = bonus;
    }
  }
  __syncthreads();
  int bonus = s_bonus;
  if (bonus < 0)                                                          // block-uniform
    bonus = last_resort<kVsWalkWaves>(t, s_nrm, x, (double)s_max[cur], a.temperature, V, tid);
  if (tid == 0) {
    a.accept_len[b] = len;
    a.bonus_token[b] = bonus;
    stats_end(a.stats, sp, a.B, len);
  }
}

// Whether the leaves' rows are summed up too.  A walk that ends at a leaf without them takes 4 to 5 us longer, and of a batch's walks one
// usually does where trees are small.  With them and without, us a call: 8 MB of logits 11.9 and 12.3, 16 MB 14.5 and 14.4, 24 MB in rows of
// 16 KB 17.4 and 18.4, 23 MB in rows of 128 KB 17.2 and 16.3, 31 MB 20.8 and 19.7, 47 MB 21.3 and 19.0; trees of 26 nodes 53 MB 21.8 and 23.0,
// of 17 70 MB 24.1 and 23.1.  The more sequences, the surer: from 24 on, 25 MB 17.5 and 19.4, 33 MB 18.9 and 20.5 (25.2 and 26.3 at V = 5000), 38
// MB 20.5 and 21.0, 44 MB 22.3 and 21.5; with fewer about as often the one as the other.
static bool sums_of_leaves(const VerifySampleArgs& a) {
  const long long bytes = (long long)a.B * (a.m + 1) * a.V * 4;
  return bytes <= 24LL << 20 || (a.B >= 24 && bytes <= 38LL << 20) || (a.m <= 32 && bytes <= 64LL << 20);
}
// Where they are not, trees of so many rows have them all the same: a round that stopped after its first call leaves k leaves under the
// root, and every walk that accepts a token ends at one.  Ahead and on demand, V = 32000, m = 60, us a call where every node is accepted: 4
// sequences with 4 / 10 / 20 nodes 11.0 and 13.9, 12.5 and 14.6, 13.2 and 15.0; 8 with 4 / 10 / 20 12.0 and 15.2, 14.2 and 15.4, 16.2 and
// 17.0; 16 with 4 / 10 15.0 and 17.8, 16.0 and 17.7.  Where about half of the tokens are, the walks that end at the root are the longest and
// the rows ahead cost more: 8 sequences with 4 / 10 / 20 nodes 13.0 and 14.8, 16.9 and 15.0, 16.9 and 15.7.  The line, 10 MB, has both in mind.
static int rows_with_leaves(const VerifySampleArgs& a) {
  return sums_of_leaves(a) ? a.m + 1 : (int)((10LL << 20) / ((long long)a.B * a.V * 4));
}

// Whether the roots are decided by a launch of their own.  It takes 8 us and leaves the next one half of the rows where 0.65 of the nodes
// agree and none where the root rejects all its children.  With it and without, 61 nodes, us a call, root alone / one or two rows more / 0.65 of
// the nodes: V = 32000, 18 sequences (134 MiB) 20.3 and 29.5 / 25.6 and 29.3 / 30.1 and 29.9, 32 21.6 and 40.9 / 28.2 and 41.0 / 33.8 and 40.7, 37
// 22.1 and 45.1 / 28.6 and 44.9 / 34.9 and 45.3; V = 128256, 8 26.6 and 41.9 / 38.4 and 41.8 / 37.9 and 40.8.  Below the line two launches are
// as fast where nodes agree (119 MiB 27.7).
static bool roots_first(const VerifySampleArgs& a) { return (long long)a.B * (a.m + 1) * a.V * 4 > 128LL << 20; }

// The launches in front of the walk.
template <int CPB>
static hipError_t launch_sums(const VerifySampleArgs& a, hipStream_t stream) {
  const dim3 wg(kVsPartWaves * kWave);
  if (!roots_first(a)) {
    hipLaunchKernelGGL((verify_row_sums_kernel<CPB>), dim3(a.parts, a.m + 1, a.B), wg, 0, stream, a);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((verify_root_kernel<CPB>), dim3(a.parts, a.B), wg, 0, stream, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((verify_reached_sums_kernel<CPB>), dim3(a.parts, kVsReached, a.B), wg, 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_verify_sample(VerifySampleArgs a, hipStream_t stream) {
  if (a.m > DDD_MMAX) return hipErrorInvalidValue;      // the kernels keep the tree in LDS
  a.beta2 = 1.4426950408889634 / (double)a.temperature;
  a.span = 1000.0 / a.beta2;
  const int cpb = (a.V + kVsSub * kVsChunk - 1) / (kVsSub * kVsChunk);   // chunks of 256 tokens per block
  if (a.rows != nullptr) {
    a.parts = vs_parts(a.V);
    a.leaf_rows = rows_with_leaves(a);
    const bool leaves = a.leaf_rows > a.m;
    hipError_t e = hipSuccess;
    if (cpb == 1)
      e = launch_sums<1>(a, stream);
    else if (cpb == 2)
      e = launch_sums<2>(a, stream);
    else if (cpb == 3)
      e = launch_sums<3>(a, stream);
    else if (cpb == 4)
      e = launch_sums<4>(a, stream);
    else
      e = launch_sums<0>(a, stream);
    if (e != hipSuccess) return e;
    const dim3 walk(leaves ? 1 : a.parts, a.B), wg(kVsWalkThreads);
    if (leaves && a.parts == kVsParts)
      hipLaunchKernelGGL((verify_sample_from_sums_kernel<0, true, true>), walk, wg, 0, stream, a);
    else if (leaves)
      hipLaunchKernelGGL((verify_sample_from_sums_kernel<0, true, false>), walk, wg, 0, stream, a);
    else if (cpb == 1)
      hipLaunchKernelGGL((verify_sample_from_sums_kernel<1, false, false>), walk, wg, 0, stream, a);
    else
      hipLaunchKernelGGL((verify_sample_from_sums_kernel<0, false, false>), walk, wg, 0, stream, a);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(verify_sample_kernel, dim3(a.B), dim3(kVsThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace ddd
