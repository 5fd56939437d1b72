// Tree attention of the verification pass: the consumer of the final tree's mask (Section 1, EAGLE
// paragraph: the whole draft tree goes through the target model in one pass, every node seeing
// the prompt, its ancestors and itself).
//
//   out[i] = sum_j softmax_j(q_i . k_j / sqrt(128)) v_j   over the L prompt keys and the tree keys
//                                                         j with mask[i][j] = 1, per sequence and head
//
// The prompt's keys and values are read once (HBM-bound: 2 * L * 256 bytes per head), so the kernel is a split-key
// ("flash decoding") pass for tiles of 64 queries.  A workgroup of NW = 4 or 8 waves takes NW chunks of 32 keys at a time: every
// wave makes the scores of one chunk, the waves agree on each query's softmax reference through LDS and leave the weights
// there, and then every wave sums its own tile of the output (32 elements of the head for 64 or 32 queries) over all the
// chunks.  No wave's output is merged with another's and a wave holds 16 or 32 accumulators instead of 128: three workgroups
// of four share a CU, so loads fly under other waves' products (64 users, L = 2048: 495 -> 428 us, 5.4 TB/s), and the code of a
// pass is short where it runs once (one user, L = 1999: 27.3 -> 23.8 us).
// Both products run on v_mfma_f32_32x32x16_bf16 in transposed form, which puts one
// query in one lane, so the softmax rescaling is a per-lane scalar:
//   S^T[key][query]  = K[key][d]   Q^T[d][query]     (A = 32 keys x 16 d from the key cache as stored)
//   O^T[d][query]   += V^T[d][key] P^T[key][query]   (A = 32 d x 16 keys from the transposed value cache)
// The accumulator of the first product holds, per lane, keys g*8 + 4*lh + 0..3 (g = 0..3), which is
// not the 8 consecutive keys a B operand wants; the second product simply contracts over the keys
// in that order, by loading V^T as two 4-key pieces per operand.
// Where a head is split over workgroups, a second kernel merges their partials.
#include "ddd_device.hpp"
#include "ddd_kernels.hpp"
#include "tree_attn_plan.hpp"

namespace ddd {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;

constexpr int kAD = 128;        // head dimension
constexpr int kPartFloats = kAD * kQT + 2 * kQT;   // one partial: O^T[128][64], m[64], l[64]
constexpr int kOutPitch = kAD + 4;                 // O[query][d] in LDS at the end: rows padded, 16 bytes aligned
// Waves of a workgroup = chunks of 32 keys of a step: a wave of four sums a quarter of the head for all 64 queries, one of
// eight for half of them.
template <int NW>
struct AttnCfg {
  static constexpr int NQ = 8 / NW;                          // blocks of 32 queries of a wave's output
  static constexpr int kLdsQ = 16 * 64, kLdsP = NW * 8 * 64;   // 16-byte pieces: the queries, the weights of a step (two halves)
  static constexpr int kTile = (kLdsQ + kLdsP) * 16 > kQT * kOutPitch * 4 ? (kLdsQ + kLdsP) * 16 : kQT * kOutPitch * 4;
  static constexpr int kLdsBytes = kTile + NW * kQT * 4;     // ... and the chunks' maxima (in the end: sums) per query
};
constexpr float kLazy = 11.0f;  // how far (in powers of two) a score may exceed a query's softmax reference before it moves

typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef uint32_t u32_of_bytes __attribute__((aligned(1)));   // a row of the mask starts on any byte
typedef f32x4 f32x4_of_floats __attribute__((aligned(4)));   // the caller's output starts on any float
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {   // round to nearest even (one v_cvt_pk_bf16_f32)
  const f32x2 f = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
}

// Operands of one step for one wave.
template <int NW>
struct Operands {
  bf16x8 kf[8];           // its chunk's keys as A operands: lane (l32, lh) holds d = s*16 + lh*8 .. +7 of key c0 + l32
  bf16x8 vf[NW][2];       // every chunk's values for its quarter of the head as A operands: lane (l32, lh) holds, for
                          // d = db*32 + l32 and 16-key step t, the keys c0 + 16t + 4*lh + 0..3 and
                          // c0 + 16t + 8 + 4*lh + 0..3 (the order the first product leaves them in)
};

// Prompt chunks come from the packed cache (fragment order: every operand of a wave is 1 KB of consecutive memory, 16 bytes per
// lane), 512 16-byte pieces of keys and as many of values per chunk.
__device__ __forceinline__ const u32x4* prompt_chunk(const TreeAttnArgs& a, const uint16_t* base, int c, int b, int h) {
  return reinterpret_cast<const u32x4*>(base) + (((size_t)b * a.nh + h) * ((a.L + 31) >> 5) + c) * 512;
}

// Keys of chunk c of the prompt, or of chunk i of the tree, for one wave, and which of the lane's 16 keys count for its two queries:
// bit e of vis as the accumulator registers go.
__device__ __forceinline__ void load_prompt_keys(const TreeAttnArgs& a, int c, int b, int h, int lane, bf16x8 (&kf)[8], uint32_t (&vis)[2]) {
  const u32x4* kp = prompt_chunk(a, a.k_prompt, c, b, h);
#pragma unroll
  for (int s = 0; s < 8; ++s) kf[s] = __builtin_bit_cast(bf16x8, kp[s * 64 + lane]);
  vis[0] = 0u;
#pragma unroll
  for (int e = 0; e < 16; ++e) vis[0] |= (c * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3) < a.L) ? (1u << e) : 0u;
  vis[1] = vis[0];
}
__device__ __forceinline__ void load_tree_keys(const TreeAttnArgs& a, int i, int b, int h, int qt, int lane, bf16x8 (&kf)[8], uint32_t (&vis)[2]) {
  const int l32 = lane & 31, lh = lane >> 5, c0 = i * 32, kj = min(c0 + l32, a.T - 1);
  const uint16_t* kp = a.k_tree + (((size_t)b * a.T + kj) * a.nh + h) * kAD + lh * 8;
#pragma unroll
  for (int s = 0; s < 8; ++s) kf[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(kp + s * 16));
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    const int qi = qt * kQT + qb * 32 + l32;
    const uint8_t* mrow = a.mask + ((size_t)b * a.T + min(qi, a.T - 1)) * a.T;
    vis[qb] = 0u;
    if (a.T >= 4) {                          // four keys a load, the last ones from the row's last four (32 loads of a byte: 1.7 us more)
      uint32_t w[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) w[g] = *reinterpret_cast<const u32_of_bytes*>(mrow + min(c0 + g * 8 + lh * 4, a.T - 4));
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int k0 = c0 + (e >> 2) * 8 + lh * 4, key = k0 + (e & 3);
        const uint32_t on = (w[e >> 2] >> (8 * ((key - min(k0, a.T - 4)) & 3))) & 0xFFu;
        vis[qb] |= (key < a.T && qi < a.T && on != 0u) ? (1u << e) : 0u;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int key = c0 + (e >> 2) * 8 + lh * 4 + (e & 3);
        const uint8_t on = mrow[min(key, a.T - 1)];
        vis[qb] |= (key < a.T && qi < a.T && on != 0) ? (1u << e) : 0u;
      }
    }
  }
}
// Values of chunk c of the prompt, or of chunk i of the tree, for a wave's quarter db of the head.
__device__ __forceinline__ void load_prompt_values(const TreeAttnArgs& a, int c, int b, int h, int db, int lane, bf16x8 (&vf)[2]) {
  const u32x4* vp = prompt_chunk(a, a.v_prompt, c, b, h) + db * 128 + lane;
#pragma unroll
  for (int t = 0; t < 2; ++t) vf[t] = __builtin_bit_cast(bf16x8, vp[t * 64]);
}
__device__ __forceinline__ void load_tree_values(const TreeAttnArgs& a, int i, int b, int h, int db, int lane, bf16x8 (&vf)[2]) {
  const uint16_t* vp = a.vt_tree + (((size_t)b * a.nh + h) * kAD + db * 32 + (lane & 31)) * a.Tp + (lane >> 5) * 4 + i * 32;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const u32x2 lo = *reinterpret_cast<const u32x2*>(vp + t * 16), hi = *reinterpret_cast<const u32x2*>(vp + t * 16 + 8);
    vf[t] = __builtin_bit_cast(bf16x8, u32x4{lo[0], lo[1], hi[0], hi[1]});
  }
}

// A step of prompt keys and tree keys that are not all there (the steps after the whole ones of the prompt).  Chunk ch
// of the step is chunk i = first + ch of the rest: prompt chunks, then the tree's, then nothing.
template <int NW>
__device__ __forceinline__ void load_rest(const TreeAttnArgs& a, int first, int c_rest, int n_prompt, int n_rest, int b, int h,
                                          int qt, int wave, int lane, Operands<NW>& x, uint32_t (&vis)[2]) {
  const int db = wave / (NW / 4), i = first + wave;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  vis[0] = vis[1] = 0u;
  if (i < n_prompt) {
    load_prompt_keys(a, c_rest + i, b, h, lane, x.kf, vis);
  } else if (i < n_rest) {
    load_tree_keys(a, i - n_prompt, b, h, qt, lane, x.kf, vis);
  } else {
#pragma unroll
    for (int s = 0; s < 8; ++s) x.kf[s] = __builtin_bit_cast(bf16x8, zero);
  }
#pragma unroll
  for (int ch = 0; ch < NW; ++ch) {
    const int j = first + ch;                                // uniform
    if (j < n_prompt)
      load_prompt_values(a, c_rest + j, b, h, db, lane, x.vf[ch]);
    else if (j < n_rest)
      load_tree_values(a, j - n_prompt, b, h, db, lane, x.vf[ch]);
    else
      x.vf[ch][0] = x.vf[ch][1] = __builtin_bit_cast(bf16x8, zero);
  }
}

// LDS is exchanged, loads from global memory stay in flight (__syncthreads() would wait for them).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Softmax state of the queries: reference and this wave's share of the sum for the lane's query of both blocks (the
// references are the same in every wave), and the wave's output tile (d = db*32 .., query qb*32 + l32).
template <int NW>
struct QueryState {
  f32x16 o[AttnCfg<NW>::NQ];
  float m[2], l[2];
};

// One step.  NEXT: the operands of the next whole step are requested from kn and vn, each as soon as its register has been used.
template <int NW, bool REST, bool NEXT>
__device__ __forceinline__ void attend_step(Operands<NW>& x, const u32x4* qlds, u32x4* plds, float* cmax_lds,
                                            const uint32_t (&vis)[2], const u32x4* kn, const u32x4* vn, int wave, int lane,
                                            QueryState<NW>& st) {
  // scores are kept in units of ln 2: exp(s - m) = exp2(s' - m') with s' = s * log2(e) / sqrt(128)
  const float scale = 0.08838834764831845f * 1.4426950408889634f;
  const int l32 = lane & 31;
  float sv[2][16];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    f32x16 sacc;
#pragma unroll
    for (int e = 0; e < 16; ++e) sacc[e] = 0.f;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const bf16x8 qf = __builtin_bit_cast(bf16x8, qlds[(qb * 8 + s) * 64 + lane]);
      sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.kf[s], qf, sacc, 0, 0, 0);
      if (NEXT && qb == 1) x.kf[s] = __builtin_bit_cast(bf16x8, kn[s * 64 + lane]);
    }
    // register e of the lane: key c0 + (e>>2)*8 + lh*4 + (e&3), query qb*32 + l32
    float cmax = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      sv[qb][e] = (!REST || ((vis[qb] >> e) & 1u)) ? sacc[e] * scale : -INFINITY;
      cmax = fmaxf(cmax, sv[qb][e]);
    }
    cmax = fmaxf(cmax, __shfl_xor(cmax, 32, 64));            // the other half of the query's keys
    if (lane < 32) cmax_lds[wave * kQT + qb * 32 + l32] = cmax;
  }
  lds_barrier();
  float alpha[2];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    float cmax = cmax_lds[qb * 32 + l32];
#pragma unroll
    for (int w = 1; w < NW; ++w) cmax = fmaxf(cmax, cmax_lds[w * kQT + qb * 32 + l32]);
    // The reference m of a query only moves when a score exceeds it by more than kLazy: until then the
    // weights 2^(s - m) may grow to 2^kLazy (harmless in fp32 and in bf16), and outputs need no rescaling.
    const float m_new = (cmax > st.m[qb] + kLazy || st.m[qb] == -INFINITY) ? cmax : st.m[qb];
    alpha[qb] = (m_new == st.m[qb]) ? 1.f : exp2f(st.m[qb] - m_new);
#pragma unroll
    for (int e = 0; e < 16; ++e) sv[qb][e] = __builtin_amdgcn_exp2f(sv[qb][e] - m_new);   // exp2(-inf) = 0 for hidden keys; m_new
    if (m_new == -INFINITY) {                                  // is finite whenever a key of the query has been seen
#pragma unroll
      for (int e = 0; e < 16; ++e) sv[qb][e] = 0.f;            // nothing visible yet: all weights are zero, not NaN
    }
    // the weights go in as two bf16 halves, hi + lo to 2^-17 relative: rounded to one, relative to a reference that a step's
    // chunks share, they were up to a sixth further from 64 bits than relative to every chunk's own (1.35e-3 against 1.15e-3)
    float psum = 0.f;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      u32x4 hi, lo;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float p0 = sv[qb][8 * t + 2 * i], p1 = sv[qb][8 * t + 2 * i + 1];
        psum += p0 + p1;
        hi[i] = pack_bf16x2(p0, p1);
        lo[i] = pack_bf16x2(p0 - __uint_as_float(hi[i] << 16), p1 - __uint_as_float(hi[i] & 0xFFFF0000u));
      }
      plds[((wave * 2 + qb) * 4 + t) * 64 + lane] = hi;
      plds[((wave * 2 + qb) * 4 + 2 + t) * 64 + lane] = lo;
    }
    st.l[qb] = st.l[qb] * alpha[qb] + psum;
    st.m[qb] = m_new;
  }
  constexpr int NQ = AttnCfg<NW>::NQ;
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const float al = (NQ == 2 ? i == 1 : (wave & 1) != 0) ? alpha[1] : alpha[0];
    if (__any(al != 1.f)) {                                    // uniform
#pragma unroll
      for (int e = 0; e < 16; ++e) st.o[i][e] *= al;
    }
  }
  lds_barrier();
#pragma unroll
  for (int ch = 0; ch < NW; ++ch)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        const int qb = NQ == 2 ? i : (wave & 1);
#pragma unroll
        for (int half = 0; half < 2; ++half)
          st.o[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              x.vf[ch][t], __builtin_bit_cast(bf16x8, plds[((ch * 2 + qb) * 4 + half * 2 + t) * 64 + lane]), st.o[i], 0, 0, 0);
      }
      if (NEXT) x.vf[ch][t] = __builtin_bit_cast(bf16x8, vn[ch * 512 + t * 64 + lane]);
    }
}

// Workgroups of one head get numbers that are equal modulo 8, i.e. one XCD: its query tiles read the keys and
// values through one L2, and the merge finds the partials there (32 heads, L = 1999: one user in one pass 18.9 -> 18.2 us;
// two query tiles, one user 30.3 -> 27.2, sixteen 199 -> 171; one tile and several steps: 17.7 -> 18.0, so not there).
__device__ __forceinline__ void head_on_xcd(int& x, int& h) {
  const int X = gridDim.x, id = x + X * h;
  if ((gridDim.y & 7) != 0) return;
  h = (id & 7) + 8 * (id / (8 * X));
  x = (id >> 3) % X;
}

template <int NW>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 3 : 2) void tree_attn_partial_kernel(TreeAttnArgs a) {
  using C = AttnCfg<NW>;
  __shared__ __align__(16) unsigned char lds[C::kLdsBytes];
  u32x4* qlds = reinterpret_cast<u32x4*>(lds);         // [qb * 8 + s][lane] queries as B operands
  u32x4* plds = qlds + C::kLdsQ;                          // [chunk][qb][half][t][lane] weights as B operands
  float* cmax_lds = reinterpret_cast<float*>(lds + C::kTile);   // [chunk][query]
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
  const int db = wave / (NW / 4);
  const int nqt = (a.T + kQT - 1) / kQT;
  int bx = blockIdx.x, h = blockIdx.y;
  if (nqt > 1) head_on_xcd(bx, h);
  const int split = bx / nqt, qt = bx - split * nqt, b = blockIdx.z;
  const AttnSteps n = attn_steps(a.L, a.T, NW);

  // the first step's operands are on their way while the queries are staged; the workgroup takes steps split, split + nsplit, ...
  int sc = split;
  Operands<NW> x;
  const u32x4 *kp = nullptr, *vp = nullptr;
  uint32_t vis[2];
  if (sc < n.full) {
    kp = prompt_chunk(a, a.k_prompt, sc * NW + wave, b, h);
    vp = prompt_chunk(a, a.v_prompt, sc * NW, b, h) + db * 128;
#pragma unroll
    for (int s = 0; s < 8; ++s) x.kf[s] = __builtin_bit_cast(bf16x8, kp[s * 64 + lane]);
#pragma unroll
    for (int ch = 0; ch < NW; ++ch)
#pragma unroll
      for (int t = 0; t < 2; ++t) x.vf[ch][t] = __builtin_bit_cast(bf16x8, vp[ch * 512 + t * 64 + lane]);
  }
  {
    // lane (l32, lh) holds d = s*16 + lh*8 .. +7 of query qb*32 + l32
    u32x4 u[16 / NW];
#pragma unroll
    for (int i = 0; i < 16 / NW; ++i) {
      const int f = wave * (16 / NW) + i, qi = qt * kQT + (f >> 3) * 32 + l32;
      u[i] = u32x4{0u, 0u, 0u, 0u};
      if (qi < a.T) u[i] = *reinterpret_cast<const u32x4*>(a.q + (((size_t)b * a.T + qi) * a.nh + h) * kAD + lh * 8 + (f & 7) * 16);
    }
#pragma unroll
    for (int i = 0; i < 16 / NW; ++i) qlds[(wave * (16 / NW) + i) * 64 + lane] = u[i];
  }
  QueryState<NW> st;
#pragma unroll
  for (int i = 0; i < C::NQ; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) st.o[i][e] = 0.f;
  st.m[0] = st.m[1] = -INFINITY;
  st.l[0] = st.l[1] = 0.f;
  lds_barrier();

  if (sc < n.full) {
    const size_t stride = (size_t)a.nsplit * NW * 512;
#pragma unroll 1
    for (; sc + a.nsplit < n.full; sc += a.nsplit) {
      kp += stride;
      vp += stride;
      attend_step<NW, false, true>(x, qlds, plds, cmax_lds, vis, kp, vp, wave, lane, st);
    }
    attend_step<NW, false, false>(x, qlds, plds, cmax_lds, vis, nullptr, nullptr, wave, lane, st);
    sc += a.nsplit;
  }
#pragma unroll 1
  for (; sc < n.all; sc += a.nsplit) {
    load_rest<NW>(a, (sc - n.full) * NW, n.full * NW, n.rest_prompt, n.rest, b, h, qt, wave, lane, x, vis);
    attend_step<NW, true, false>(x, qlds, plds, cmax_lds, vis, nullptr, nullptr, wave, lane, st);
  }

  // the waves' shares of the queries' sums
  lds_barrier();
#pragma unroll
  for (int q2 = 0; q2 < 2; ++q2) {
    const float l = st.l[q2] + __shfl_xor(st.l[q2], 32, 64);
    if (lane < 32) cmax_lds[wave * kQT + q2 * 32 + l32] = l;
  }
  lds_barrier();
  float* ol = reinterpret_cast<float*>(lds);             // [query][d]
#pragma unroll
  for (int i = 0; i < C::NQ; ++i) {
    const int qb = C::NQ == 2 ? i : (wave & 1), q = qb * 32 + l32;
    float lsum = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) lsum += cmax_lds[w * kQT + q];   // fixed order
    if (a.nsplit == 1) {
      const float inv = 1.f / lsum;
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<f32x4*>(ol + q * kOutPitch + db * 32 + g * 8 + lh * 4) =
            f32x4{st.o[i][g * 4] * inv, st.o[i][g * 4 + 1] * inv, st.o[i][g * 4 + 2] * inv, st.o[i][g * 4 + 3] * inv};
    } else {
      float* part = a.part + ((((size_t)b * a.nh + h) * nqt + qt) * a.nsplit + split) * kPartFloats + q;
#pragma unroll
      for (int e = 0; e < 16; ++e) part[(db * 32 + (e >> 2) * 8 + lh * 4 + (e & 3)) * kQT] = st.o[i][e];
      if (db == 0 && lane < 32) {
        part[kAD * kQT] = qb != 0 ? st.m[1] : st.m[0];
        part[kAD * kQT + kQT] = lsum;
      }
    }
  }
  if (a.nsplit == 1) {
    // the only partial of its queries: finish here, no merge pass; through LDS, so that whole rows are written
    lds_barrier();
    const int d = (tid & 31) * 4;
#pragma unroll
    for (int q = tid >> 5; q < kQT; q += 2 * NW) {
      const int qi = qt * kQT + q;
      f32x4 v = *reinterpret_cast<const f32x4*>(ol + q * kOutPitch + d);
      if (qi < a.T) {
        if (qi > a.n_sel[b]) v = f32x4{0.f, 0.f, 0.f, 0.f};   // tree indices past n_sel are padding: zero rows
        *reinterpret_cast<f32x4_of_floats*>(a.out + (((size_t)b * a.T + qi) * a.nh + h) * kAD + d) = v;
      }
    }
  }
}

// Few tiles whose heads are a little more than one step of eight waves per workgroup (one user of 32 heads: 65 chunks of 32 keys for
// L = 1999 and eight workgroups a head): a second step for the last chunks costs as much as the first, 5 us of loads, barriers and
// products one after the other.  Here a workgroup takes up to sixteen consecutive chunks in one pass - a wave the scores of two -, so
// there is one reference, and nothing is rescaled.  The keys and the first eight chunks' values are on their way before the first
// product, the other values where the keys were, behind it; a wave that holds a chunk of the tree waits for the mask's words first.
// L = 1999, 32 heads, one user: 24.0 -> 18.9 us with the merge, 1.7 of it by reading the mask four keys at a time.  (Nine workgroups a
// head instead, two to a CU: 26.3.)

__global__ __launch_bounds__(512, 2) void tree_attn_pass_kernel(TreeAttnArgs a, int per) {
  constexpr int NW = 8, kLdsQ = AttnCfg<NW>::kLdsQ;
  __shared__ __align__(16) unsigned char lds[(kLdsQ + kPassChunks * 8 * 64) * 16 + NW * kQT * 4];
  u32x4* qlds = reinterpret_cast<u32x4*>(lds);            // [qb * 8 + s][lane] queries as B operands
  u32x4* plds = qlds + kLdsQ;                             // [chunk][qb][half][t][lane] weights as B operands
  float* cmax_lds = reinterpret_cast<float*>(plds + kPassChunks * 8 * 64);   // [wave][query]
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
  const int db = wave >> 1, nqt = (a.T + kQT - 1) / kQT;
  int bx = blockIdx.x, h = blockIdx.y;
  head_on_xcd(bx, h);
  const int split = bx / nqt, qt = bx - split * nqt, b = blockIdx.z;
  const int n_prompt = (a.L + 31) >> 5, first = split * per, n = min(per, n_prompt + ((a.T + 31) >> 5) - first);   // >= 1 chunks

  bf16x8 kf[2][8], vf[kPassChunks][2];
  uint32_t vis[2][2] = {{0u, 0u}, {0u, 0u}};
  auto load_values = [&](int ch) {                        // ch < n is uniform
    if (ch < n) {
      if (first + ch < n_prompt)
        load_prompt_values(a, first + ch, b, h, db, lane, vf[ch]);
      else
        load_tree_values(a, first + ch - n_prompt, b, h, db, lane, vf[ch]);
    }
  };
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int c = first + wave + NW * u;
    if (wave + NW * u < n) {                              // wave-uniform
      if (c < n_prompt)
        load_prompt_keys(a, c, b, h, lane, kf[u], vis[u]);
      else
        load_tree_keys(a, c - n_prompt, b, h, qt, lane, kf[u], vis[u]);
    }
  }
#pragma unroll
  for (int ch = 0; ch < NW; ++ch) load_values(ch);
  {
    // lane (l32, lh) holds d = s*16 + lh*8 .. +7 of query qb*32 + l32
    u32x4 q[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int f = wave * 2 + i, qi = qt * kQT + (f >> 3) * 32 + l32;
      q[i] = u32x4{0u, 0u, 0u, 0u};
      if (qi < a.T) q[i] = *reinterpret_cast<const u32x4*>(a.q + (((size_t)b * a.T + qi) * a.nh + h) * kAD + lh * 8 + (f & 7) * 16);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) qlds[(wave * 2 + i) * 64 + lane] = q[i];
  }
  lds_barrier();

  const float scale = 0.08838834764831845f * 1.4426950408889634f;   // scores in units of ln 2
  float sv[2][2][16], cmax[2] = {-INFINITY, -INFINITY};
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      if (wave + NW * u >= n) continue;                   // wave-uniform
      f32x16 acc;
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
      for (int s = 0; s < 8; ++s)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[u][s], __builtin_bit_cast(bf16x8, qlds[(qb * 8 + s) * 64 + lane]), acc, 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        sv[u][qb][e] = ((vis[u][qb] >> e) & 1u) ? acc[e] * scale : -INFINITY;
        cmax[qb] = fmaxf(cmax[qb], sv[u][qb][e]);
      }
    }
#pragma unroll
  for (int ch = NW; ch < kPassChunks; ++ch) load_values(ch);   // where the keys were
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    const float m = fmaxf(cmax[qb], __shfl_xor(cmax[qb], 32, 64));   // the other half of the query's keys
    if (lane < 32) cmax_lds[wave * kQT + qb * 32 + l32] = m;
  }
  lds_barrier();
  float m[2], l[2] = {0.f, 0.f};
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    m[qb] = cmax_lds[qb * 32 + l32];
#pragma unroll
    for (int w = 1; w < NW; ++w) m[qb] = fmaxf(m[qb], cmax_lds[w * kQT + qb * 32 + l32]);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (wave + NW * u >= n) continue;
      // the weights go in as two bf16 halves, hi + lo to 2^-17 relative (attend_step)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        u32x4 hi, lo;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float p0 = __builtin_amdgcn_exp2f(sv[u][qb][8 * t + 2 * i] - m[qb]), p1 = __builtin_amdgcn_exp2f(sv[u][qb][8 * t + 2 * i + 1] - m[qb]);
          if (m[qb] == -INFINITY) p0 = p1 = 0.f;          // nothing visible: all weights are zero, not NaN
          l[qb] += p0 + p1;
          hi[i] = pack_bf16x2(p0, p1);
          lo[i] = pack_bf16x2(p0 - __uint_as_float(hi[i] << 16), p1 - __uint_as_float(hi[i] & 0xFFFF0000u));
        }
        plds[(((wave + NW * u) * 2 + qb) * 4 + t) * 64 + lane] = hi;
        plds[(((wave + NW * u) * 2 + qb) * 4 + 2 + t) * 64 + lane] = lo;
      }
    }
  }
  lds_barrier();                                          // the weights are there, and the maxima have been read
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    const float s = l[qb] + __shfl_xor(l[qb], 32, 64);
    if (lane < 32) cmax_lds[wave * kQT + qb * 32 + l32] = s;
  }
  f32x16 o;
#pragma unroll
  for (int e = 0; e < 16; ++e) o[e] = 0.f;
  const int qb = wave & 1, q = qb * 32 + l32;
#pragma unroll
  for (int ch = 0; ch < kPassChunks; ++ch) {
    if (ch >= n) continue;                                // uniform
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int half = 0; half < 2; ++half)
        o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            vf[ch][t], __builtin_bit_cast(bf16x8, plds[((ch * 2 + qb) * 4 + half * 2 + t) * 64 + lane]), o, 0, 0, 0);
  }
  lds_barrier();
  float lsum = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) lsum += cmax_lds[w * kQT + q];   // fixed order
  float* part = a.part + ((((size_t)b * a.nh + h) * nqt + qt) * a.nsplit + split) * kPartFloats + q;
#pragma unroll
  for (int e = 0; e < 16; ++e) part[(db * 32 + (e >> 2) * 8 + lh * 4 + (e & 3)) * kQT] = o[e];
  if (db == 0 && lane < 32) {
    part[kAD * kQT] = qb != 0 ? m[1] : m[0];
    part[kAD * kQT + kQT] = lsum;
  }
}

// Merge of the workgroups' partials: one workgroup per (query tile x eighth of the head, head, sequence).  Every thread asks for
// its partials eight at a time, the references and sums together with the outputs: one or two memory latencies in all.
constexpr int kMergeD = 16;   // elements of the head per workgroup

// MAPPED: the workgroups of a head on one XCD, where the partials' were (elsewhere it costs 0.2 us: 32 heads, L = 300 to 1500, 17 tree
// indices 11.4 to 14.4 us against 11.2 to 14.2).
template <bool MAPPED>
__global__ __launch_bounds__(256) void tree_attn_merge_kernel(TreeAttnArgs a) {
  const int nqt = (a.T + kQT - 1) / kQT;
  int bx = blockIdx.x, h = blockIdx.y;
  if (MAPPED) head_on_xcd(bx, h);
  const int qt = bx / (kAD / kMergeD), dq0 = (bx % (kAD / kMergeD)) * kMergeD, b = blockIdx.z, tid = threadIdx.x;
  const float* part = a.part + (((size_t)b * a.nh + h) * nqt + qt) * a.nsplit * kPartFloats;
  const int qx = tid & (kQT - 1), qi = qt * kQT + qx;
  if (qi >= a.T) return;
  const float* pm = part + kAD * kQT + qx;                         // reference of partial p at pm[p * kPartFloats], its sum kQT on
  const float* po = part + (size_t)(dq0 + (tid >> 6)) * kQT + qx;
  constexpr int kRows = kMergeD / 4;
  float M = -INFINITY, den = 0.f, num[kRows];
#pragma unroll
  for (int i = 0; i < kRows; ++i) num[i] = 0.f;
  for (int p0 = 0; p0 < a.nsplit; p0 += 8) {                       // fixed order
    float m8[8], l8[8], o8[8][kRows];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const size_t at = (size_t)min(p0 + j, a.nsplit - 1) * kPartFloats;
      m8[j] = pm[at];
      l8[j] = pm[at + kQT];
#pragma unroll
      for (int i = 0; i < kRows; ++i) o8[j][i] = po[at + (size_t)4 * i * kQT];
      if (p0 + j >= a.nsplit) m8[j] = -INFINITY;
    }
    float M2 = M;
#pragma unroll
    for (int j = 0; j < 8; ++j) M2 = fmaxf(M2, m8[j]);
    const float w = (M == -INFINITY) ? 0.f : exp2f(M - M2);
    M = M2;
    den *= w;
#pragma unroll
    for (int i = 0; i < kRows; ++i) num[i] *= w;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float wj = (m8[j] == -INFINITY) ? 0.f : exp2f(m8[j] - M);
      den += wj * l8[j];
#pragma unroll
      for (int i = 0; i < kRows; ++i) num[i] += wj * o8[j][i];
    }
  }
  const bool live = qi <= a.n_sel[b];     // tree indices past n_sel are padding: zero rows
  float* orow = a.out + (((size_t)b * a.T + qi) * a.nh + h) * kAD;
#pragma unroll
  for (int i = 0; i < kRows; ++i) orow[dq0 + (tid >> 6) + 4 * i] = live ? num[i] / den : 0.f;
}

// Prompt cache in fragment order: per (sequence, head, chunk of 32 keys) 8 KB of keys, [s][lane] x 8 bf16 =
// K[key c*32 + l32][d s*16 + lh*8 + 0..7], and 8 KB of values, [db*2 + t][lane] x 8 bf16 =
// V[key c*32 + 16t + 4*lh + 0..3, then c*32 + 16t + 8 + 4*lh + 0..3][d db*32 + l32]; keys past L are zero.
__global__ __launch_bounds__(64) void kv_pack_kernel(const uint16_t* k, const uint16_t* v, uint16_t* kp, uint16_t* vp,
                                                     int L, int nh) {
  const int c = blockIdx.x, h = blockIdx.y, b = blockIdx.z, lane = threadIdx.x, l32 = lane & 31, lh = lane >> 5;
  const int ncp = gridDim.x;
  const size_t blk = (((size_t)b * nh + h) * ncp + c) * 8 * 64 * 8;   // in bf16 elements
  const int key = c * 32 + l32;
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    u32x4 u = {0u, 0u, 0u, 0u};
    if (key < L) u = *reinterpret_cast<const u32x4*>(k + (((size_t)b * L + key) * nh + h) * kAD + s * 16 + lh * 8);
    *reinterpret_cast<u32x4*>(kp + blk + ((size_t)s * 64 + lane) * 8) = u;
  }
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      uint16_t e[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int kk = c * 32 + 16 * t + (i >> 2) * 8 + 4 * lh + (i & 3);
        e[i] = (kk < L) ? v[(((size_t)b * L + kk) * nh + h) * kAD + db * 32 + l32] : (uint16_t)0;
      }
      const u32x4 u = {(uint32_t)e[0] | ((uint32_t)e[1] << 16), (uint32_t)e[2] | ((uint32_t)e[3] << 16),
                       (uint32_t)e[4] | ((uint32_t)e[5] << 16), (uint32_t)e[6] | ((uint32_t)e[7] << 16)};
      *reinterpret_cast<u32x4*>(vp + blk + ((size_t)(db * 2 + t) * 64 + lane) * 8) = u;
    }
}

hipError_t launch_kv_pack(const uint16_t* k, const uint16_t* v, uint16_t* kp, uint16_t* vp, int B, int L, int nh,
                          hipStream_t stream) {
  if (L <= 0) return hipSuccess;
  hipLaunchKernelGGL(kv_pack_kernel, dim3((L + 31) / 32, nh, B), dim3(64), 0, stream, k, v, kp, vp, L, nh);
  return hipGetLastError();
}

size_t tree_attention_part_floats() { return (size_t)kPartFloats; }

hipError_t launch_tree_attention(TreeAttnArgs a, int n_cu, hipStream_t stream) {
  const AttnLaunch p = attn_launch(a.B, a.nh, a.T, a.L, n_cu);
  a.nsplit = p.nsplit;
  const int nqt = (a.T + kQT - 1) / kQT;
  const dim3 grid(a.nsplit * nqt, a.nh, a.B);
  if (p.per > 0)
    hipLaunchKernelGGL(tree_attn_pass_kernel, grid, dim3(512), 0, stream, a, p.per);
  else if (p.nw == 8)
    hipLaunchKernelGGL(tree_attn_partial_kernel<8>, grid, dim3(64 * 8), 0, stream, a);
  else
    hipLaunchKernelGGL(tree_attn_partial_kernel<4>, grid, dim3(64 * 4), 0, stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.nsplit == 1) return e;
  const dim3 merge(nqt * (kAD / kMergeD), a.nh, a.B);
  if (p.per > 0 || nqt > 1)
    hipLaunchKernelGGL(tree_attn_merge_kernel<true>, merge, dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL(tree_attn_merge_kernel<false>, merge, dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace ddd
