// Stand-in draft layer: the kernels between two LM-head calls when the draft model's body is a
// real (synthetically weighted) EAGLE-shaped layer instead of a hook (Section 1, EAGLE paragraph:
// token embedding and parent feature -> FC -> one decoder layer -> the target's LM head; EAGLE-2
// paragraph: one input row per beam node, attending to the prompt and to its ancestors).
//
//   linear_stream_kernel   y (+)= x W^T for <= 16 rows: every weight matrix of the layer is read
//                          once per call, so these are HBM weight streams like the LM head
//                          (same streaming waves, plain store epilogue).
//                          Input rows are gathered in place (embedding row of the token, feature row of
//                          the parent).
//   rmsnorm_kernel         bf16(x / sqrt(mean x^2 + eps) * g)
//   body_attention_kernel  RoPE, bf16 key / value store, softmax over prompt + ancestors + self: one workgroup per
//                          (row, head); batched rounds: one per (sequence, head), by ordinary arithmetic
//                          (body_attention_seq_kernel) or with the prompt part on the matrix cores
//                          (body_attention_mfma_kernel)
//   pack_x0_kernel         the FC's input rows assembled for the MFMA path of calls with more than 16 rows
//   The SiLU gate and the final bf16 rounding of the hidden rows ride in the epilogues of the
//   linears that produce their inputs.
// Rows of stopped sequences are skipped; a launch whose rows are all inactive exits at once.
#include "attn_plan.hpp"
#include "body_kernels.hpp"
#include "ddd_device.hpp"
#include "gemm_plan.hpp"
#include "stream_tile.hpp"

namespace ddd {

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float x) {   // finite inputs
  uint32_t u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

typedef u32x4 u32x4_of_halves __attribute__((aligned(2)));   // the caller's prompt values start on any element,
typedef f32x4 f32x4_of_floats __attribute__((aligned(4)));   // its norm weights on any float

// LDS is exchanged, loads from global memory stay in flight (__syncthreads() would wait for them).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Output rows n0 .. n1 - 1 of a weight stream's workgroup: dealt in units of 4.
__device__ __forceinline__ void slice_rows(int N, int nslice, int slice, int& n0, int& n1) {
  const int nq = (N + 3) >> 2;
  n0 = (int)(((long long)slice * nq) / nslice) * 4;
  n1 = min((int)(((long long)(slice + 1) * nq) / nslice) * 4, N);
}

// ---- y (+)= x W^T ----------------------------------------------------------------------------
// MULTI: several K ranges, the last of any number of units; otherwise one whole range, and the input rows stay in registers
// for the whole kernel.
template <int G, bool MULTI>
__global__ __launch_bounds__((kLinearWaves + 1) * 64) void linear_stream_kernel(LinearArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int NW = a.nw;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;

  // In front of the first request for W, though that costs each launch that does run a look at the flags: a launch that every row
  // skips (calls enqueued behind a round's end, most of a captured round's) would read 45 MB for nothing.  Rounds of 3.45 calls with
  // the check behind the first tile and in front of it: 734 and 706 us paced by the host, 1026 and 811 captured; three calls of
  // which none is skipped 395 and 402.
  unsigned long long rows_on = ~0ull;
  // Source row of operand column lane & 15 in each range: on its way with the flags.
  int src[kLinearRanges];
  if (MULTI) {
    const int nr = min(lane & 15, a.R - 1);        // columns past the last row repeat it
#pragma unroll
    for (int g = 0; g < kLinearRanges; ++g) {
      const LinearRange& rg = a.rg[g < a.n_ranges ? g : 0];
      src[g] = nr;
      if (rg.gather_mode == kGatherIndex) src[g] = rg.gather_idx[nr];
      else if (rg.gather_mode == kGatherInBlock) src[g] = (nr / a.gather_k) * a.gather_k + rg.gather_idx[nr];
      else if (rg.gather_mode == kGatherBlock) src[g] = nr / a.gather_k;
    }
  }
  if (a.row_active != nullptr) {   // uniform
    const int on = (lane < a.R) ? a.row_active[lane] : 0;
    rows_on = __ballot(on != 0);
    if (rows_on == 0ull) return;
  }
  const int nslice = gridDim.x, slice = blockIdx.x;
  // Output rows are dealt to the workgroups in units of 4 (an epilogue lane's outputs, and whole gate/up
  // pairs), not in tiles of 16: every workgroup streams the same number of weight rows; a slice's last tile
  // is ragged, its missing rows repeat the slice's last row and are not written.
  int n0, n1;
  slice_rows(a.N, nslice, slice, n0, n1);
  const int nt = (n1 - n0 + 15) >> 4;

  const int NR = MULTI ? a.n_ranges : 1;
  float* red = reinterpret_cast<float*>(smem);      // [2][NR][NW][256] fp32 partial tiles
  unsigned char* stage = smem + 2 * NR * NW * 1024; // [NW][kStageBytes]

  const int total = nt * NR;          // (tile, range) steps of this workgroup, ranges innermost
  // Neighbours start with different ranges: rows of 16 KB whose first halves every workgroup reads at the same time do not reach the
  // whole memory, and a short last range keeps no workgroup waiting at the same moment.  Three calls of one user (H = 4096, F = 11008)
  // 404.3 -> 397.5 us; the down product of ten rows 27.5 -> 25.2.  The ranges are added up in order, which few workgroups, far from the memory's
  // limit, only wait for: 64 of them (N = 1024, K = 11008, ten rows) 13.1 us and 13.9 rotated, 128 (N = 2048, K = 5632) 8.5 both.
  const bool late = MULTI && a.late_rows;
  const int rot = MULTI && nslice >= 192 && !late ? slice % NR : 0;
  auto range_at = [&](int i) { const int r = i + rot; return r < NR ? r : r - NR; };   // 0 <= i < NR

  if (wave < NW) {
    // streaming wave: K-slice [wave*128*G, +128*G) of every range, its share of x resident as B operands
    const int ks = wave * (128 * G);
    const int n = lane & 15, q = lane >> 4;
    const int lrow = lane >> 4, c = lane & 15;
    unsigned char* mystage = stage + wave * kStageBytes;
    const int wr_off = lrow * kStagePitch + c * 16;
    const int rd_off = n * kStagePitch + q * 16;
    const int woff = ks + c * 8;       // this lane's element offset inside a row of any range
    const uint16_t* wb0 = a.rg[range_at(0)].W + woff;
    const int vlast = max(n1 - 1, 0);
    // groups of 128 this wave has in the last range: a whole range unless K ends inside it (MULTI; wave-uniform)
    const int n_last = MULTI ? min(max(a.last_units - wave * G, 0), G) : G;

    u32x4 ring[G][4];
    bf16x8 bfrag[G][4];
    auto x_of = [&](int r) {           // this lane's source row in range r, first element
      const LinearRange& rg = a.rg[r];
      const int from = !MULTI ? min(n, a.R - 1) : r == 0 ? src[0] : r == 1 ? src[1] : src[2];
      return rg.x + (size_t)from * rg.ldx + ks + q * 8;
    };
    const int n_first = (MULTI && range_at(0) == NR - 1) ? n_last : G;
    // Loads return in order, so the input rows of a group follow its weights: the first group can be multiplied, and its weights
    // of the next tile requested, when its own share of the tile and rows (a quarter of them with G = 4) is there.  With the rows behind
    // the whole tile the memory was idle until they had come too: three calls of one user 397.5 -> 385.6 us, gate/up of ten rows 38.8 ->
    // 36.4, q/k/v 23.5 -> 22.4.  (late: see the launch.)
    const uint16_t* xp0 = x_of(range_at(0));
    auto load_x = [&](int g) {
#pragma unroll
      for (int j = 0; j < 4; ++j) bfrag[g][j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(xp0 + g * 128 + j * 32));
    };
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (MULTI && g >= n_first) continue;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = min(n0 + i * 4 + lrow, vlast);
        ring[g][i] = *reinterpret_cast<const u32x4*>(wb0 + (size_t)row * a.ldw + g * 128);
      }
      if (!late) load_x(g);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (late) {
      lds_barrier();
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (MULTI && g >= n_first) continue;
        load_x(g);
      }
    }
#pragma unroll 1
    for (int it = 0; it < total; ++it) {
      __builtin_amdgcn_sched_barrier(0);   // the previous step's operands are dead before the next ones are requested
      const int r = range_at(it % NR), r1 = range_at((it + 1) % NR);
      f32x4 acc;
      const int n_cur = (MULTI && r == NR - 1) ? n_last : G;
      if (it + 1 < total) {          // refill the ring with the next step's tile while this one is consumed
        const uint16_t* wn = a.rg[r1].W + woff;
        const int next_row0 = n0 + ((it + 1) / NR) * 16 + lrow, n_next = (MULTI && r1 == NR - 1) ? n_last : G;
        acc = stream_tile<G, true, MULTI, MULTI>(ring, bfrag, mystage, wr_off, rd_off, wn, a.ldw, next_row0, vlast, n_cur, n_next,
                                                  x_of(r1));
      } else {
        acc = stream_tile<G, false, MULTI>(ring, bfrag, mystage, wr_off, rd_off, wb0, a.ldw, 0, vlast, n_cur);
      }
      *reinterpret_cast<f32x4*>(red + ((((it / NR) & 1) * NR + r) * NW + wave) * 256 + lane * 4) = acc;
      __syncthreads();
    }
  } else {
    // epilogue wave: lane = (vb, r) owns outputs 4*vb .. 4*vb+3 of the tile for input row r
    const int r = lane & 15, vb = lane >> 4;
    const bool active = r < a.R && ((rows_on >> r) & 1ull) != 0;   // rows of stopped sequences stay untouched
    if (late) lds_barrier();
    for (int t = 0; t < nt; ++t) {
      const int v0 = n0 + t * 16 + vb * 4;
      float* const yp = a.y + (size_t)r * a.ldy + v0;
      float y0[4] = {0.f, 0.f, 0.f, 0.f};
      if (a.mode == kLinearAccumulate && active) {   // on their way while the tile is multiplied
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (v0 + e < n1) y0[e] = yp[e];
      }
      // The sums run along K whatever range came first, so an output does not depend on the workgroup that makes it: a range is added
      // when those in front of it have been, the ones that came early (NR - rot of them) behind the tile's last.
      f32x4 s = {0.f, 0.f, 0.f, 0.f};
      const float* tile = red + (t & 1) * NR * NW * 256 + lane * 4;
      for (int i = 0; i < NR; ++i) {
        __syncthreads();
        if (i < NR - rot && rot != 0) continue;
        const int r0 = range_at(i), r1 = i == NR - 1 ? NR : r0 + 1;
#pragma unroll 5   // reads in flight together: down of ten rows 0.4 us
        for (int w = r0 * NW; w < r1 * NW; ++w) s += *reinterpret_cast<const f32x4*>(tile + w * 256);
      }
      if (active) {
        if (a.mode == kLinearSiluPairs) {   // outputs (v0, v0+1) and (v0+2, v0+3) are (gate, up) pairs
#pragma unroll
          for (int e = 0; e < 4; e += 2)
            if (v0 + e + 1 < n1) {
              const float g = s[e], u = s[e + 1];
              a.out16[(size_t)r * a.ld16 + ((v0 + e) >> 1)] = f32_to_bf16_rne(g / (1.0f + __expf(-g)) * u);
            }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (v0 + e < n1) {
              const float y = (a.mode == kLinearAccumulate) ? y0[e] + s[e] : s[e];
              yp[e] = y;
              if (a.out16 != nullptr) {
                const uint16_t yb = f32_to_bf16_rne(y);
                a.out16[(size_t)r * a.ld16 + v0 + e] = yb;
                if (a.out16b != nullptr) a.out16b[(size_t)r * a.ld16 + v0 + e] = yb;
              }
            }
        }
      }
    }
  }
}

template <int G>
static hipError_t launch_linear_g(LinearArgs a, int nslice, hipStream_t stream) {
  // Rows of W whole 16 KB apart and few input rows: these behind all of the first tile, requested when every wave's weights have been, and no
  // rotation.  Late against behind each group, N = 4096, K = 8192, weights from HBM, us: one row 18.5 and 19.7, four 19.0 and 19.8, five 19.1 and
  // 19.75, eight 19.95 and 19.8, ten 20.5 and 19.8; at other pitches late rows are the slower ones (K = 6144, ten rows 15.1 and 14.4).
  a.late_rows = (a.ldw & 8191) == 0 && a.R <= 6;
  const dim3 grid(nslice), block((a.nw + 1) * 64);
  const size_t lds = (size_t)2 * a.n_ranges * a.nw * 1024 + (size_t)a.nw * kStageBytes;
  if (a.n_ranges > 1 || a.last_units < a.nw * G || a.rg[0].gather_mode != kGatherNone)
    hipLaunchKernelGGL((linear_stream_kernel<G, true>), grid, block, lds, stream, a);
  else
    hipLaunchKernelGGL((linear_stream_kernel<G, false>), grid, block, lds, stream, a);
  return hipGetLastError();
}

template <int G>
static hipError_t prepare_linear_g() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&linear_stream_kernel<G, true>), hipFuncAttributeMaxDynamicSharedMemorySize,
                             2 * kLinearRanges * kLinearWaves * 1024 + kLinearWaves * kStageBytes);
}
hipError_t prepare_linear_stream() {
  hipError_t e = prepare_linear_g<1>();
  if (e == hipSuccess) e = prepare_linear_g<2>();
  if (e == hipSuccess) e = prepare_linear_g<4>();
  return e;
}

hipError_t launch_linear_stream(const LinearArgs& a, int G, int nslice, hipStream_t stream) {
  switch (G) {
    case 1: return launch_linear_g<1>(a, nslice, stream);
    case 2: return launch_linear_g<2>(a, nslice, stream);
    case 4: return launch_linear_g<4>(a, nslice, stream);
    default: return hipErrorInvalidValue;
  }
}

// ---- weights ahead ----------------------------------------------------------------------------
// The attention of a few rows leaves most of the chip and the memory idle for 5 to 10 us, and the product behind it is a weight stream
// that starts from nothing.  Workgroups beside its own read what the stream's workgroups start with; workgroup number % 8 is the XCD
// of both, so the stream finds it in its own L2.  (Beside the norms too: 404.1 -> 403.0 us for three calls of one user with k = 10,
// L = 256, H = 4096, F = 11008, but every other size tried lost 0.2 to 0.5 %, up to 2 us.)
__device__ __forceinline__ void read_ahead(const WeightsAhead& w, const uint8_t* row_active, int R, int tid, int threads) {
  if (row_active != nullptr) {   // the stream will not run if every row is inactive
    const int lane = tid & 63;
    if (__ballot(lane < R && row_active[min(lane, R - 1)] != 0) == 0ull) return;
  }
  int n0, n1;
  slice_rows(w.N, w.nslice, (int)blockIdx.x % w.nslice, n0, n1);
  const unsigned char* p = reinterpret_cast<const unsigned char*>(w.W + (size_t)n0 * w.K);
  const int len = (int)min((long long)w.bytes, (long long)(n1 - n0) * w.K * 2);
  for (int i0 = tid * 16; i0 < len; i0 += threads * 64) {
    u32x4 u[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) u[j] = *reinterpret_cast<const u32x4*>(p + min(i0 + j * threads * 16, len - 16));
#pragma unroll
    for (int j = 0; j < 4; ++j) asm volatile("" ::"v"(u[j]));
  }
}

// ---- rmsnorm ----------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void rmsnorm_kernel(RmsNormArgs a) {
  __shared__ float part[16];
  const int r = blockIdx.x, tid = threadIdx.x;
  if (a.row_active != nullptr && a.row_active[r] == 0) return;   // uniform over the block
  const float* x = a.x + (size_t)r * a.H;
  float xv[8], gv[8];                                            // H <= 8192; the weights arrive with the row
  float ss = 0.f;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int i = tid + 1024 * j;
    xv[j] = (i < a.H) ? x[i] : 0.f;
    gv[j] = (i < a.H) ? a.g[i] : 0.f;
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) ss += xv[j] * xv[j];
  ss = wave_sum_f32(ss);
  if ((tid & 63) == 0) part[tid >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < 16; ++w) tot += part[w];                  // fixed order
  const float inv = 1.0f / sqrtf(tot / (float)a.H + 1e-6f);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int i = tid + 1024 * j;
    if (i < a.H) a.out[(size_t)r * a.H + i] = f32_to_bf16_rne(xv[j] * inv * gv[j]);
  }
}

hipError_t launch_rmsnorm(const RmsNormArgs& a, hipStream_t stream) {
  if (a.H > 8192) return hipErrorInvalidValue;
  hipLaunchKernelGGL(rmsnorm_kernel, dim3(a.R), dim3(1024), 0, stream, a);
  return hipGetLastError();
}

// ---- partial sums of a split product added up by their reader --------------------------------------------------
// What a thread needs to read the sums: every value is a few independent loads whose lines lie n_act * N floats apart.
struct SumsView {
  const float* part;
  size_t stride;   // floats between two K ranges
  int N, S;
};
__device__ __forceinline__ int sums_rows(const SplitSums& a) { return a.n_act_ptr != nullptr ? *a.n_act_ptr : a.n_rows; }
// Called by all 64 lanes of a wave.
__device__ __forceinline__ SumsView sums_view(const SplitSums& a, int n_act, int lane) {
  const GemmPlan p = gemm_plan(a.shape, n_act, lane);
  return SumsView{a.part, (size_t)n_act * a.shape.N, a.shape.N, p.S};
}
__device__ __forceinline__ f32x4 sums_at4(const SumsView& v, int n, int col) {   // in the order of the ranges
  const float* p = v.part + (size_t)n * v.N + col;
  f32x4 t[8];
#pragma unroll
  for (int s = 0; s < 8; ++s)
    t[s] = s < v.S ? *reinterpret_cast<const f32x4*>(p + s * v.stride) : f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 y = t[0];
#pragma unroll
  for (int s = 1; s < 8; ++s)
    if (s < v.S) y += t[s];
  return y;
}
__device__ __forceinline__ float sums_at(const SumsView& v, int n, int col) {
  const float* p = v.part + (size_t)n * v.N + col;
  float t[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) t[s] = s < v.S ? p[s * v.stride] : 0.f;
  float y = t[0];
#pragma unroll
  for (int s = 1; s < 8; ++s)
    if (s < v.S) y += t[s];
  return y;
}

// The residual stream behind a split product, and its norm: one workgroup per active row, 16 bytes per load.  Reads
// 4 * (ranges + 1) bytes per element once; the separate accumulating epilogue and norm read and wrote them twice.
__global__ __launch_bounds__(512) void sum_rmsnorm_kernel(SumRmsNormArgs a) {
  __shared__ float part[8];
  const int n = blockIdx.x, tid = threadIdx.x;
  const int n_act = sums_rows(a.sums);
  if (n >= n_act) return;                                        // uniform over the block
  const int r = a.row_list != nullptr ? a.row_list[n] : n;
  const SumsView v = sums_view(a.sums, n_act, tid & 63);
  float* x = a.x + (size_t)r * a.H;
  f32x4 xv[3];                                                   // H <= 5120, a multiple of 128
  float ss = 0.f;
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int i = (tid + 512 * j) * 4;
    xv[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (i < a.H) {
      const f32x4 s = sums_at4(v, n, i);
      xv[j] = a.add ? *reinterpret_cast<const f32x4*>(x + i) + s : s;
      *reinterpret_cast<f32x4*>(x + i) = xv[j];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) ss += xv[j][e] * xv[j][e];
  }
  ss = wave_sum_f32(ss);
  if ((tid & 63) == 0) part[tid >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < 8; ++w) tot += part[w];                   // fixed order
  const float inv = 1.0f / sqrtf(tot / (float)a.H + 1e-6f);
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int i = (tid + 512 * j) * 4;
    if (i < a.H) {
      const f32x4 g = *reinterpret_cast<const f32x4_of_floats*>(a.g + i);
      uint32_t o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = f32_to_bf16_rne(xv[j][e] * inv * g[e]);
      *reinterpret_cast<uint2*>(a.out + (size_t)r * a.H + i) = make_uint2(o[0] | (o[1] << 16), o[2] | (o[3] << 16));
    }
  }
}

hipError_t launch_sum_rmsnorm(const SumRmsNormArgs& a, hipStream_t stream) {
  if (a.H > 3 * 512 * 4) return hipErrorInvalidValue;
  hipLaunchKernelGGL(sum_rmsnorm_kernel, dim3(a.R), dim3(512), 0, stream, a);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void sum_rows_kernel(SumRowsArgs a) {
  const int n = blockIdx.x, tid = threadIdx.x;
  const int n_act = sums_rows(a.sums);
  if (n >= n_act) return;                                        // uniform over the block
  const int r = a.row_list != nullptr ? a.row_list[n] : n;
  const SumsView v = sums_view(a.sums, n_act, tid & 63);
  for (int i = tid * 4; i < v.N; i += 256 * 4) {                 // N is a multiple of 4
    const f32x4 y = *reinterpret_cast<const f32x4*>(a.y + (size_t)r * v.N + i) + sums_at4(v, n, i);
    const uint2 o = make_uint2(f32_to_bf16_rne(y[0]) | ((uint32_t)f32_to_bf16_rne(y[1]) << 16),
                               f32_to_bf16_rne(y[2]) | ((uint32_t)f32_to_bf16_rne(y[3]) << 16));
    *reinterpret_cast<uint2*>(a.out16 + (size_t)r * v.N + i) = o;
    *reinterpret_cast<uint2*>(a.out16b + (size_t)r * v.N + i) = o;
  }
}

hipError_t launch_sum_rows(const SumRowsArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL(sum_rows_kernel, dim3(a.R), dim3(256), 0, stream, a);
  return hipGetLastError();
}

// ---- RoPE + key/value store + tree attention: one workgroup of 8 or 16 waves per (row, head) ----------
// A chain of memory round trips: the first 256 keys and values are in flight while the query is rotated and the ancestors are
// looked up, sixteen threads read a key or value of 256 bytes together (one key per thread, 64 rows in a wave's
// load, and 2-byte reads of the values took 15.3 us for ten rows, 32 heads, L = 256, now 9.4).
constexpr int kAttnKeys = 8;     // keys of a thread in flight

template <int TH>
__device__ __forceinline__ float block_max_f32(float x, float* red, int tid) {
  x = wave_max_f32(x);
  __syncthreads();              // red may still be read from an earlier reduction
  if ((tid & 63) == 0) red[tid >> 6] = x;
  __syncthreads();
  float m = red[0];
#pragma unroll
  for (int w = 1; w < TH / 64; ++w) m = fmaxf(m, red[w]);
  return m;
}
template <int TH>
__device__ __forceinline__ float block_sum_f32(float x, float* red, int tid) {
  x = wave_sum_f32(x);
  __syncthreads();
  if ((tid & 63) == 0) red[tid >> 6] = x;
  __syncthreads();
  float s = 0.f;
#pragma unroll
  for (int w = 0; w < TH / 64; ++w) s += red[w];      // fixed order
  return s;
}

__device__ __forceinline__ SumsView qkv_view(const BodyAttnArgs& a, int lane) {   // by all 64 lanes of a wave
  return a.sums.part != nullptr ? sums_view(a.sums, sums_rows(a.sums), lane) : SumsView{nullptr, 0, 0, 0};
}
// Elements p and p + 64 of the query, key and value of row r, head h.
__device__ __forceinline__ void load_qkv_pair(const BodyAttnArgs& a, const SumsView& v, int r, int h, int p, float& q0, float& q1,
                                              float& k0, float& k1, float& v0, float& v1) {
  const int c = h * kHeadDim + p;
  if (a.sums.part != nullptr) {                                  // uniform: a split product, added up here
    const int n = a.row_pos != nullptr ? a.row_pos[r] : r;
    q0 = sums_at(v, n, c);
    q1 = sums_at(v, n, c + 64);
    k0 = sums_at(v, n, a.H + c);
    k1 = sums_at(v, n, a.H + c + 64);
    v0 = sums_at(v, n, 2 * a.H + c);
    v1 = sums_at(v, n, 2 * a.H + c + 64);
    return;
  }
  const float* row = a.qkv + (size_t)r * 3 * a.H + c;
  q0 = row[0], q1 = row[64];
  k0 = row[a.H], k1 = row[a.H + 64];
  v0 = row[2 * a.H], v1 = row[2 * a.H + 64];
}

__device__ __forceinline__ float row16_sum_f32(float x) {   // over the 16 lanes of a DPP row, the same in all of them
  x += dpp_move_f32<0xB1>(x);
  x += dpp_move_f32<0x4E>(x);
  x += dpp_move_f32<0x141>(x);
  x += dpp_move_f32<0x140>(x);
  return x;
}
__device__ __forceinline__ void unpack_bf16x8(const u32x4& u, float (&f)[8]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f[2 * e] = __uint_as_float(u[e] << 16);
    f[2 * e + 1] = __uint_as_float(u[e] & 0xFFFF0000u);
  }
}

template <int TH>
constexpr int kAttnLdsFloats = 400 + (TH / 64) * kHeadDim;   // in front of the scores

template <int TH>
__global__ __launch_bounds__(TH, 4) void body_attention_kernel(BodyAttnArgs a) {
  extern __shared__ __align__(16) float sm[];
  const int nh = a.H / kHeadDim;
  const int r = blockIdx.x / nh, h = blockIdx.x % nh, tid = threadIdx.x;
  if (r >= a.R) {                  // uniform: workgroups beside the rows'
    read_ahead(a.ahead, a.row_active, a.R, tid, TH);
    return;
  }
  const int b = (a.step == 0) ? r : r / a.k;
  const int n_vis = a.L + a.step + 1;
  float* qs = sm;                  // [128] rotated query
  float* ks = sm + 128;            // [128] own key as stored (bf16 values)
  float* vs = sm + 256;            // [128] own value as stored
  float* red = sm + 384;           // [TH / 64] block reductions
  float* part = sm + 400;          // [TH / 64][128] partial outputs
  float* sc = sm + kAttnLdsFloats<TH>;                                // [n_vis] scores, then weights
  int* anc = reinterpret_cast<int*>(sc + ((n_vis + 3) & ~3));    // [step] row of the ancestor in each earlier call

  // thread (kg, sub): elements sub*8 .. +7 of keys kg, kg + kGroups, ...; the first 256 (512) keys are requested before anything else
  constexpr int kGroups = TH / 16;
  const int kg = tid >> 4, sub = tid & 15;
  const size_t at0 = (size_t)b * a.L * a.H + h * kHeadDim + sub * 8;
  u32x4 kb[kAttnKeys], vb[kAttnKeys];
  auto load_block = [&](const uint16_t* base, int j0, u32x4 (&u)[kAttnKeys]) {
#pragma unroll
    for (int i = 0; i < kAttnKeys; ++i) {
      const int j = j0 + kGroups * i + kg;
      if (j < a.L) u[i] = *reinterpret_cast<const u32x4_of_halves*>(base + at0 + (size_t)j * a.H);
    }
  };
  load_block(a.Kp, 0, kb);
  if (a.row_active != nullptr && a.row_active[r] == 0) return;   // uniform
  const SumsView sv = qkv_view(a, tid & 63);

  if (tid < 64) {
    // pair (tid, tid + 64) of the head rotates by pos * base^(-2*tid/128)
    const float inv_freq = exp2f(-(float)(2 * tid) / (float)kHeadDim * 13.287712379549449f);   // log2(10000)
    float sn, cs;
    sincosf((float)(a.L + a.step) * inv_freq, &sn, &cs);
    float q0, q1, k0, k1, v0, v1;
    load_qkv_pair(a, sv, r, h, tid, q0, q1, k0, k1, v0, v1);
    qs[tid] = q0 * cs - q1 * sn;
    qs[tid + 64] = q1 * cs + q0 * sn;
    const uint16_t kb0 = f32_to_bf16_rne(k0 * cs - k1 * sn), kb1 = f32_to_bf16_rne(k1 * cs + k0 * sn);
    const uint16_t vb0 = f32_to_bf16_rne(v0), vb1 = f32_to_bf16_rne(v1);
    const size_t slot = ((size_t)a.step * a.hist_rows + r) * a.H + h * kHeadDim;
    a.k_hist[slot + tid] = kb0;
    a.k_hist[slot + tid + 64] = kb1;
    a.v_hist[slot + tid] = vb0;
    a.v_hist[slot + tid + 64] = vb1;
    ks[tid] = bf16_to_f32(kb0);
    ks[tid + 64] = bf16_to_f32(kb1);
    vs[tid] = bf16_to_f32(vb0);
    vs[tid + 64] = bf16_to_f32(vb1);
  } else if (tid < 64 + a.step) {   // walk the parent slots back from this row to call number c
    const int c = tid - 64;
    int cur = r;
    for (int s = a.step; s > c; --s) {
      // this call's slots are still in the beam (and are recorded below); earlier calls' were recorded then
      const int pslot = (s == a.step) ? a.beam_parent_slot[cur] : a.par_hist[s * a.hist_rows + cur];
      cur = (s - 1 == 0) ? b : b * a.k + pslot;
    }
    anc[c] = cur;
  } else if (tid == 128 && h == 0 && a.step >= 1) {
    a.par_hist[a.step * a.hist_rows + r] = a.beam_parent_slot[r];
  }
  __builtin_amdgcn_sched_barrier(0);
  load_block(a.Vp, 0, vb);         // ... the values behind the query's registers
  lds_barrier();                   // the loads stay in flight

  // scores: sixteen threads per key
  const float scale = 0.08838834764831845f;   // 1 / sqrt(128)
  float q8[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) q8[e] = qs[sub * 8 + e];
  // ancestor kg (or, as the last, the row itself): at most DDD_DMAX + 1 of them, one per group of sixteen threads
  static_assert(DDD_DMAX + 1 <= kGroups, "one pass over the ancestors");
  float ke[8], ve[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) ke[e] = ve[e] = 0.f;
  if (kg < a.step) {
    const size_t at = ((size_t)kg * a.hist_rows + anc[kg]) * a.H + h * kHeadDim + sub * 8;
    unpack_bf16x8(*reinterpret_cast<const u32x4*>(a.k_hist + at), ke);
    unpack_bf16x8(*reinterpret_cast<const u32x4*>(a.v_hist + at), ve);
  } else if (kg == a.step) {
#pragma unroll
    for (int e = 0; e < 8; ++e) ke[e] = ks[sub * 8 + e], ve[e] = vs[sub * 8 + e];
  }
  float mx = -INFINITY;
  auto score = [&](const float (&f)[8], int j, bool on) {
    float dot = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) dot += q8[e] * f[e];
    dot = row16_sum_f32(dot) * scale;
    if (on) {
      if (sub == 0) sc[j] = dot;
      mx = fmaxf(mx, dot);
    }
  };
  for (int j0 = 0; j0 < a.L; j0 += kGroups * kAttnKeys) {
    if (j0 > 0) load_block(a.Kp, j0, kb);
#pragma unroll
    for (int i = 0; i < kAttnKeys; ++i) {
      const int j = j0 + kGroups * i + kg;
      float f[8];
      unpack_bf16x8(kb[i], f);
      score(f, j, j < a.L);
    }
  }
  score(ke, a.L + kg, kg <= a.step);
  mx = block_max_f32<TH>(mx, red, tid);            // its barriers also publish the scores
  float sum = 0.f;
  for (int j = tid; j < n_vis; j += TH) {
    const float p = __expf(sc[j] - mx);
    sc[j] = p;
    sum += p;
  }
  sum = block_sum_f32<TH>(sum, red, tid);          // ... and these the weights

  // values: the thread's eight elements over its keys, then over the groups
  float o[8];
  const float pe = kg <= a.step ? sc[a.L + kg] : 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = pe * ve[e];
  for (int j0 = 0; j0 < a.L; j0 += kGroups * kAttnKeys) {
    if (j0 > 0) load_block(a.Vp, j0, vb);
#pragma unroll
    for (int i = 0; i < kAttnKeys; ++i) {
      const int j = j0 + kGroups * i + kg;
      if (j < a.L) {
        float f[8];
        unpack_bf16x8(vb[i], f);
        const float p = sc[j];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] += p * f[e];
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    o[e] += __shfl_xor(o[e], 16, 64);
    o[e] += __shfl_xor(o[e], 32, 64);
  }
  if ((tid & 63) < 16) {
#pragma unroll
    for (int e = 0; e < 8; ++e) part[(tid >> 6) * kHeadDim + sub * 8 + e] = o[e];
  }
  __syncthreads();
  if (tid < kHeadDim) {
    float t = 0.f;
#pragma unroll
    for (int g = 0; g < TH / 64; ++g) t += part[g * kHeadDim + tid];   // fixed order
    a.o[(size_t)r * a.H + h * kHeadDim + tid] = f32_to_bf16_rne(t / sum);
  }
}

// ---- rows of [E[token], parent feature] for the GEMM path: one workgroup per row ------------------------------
__global__ __launch_bounds__(256) void pack_x0_kernel(PackX0Args a) {
  const int r = blockIdx.x, tid = threadIdx.x;
  if (r == a.R) {   // one more workgroup beside the rows' (with row_active): the list of active rows
    __shared__ int cnt[4];
    const int lane = tid & 63, wave = tid >> 6;
    int base = 0;
    for (int r0 = 0; r0 < a.R; r0 += 256) {
      const int q = r0 + tid;
      const bool on = q < a.R && a.row_active[q] != 0;
      const unsigned long long m = __ballot(on);
      if (lane == 0) cnt[wave] = __popcll(m);
      __syncthreads();
      int pos = base + __popcll(m & ((1ull << lane) - 1ull));
      for (int w = 0; w < wave; ++w) pos += cnt[w];
      if (on) {
        a.row_list[pos] = q;
        a.row_pos[q] = pos;
      }
      base += cnt[0] + cnt[1] + cnt[2] + cnt[3];
      __syncthreads();                                           // the counts are used again
    }
    if (tid == 0) *a.n_act = base;
    return;
  }
  if (a.row_active != nullptr && a.row_active[r] == 0) return;   // uniform
  int fr = r;
  if (a.feat_mode == kGatherBlock) fr = r / a.k;
  else if (a.feat_mode == kGatherInBlock) fr = (r / a.k) * a.k + a.parent_slot[r];
  const u32x4* e = reinterpret_cast<const u32x4*>(a.E + (size_t)a.token[r] * a.H);
  const u32x4* f = reinterpret_cast<const u32x4*>(a.feat + (size_t)fr * a.H);
  u32x4* out = reinterpret_cast<u32x4*>(a.x0 + (size_t)r * 2 * a.H);
  const int n = a.H / 8;                                         // 16-byte pieces of a half
  for (int i = tid; i < n; i += 256) {
    out[i] = e[i];
    out[n + i] = f[i];
  }
}

hipError_t launch_pack_x0(const PackX0Args& a, hipStream_t stream) {
  hipLaunchKernelGGL(pack_x0_kernel, dim3(a.R + (a.row_active != nullptr ? 1 : 0)), dim3(256), 0, stream, a);
  return hipGetLastError();
}

// ---- the same attention for batched rounds: one workgroup per (sequence, head) ---------------------------------
// The k rows of a sequence share the prompt's keys and values, which are most of what the attention reads: with one
// workgroup per (row, head) they would be fetched k times and the launch would be hundreds of small latency-bound
// workgroups per CU (measured at B = 64, k = 10, L = 256: 510 us per call against 187 us).  Here each prompt key is
// read once and multiplied with all k queries (four threads per key, 32 elements each), each value once and
// weighted into all k outputs.  The arithmetic per row is that of body_attention_kernel (the same products and
// weights; sums in a different but fixed order).
constexpr int kSeqThreads = 1024;

__global__ __launch_bounds__(kSeqThreads) void body_attention_seq_kernel(BodyAttnArgs a) {
  extern __shared__ __align__(16) float sm[];
  const int nh = a.H / kHeadDim;
  const int b = blockIdx.x / nh, h = blockIdx.x % nh, tid = threadIdx.x;
  const int kk = (a.step == 0) ? 1 : a.k;                 // rows of this sequence
  const int r0 = (a.step == 0) ? b : b * a.k;
  if (a.row_active != nullptr && a.row_active[r0] == 0) return;   // uniform: a sequence's rows share their flag
  const SumsView sv = qkv_view(a, tid & 63);
  const int n_vis = a.L + a.step + 1;
  float* qs = sm;                                  // [kSeqRows][128] rotated queries
  float* ks = qs + kSeqRows * kHeadDim;            // [kSeqRows][128] own keys as stored (bf16 values)
  float* vs = ks + kSeqRows * kHeadDim;            // [kSeqRows][128] own values as stored
  float* part = vs + kSeqRows * kHeadDim;          // [8][kSeqRows][128] partial outputs
  float* rsum = part + 8 * kSeqRows * kHeadDim;    // [kSeqRows] sums of the weights
  int* anc = reinterpret_cast<int*>(rsum + kSeqRows);   // [kSeqRows][32] row of the ancestor in each earlier call
  float* sct = reinterpret_cast<float*>(anc + kSeqRows * 32);   // [n_vis][kSeqRows] scores, then weights

  if (tid < kk * 64) {
    // pair (p, p + 64) of the head of row i rotates by pos * base^(-2p/128)
    const int i = tid >> 6, p = tid & 63, r = r0 + i;
    const float inv_freq = exp2f(-(float)(2 * p) / (float)kHeadDim * 13.287712379549449f);   // log2(10000)
    float sn, cs;
    sincosf((float)(a.L + a.step) * inv_freq, &sn, &cs);
    float q0, q1, k0, k1, v0, v1;
    load_qkv_pair(a, sv, r, h, p, q0, q1, k0, k1, v0, v1);
    qs[i * kHeadDim + p] = q0 * cs - q1 * sn;
    qs[i * kHeadDim + p + 64] = q1 * cs + q0 * sn;
    const uint16_t kb0 = f32_to_bf16_rne(k0 * cs - k1 * sn), kb1 = f32_to_bf16_rne(k1 * cs + k0 * sn);
    const uint16_t vb0 = f32_to_bf16_rne(v0), vb1 = f32_to_bf16_rne(v1);
    const size_t slot = ((size_t)a.step * a.hist_rows + r) * a.H + h * kHeadDim;
    a.k_hist[slot + p] = kb0;
    a.k_hist[slot + p + 64] = kb1;
    a.v_hist[slot + p] = vb0;
    a.v_hist[slot + p + 64] = vb1;
    ks[i * kHeadDim + p] = bf16_to_f32(kb0);
    ks[i * kHeadDim + p + 64] = bf16_to_f32(kb1);
    vs[i * kHeadDim + p] = bf16_to_f32(vb0);
    vs[i * kHeadDim + p + 64] = bf16_to_f32(vb1);
  }
  if (tid < kk * 32 && (tid & 31) < a.step) {   // walk the parent slots back from row i to call number c
    const int i = tid >> 5, c = tid & 31;
    int cur = r0 + i;
    for (int s = a.step; s > c; --s) {
      const int pslot = (s == a.step) ? a.beam_parent_slot[cur] : a.par_hist[s * a.hist_rows + cur];
      cur = (s - 1 == 0) ? b : b * a.k + pslot;
    }
    anc[i * 32 + c] = cur;
  }
  if (h == 0 && a.step >= 1 && tid >= 512 && tid < 512 + kk)
    a.par_hist[a.step * a.hist_rows + r0 + tid - 512] = a.beam_parent_slot[r0 + tid - 512];
  __syncthreads();

  // ---- scores.  Prompt keys: four threads per key, 32 elements each, all rows of the sequence ----------------
  const float scale = 0.08838834764831845f;   // 1 / sqrt(128)
  {
    const int qd = tid & 3;
    for (int j = tid >> 2; j < a.L; j += kSeqThreads / 4) {
      const uint16_t* kp = a.Kp + ((size_t)(b * a.L + j) * a.H + h * kHeadDim + qd * 32);
      u32x4 u[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) u[c] = *reinterpret_cast<const u32x4*>(kp + c * 8);
      float kf[32];
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          kf[c * 8 + 2 * e] = __uint_as_float(u[c][e] << 16);
          kf[c * 8 + 2 * e + 1] = __uint_as_float(u[c][e] & 0xFFFF0000u);
        }
      for (int i = 0; i < kk; ++i) {
        const float* q = qs + i * kHeadDim + qd * 32;
        float dot = 0.f;
#pragma unroll
        for (int e = 0; e < 32; ++e) dot += q[e] * kf[e];
        dot += dpp_move_f32<0xB1>(dot);       // the four quarters of the key: lanes ^1, then ^2 (fixed order)
        dot += dpp_move_f32<0x4E>(dot);
        if (qd == 0) sct[j * kSeqRows + i] = dot * scale;
      }
    }
    // the rows' ancestors and themselves: one (row, key) pair per thread
    for (int e = tid; e < kk * (a.step + 1); e += kSeqThreads) {
      const int i = e / (a.step + 1), c = e - i * (a.step + 1);
      float dot = 0.f;
      if (c == a.step) {
        for (int x = 0; x < kHeadDim; ++x) dot += qs[i * kHeadDim + x] * ks[i * kHeadDim + x];
      } else {
        const uint16_t* kp = a.k_hist + (((size_t)c * a.hist_rows + anc[i * 32 + c]) * a.H + h * kHeadDim);
        for (int x = 0; x < kHeadDim; x += 2) {
          const uint32_t w = *reinterpret_cast<const uint32_t*>(kp + x);
          dot += qs[i * kHeadDim + x] * __uint_as_float(w << 16);
          dot += qs[i * kHeadDim + x + 1] * __uint_as_float(w & 0xFFFF0000u);
        }
      }
      sct[(a.L + c) * kSeqRows + i] = dot * scale;
    }
  }
  __syncthreads();
  // ---- softmax weights: wave i takes row i --------------------------------------------------------------------
  {
    const int i = tid >> 6, lane = tid & 63;
    if (i < kk) {
      float mx = -INFINITY;
      for (int j = lane; j < n_vis; j += 64) mx = fmaxf(mx, sct[j * kSeqRows + i]);
      mx = wave_max_f32(mx);
      float sum = 0.f;
      for (int j = lane; j < n_vis; j += 64) {
        const float p = __expf(sct[j * kSeqRows + i] - mx);
        sct[j * kSeqRows + i] = p;
        sum += p;
      }
      sum = wave_sum_f32(sum);
      if (lane == 0) rsum[i] = sum;
    }
  }
  __syncthreads();
  // ---- values: element d of the head, keys grp, grp + 8, ...; every value weighted into all rows ---------------
  const int d = tid & (kHeadDim - 1), grp = tid >> 7;
  float o[kSeqRows];
#pragma unroll
  for (int i = 0; i < kSeqRows; ++i) o[i] = 0.f;
  {
    const uint16_t* vbase = a.Vp + ((size_t)b * a.L * a.H + h * kHeadDim + d);
    int j = grp;
    for (; j + 8 * 7 < a.L; j += 8 * 8) {   // eight keys of this group in flight
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = bf16_to_f32(vbase[(size_t)(j + 8 * u) * a.H]);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const f32x4* w = reinterpret_cast<const f32x4*>(sct + (j + 8 * u) * kSeqRows);
#pragma unroll
        for (int i4 = 0; i4 < kSeqRows / 4; ++i4) {
          const f32x4 ww = w[i4];
#pragma unroll
          for (int e = 0; e < 4; ++e) o[i4 * 4 + e] += ww[e] * v[u];
        }
      }
    }
    for (; j < a.L; j += 8) {
      const float v = bf16_to_f32(vbase[(size_t)j * a.H]);
#pragma unroll
      for (int i = 0; i < kSeqRows; ++i) o[i] += sct[j * kSeqRows + i] * v;
    }
#pragma unroll
    for (int i = 0; i < kSeqRows; ++i)
      if (i < kk) {
        for (int c = grp; c < a.step; c += 8)
          o[i] += sct[(a.L + c) * kSeqRows + i] *
                  bf16_to_f32(a.v_hist[((size_t)c * a.hist_rows + anc[i * 32 + c]) * a.H + h * kHeadDim + d]);
        if (grp == 0) o[i] += sct[(n_vis - 1) * kSeqRows + i] * vs[i * kHeadDim + d];
      }
  }
#pragma unroll
  for (int i = 0; i < kSeqRows; ++i) part[(grp * kSeqRows + i) * kHeadDim + d] = o[i];
  __syncthreads();
  for (int e = tid; e < kk * kHeadDim; e += kSeqThreads) {
    const int i = e >> 7, x = e & (kHeadDim - 1);
    float t = 0.f;
#pragma unroll
    for (int g = 0; g < 8; ++g) t += part[(g * kSeqRows + i) * kHeadDim + x];   // fixed order
    a.o[(size_t)(r0 + i) * a.H + h * kHeadDim + x] = f32_to_bf16_rne(t / rsum[i]);
  }
}

// ---- batched rounds, the prompt part on the matrix cores ---------------------------------------------------------
// One workgroup of four waves per (sequence, head).  The L prompt keys are the same for every row of the sequence, so
// their scores and their part of the output are two small contractions, 16 rows at a time:
//   S[key][row] = sum_d K[key][d] q[row][d]      (v_mfma_f32_16x16x32_bf16: A = 16 keys x 32 d, B = 16 rows x 32 d)
//   O[d][row]   = sum_key V[key][d] p[row][key]  (A = 16 d x 32 keys, B = 16 rows x 32 keys)
// The fp32 operands (rotated queries, softmax weights) go in as two bf16 halves, x = hi + lo with |x - hi - lo| <=
// 2^-17 |x| (two MFMAs per tile), so no rounding point is added to the layer's definition.  Both A operands come
// straight from global memory, 16 bytes per lane.  For the first that is 8 consecutive d of one key, the cache's own
// layout.  The second wants 8 consecutive keys of one d: a lane loads 8 keys' pieces of the same 8 d and turns the
// 8 x 8 block over in its registers (32 byte permutes), and the MFMA that takes its t-th d has the d 8m + t as its row
// m - any 16 of the 128 will do.  A wave then holds all d of its keys, and the waves' sums meet in LDS.  (A copy of the
// values with the keys of an element contiguous, written by every round's prompt call, cost 72 us a round at B = 64,
// L = 256, H = 4096 and as much memory as the values.)  What bounds it: the 268 MB of prompt keys and values at 640 rows,
// 55 us at the rate of a large copy: 62 us for one row per sequence, 88 us for ten (which read 63 MB of partial sums too; 92
// with the copied values).  No operand is staged in LDS, but scores and weights of the whole prompt are: three workgroups share a
// CU up to L = 256, two up to 480, one beyond (attn_plan.hpp).  Each is a chain of dependent steps, and the others' loads run
// under it.  The rows' own keys and their ancestors' (at most
// 32 per row, different from row to row) are handled by ordinary arithmetic.  (With one workgroup per (row, head) the
// launch took 510 us at the 7B shape with 640 rows, with ordinary arithmetic per (sequence, head) 177 us.)
__device__ __forceinline__ void split_bf16x8(const float* x, bool on, bf16x8& hi, bf16x8& lo) {
  u32x4 h, l;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float x0 = on ? x[2 * e] : 0.f, x1 = on ? x[2 * e + 1] : 0.f;
    const uint32_t h0 = f32_to_bf16_rne(x0), h1 = f32_to_bf16_rne(x1);
    const uint32_t l0 = f32_to_bf16_rne(x0 - bf16_to_f32((uint16_t)h0)), l1 = f32_to_bf16_rne(x1 - bf16_to_f32((uint16_t)h1));
    h[e] = h0 | (h1 << 16);
    l[e] = l0 | (l1 << 16);
  }
  hi = __builtin_bit_cast(bf16x8, h);
  lo = __builtin_bit_cast(bf16x8, l);
}

__global__ __launch_bounds__(kMfThreads, 3) void body_attention_mfma_kernel(BodyAttnArgs a) {
  extern __shared__ __align__(16) unsigned char smb[];
  const int nh = a.H / kHeadDim;
  const int b = blockIdx.x / nh, h = blockIdx.x % nh, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kk = (a.step == 0) ? 1 : a.k;                 // rows of this sequence
  const int r0 = (a.step == 0) ? b : b * a.k;
  if (a.row_active != nullptr && a.row_active[r0] == 0) return;   // uniform: a sequence's rows share their flag
  const SumsView sv = qkv_view(a, tid & 63);
  const int L = a.L;
  const MfLds m = mf_lds(L, a.step);
  float* qs = reinterpret_cast<float*>(smb);                     // [kSeqRows][128] rotated queries
  float* rsum = reinterpret_cast<float*>(smb + m.rsum);          // [kSeqRows] sums of the weights
  int* anc = reinterpret_cast<int*>(smb + m.anc);                // [kSeqRows][32] row of the ancestor in each earlier call
  uint16_t* ks = reinterpret_cast<uint16_t*>(smb + m.ks);        // [kSeqRows][128] own keys as stored
  uint16_t* vs = reinterpret_cast<uint16_t*>(smb + m.vs);        // [kSeqRows][128] own values as stored
  float* aw = reinterpret_cast<float*>(smb + m.aw);              // [kSeqRows][step + 1]
  float* sct = reinterpret_cast<float*>(smb + m.sct);            // [kSeqRows][spitch] scores of the prompt keys
  uint16_t* ph = reinterpret_cast<uint16_t*>(smb + m.ph);        // [kSeqRows][ppitch] their weights, high halves
  uint16_t* pl = reinterpret_cast<uint16_t*>(smb + m.pl);        // ... low halves
  float* outs = sct;                                             // [wave][kSeqRows][kMfOutPitch] the prompt's part of the outputs

  // ---- the first 256 prompt keys: requested now, multiplied once the queries are rotated ------------------------
  // lane (row, dq) of the A operand holds 8 consecutive d of key `row` of the tile; tile t belongs to wave t mod 4
  const int ntile = (L + 15) >> 4;
  u32x4 kf[4][4];
  auto load_keys = [&](int t0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int key = min((t0 + wave + 4 * i) * 16 + (lane & 15), L - 1);
      const uint16_t* kp = a.Kp + ((size_t)(b * L + key) * a.H + h * kHeadDim + (lane >> 4) * 8);
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4) kf[i][s4] = *reinterpret_cast<const u32x4*>(kp + s4 * 32);
    }
  };
  load_keys(0);
  // ---- own rows: rotate, store, ancestors (as in the kernels above) -----------------------------------------------
  {
    const int p = tid & 63;                               // every row's pair (p, p + 64) turns by the same angle
    const float inv_freq = exp2f(-(float)(2 * p) / (float)kHeadDim * 13.287712379549449f);   // log2(10000)
    float sn, cs;
    sincosf((float)(L + a.step) * inv_freq, &sn, &cs);
    for (int i0 = wave; i0 < kk; i0 += 2 * kMfWaves) {    // two rows' loads in flight
      float q0[2], q1[2], k0[2], k1[2], v0[2], v1[2];
#pragma unroll
      for (int u = 0; u < 2; ++u)
        load_qkv_pair(a, sv, r0 + min(i0 + u * kMfWaves, kk - 1), h, p, q0[u], q1[u], k0[u], k1[u], v0[u], v1[u]);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int i = i0 + u * kMfWaves;
        if (i >= kk) break;                               // wave-uniform
        qs[i * kHeadDim + p] = q0[u] * cs - q1[u] * sn;
        qs[i * kHeadDim + p + 64] = q1[u] * cs + q0[u] * sn;
        const uint16_t kb0 = f32_to_bf16_rne(k0[u] * cs - k1[u] * sn), kb1 = f32_to_bf16_rne(k1[u] * cs + k0[u] * sn);
        const uint16_t vb0 = f32_to_bf16_rne(v0[u]), vb1 = f32_to_bf16_rne(v1[u]);
        const size_t slot = ((size_t)a.step * a.hist_rows + r0 + i) * a.H + h * kHeadDim;
        a.k_hist[slot + p] = kb0;
        a.k_hist[slot + p + 64] = kb1;
        a.v_hist[slot + p] = vb0;
        a.v_hist[slot + p + 64] = vb1;
        ks[i * kHeadDim + p] = kb0;
        ks[i * kHeadDim + p + 64] = kb1;
        vs[i * kHeadDim + p] = vb0;
        vs[i * kHeadDim + p + 64] = vb1;
      }
    }
  }
  for (int t = tid; t < kk * 32; t += kMfThreads) {   // walk the parent slots back from row i to call number c
    const int i = t >> 5, c = t & 31;
    if (c >= a.step) continue;
    int cur = r0 + i;
    for (int s = a.step; s > c; --s) {
      const int pslot = (s == a.step) ? a.beam_parent_slot[cur] : a.par_hist[s * a.hist_rows + cur];
      cur = (s - 1 == 0) ? b : b * a.k + pslot;
    }
    anc[i * 32 + c] = cur;
  }
  if (h == 0 && a.step >= 1 && tid < kk) a.par_hist[a.step * a.hist_rows + r0 + tid] = a.beam_parent_slot[r0 + tid];
  for (int e = tid; e < kSeqRows * m.ppitch / 2; e += kMfThreads) {   // rows and keys that do not exist weigh nothing
    reinterpret_cast<uint32_t*>(ph)[e] = 0u;
    reinterpret_cast<uint32_t*>(pl)[e] = 0u;
  }
  __syncthreads();

  // ---- scores of the prompt keys ------------------------------------------------------------------------------------
  const float scale = 0.08838834764831845f;   // 1 / sqrt(128)
  const int row = lane & 15, q4 = lane >> 4;  // operand coordinates of the lane (B: row of the sequence; A: key or d)
  {
    bf16x8 qh[4], ql[4];
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) split_bf16x8(qs + row * kHeadDim + s4 * 32 + q4 * 8, row < kk, qh[s4], ql[s4]);
    for (int t0 = 0; t0 < ntile; t0 += 16) {
      if (t0 > 0) load_keys(t0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = t0 + wave + 4 * i;
        if (t >= ntile) continue;                                    // wave-uniform
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
          const bf16x8 kfr = __builtin_bit_cast(bf16x8, kf[i][s4]);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kfr, qh[s4], acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kfr, ql[s4], acc, 0, 0, 0);
        }
        const int key = t * 16 + q4 * 4;                             // accumulator e: key + e of row lane & 15
        if (key < L) *reinterpret_cast<f32x4*>(sct + row * m.spitch + key) = acc * scale;   // spitch holds the last piece
      }
    }
  }
  // ---- the prompt's values for this wave's first two steps of 32 keys: on their way from here on -----------------
  // lane (m, kq) holds, for the 8 keys 32 st + 8 kq + j, the d 8m .. 8m + 7; step st belongs to wave st mod 4
  const int nstep = (L + 31) >> 5;
  u32x4 vf[2][8];
  auto load_values = [&](int st0) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int key = min((st0 + wave + kMfWaves * u) * 32 + q4 * 8 + j, L - 1);
        vf[u][j] = *reinterpret_cast<const u32x4*>(a.Vp + ((size_t)(b * L + key) * a.H + h * kHeadDim + row * 8));
      }
  };
  load_values(0);
  // ---- the rows' ancestors and themselves: four threads per (row, key) pair, 32 elements each ---------------------
  for (int e4 = tid; e4 < kk * (a.step + 1) * 4; e4 += kMfThreads) {
    const int e = e4 >> 2, qd = e4 & 3;
    const int i = e / (a.step + 1), c = e - i * (a.step + 1);
    const uint16_t* kp = (c == a.step) ? ks + i * kHeadDim + qd * 32
                                       : a.k_hist + (((size_t)c * a.hist_rows + anc[i * 32 + c]) * a.H + h * kHeadDim + qd * 32);
    u32x4 u[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) u[x] = *reinterpret_cast<const u32x4*>(kp + x * 8);
    const float* q = qs + i * kHeadDim + qd * 32;
    float dot = 0.f;
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int y = 0; y < 4; ++y) {
        dot += q[x * 8 + 2 * y] * __uint_as_float(u[x][y] << 16);
        dot += q[x * 8 + 2 * y + 1] * __uint_as_float(u[x][y] & 0xFFFF0000u);
      }
    dot += dpp_move_f32<0xB1>(dot);       // the four quarters of the key: lanes ^1, then ^2 (fixed order)
    dot += dpp_move_f32<0x4E>(dot);
    if (qd == 0) aw[e] = dot * scale;
  }
  __syncthreads();
  // ---- softmax weights: wave w takes rows w, w + 4, ...; the prompt's weights as two bf16 halves ------------------
  for (int i = wave; i < kk; i += kMfWaves) {
    const float* sr = sct + i * m.spitch;
    float* ar = aw + i * (a.step + 1);
    float mx = (lane <= a.step) ? ar[lane] : -INFINITY;              // at most DDD_DMAX of them
    for (int j = lane; j < L; j += 64) mx = fmaxf(mx, sr[j]);
    mx = wave_max_f32(mx);
    float sum = 0.f;
    for (int j = lane; j < L; j += 64) {
      const float p = __expf(sr[j] - mx);
      sum += p;
      const uint16_t hi = f32_to_bf16_rne(p);
      ph[i * m.ppitch + j] = hi;
      pl[i * m.ppitch + j] = f32_to_bf16_rne(p - bf16_to_f32(hi));
    }
    if (lane <= a.step) {
      const float p = __expf(ar[lane] - mx);
      sum += p;
      ar[lane] = p;
    }
    sum = wave_sum_f32(sum);
    if (lane == 0) rsum[i] = sum;
  }
  __syncthreads();
  // ---- the prompt's part of the outputs, this wave's keys ----------------------------------------------------------
  {
    f32x4 acc[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int st0 = 0; st0 < nstep; st0 += 2 * kMfWaves) {
      if (st0 > 0) load_values(st0);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int st = st0 + wave + kMfWaves * u;
        if (st >= nstep) continue;                                   // wave-uniform
        // B operand: weights of row `row`, keys 32 st + 8 q4 .. + 7
        const bf16x8 bh = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(ph + row * m.ppitch + st * 32 + q4 * 8));
        const bf16x8 bl = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(pl + row * m.ppitch + st * 32 + q4 * 8));
#pragma unroll
        for (int t = 0; t < 8; ++t) {                                // element t of every key's piece: keys j, j + 1 in a word
          u32x4 f;
#pragma unroll
          for (int x = 0; x < 4; ++x)
            f[x] = __builtin_amdgcn_perm(vf[u][2 * x + 1][t >> 1], vf[u][2 * x][t >> 1], (t & 1) ? 0x07060302u : 0x05040100u);
          const bf16x8 af = __builtin_bit_cast(bf16x8, f);
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bh, acc[t], 0, 0, 0);
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bl, acc[t], 0, 0, 0);
        }
      }
    }
    __syncthreads();                                                 // every wave is done with the scores and the weights
    // accumulator e of tile t: row lane & 15, d = 8 (4 q4 + e) + t
    float* o = outs + (wave * kSeqRows + row) * kMfOutPitch + q4 * 32;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      *reinterpret_cast<f32x4*>(o + e * 8) = f32x4{acc[0][e], acc[1][e], acc[2][e], acc[3][e]};
      *reinterpret_cast<f32x4*>(o + e * 8 + 4) = f32x4{acc[4][e], acc[5][e], acc[6][e], acc[7][e]};
    }
  }
  __syncthreads();
  // ---- ancestors and the row itself, normalisation: the values of four ancestors in flight ------------------------
  {
    const int d = tid & (kHeadDim - 1);
    for (int i = tid >> 7; i < kk; i += kMfThreads / kHeadDim) {
      float o = 0.f;
#pragma unroll
      for (int w = 0; w < kMfWaves; ++w) o += outs[(w * kSeqRows + i) * kMfOutPitch + d];   // fixed order
      const float* ar = aw + i * (a.step + 1);
      const uint16_t* vh = a.v_hist + (size_t)h * kHeadDim + d;
      int c = 0;
      for (; c + 3 < a.step; c += 4) {
        uint16_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = vh[((size_t)(c + u) * a.hist_rows + anc[i * 32 + c + u]) * a.H];
#pragma unroll
        for (int u = 0; u < 4; ++u) o += ar[c + u] * bf16_to_f32(v[u]);
      }
      for (; c < a.step; ++c) o += ar[c] * bf16_to_f32(vh[((size_t)c * a.hist_rows + anc[i * 32 + c]) * a.H]);
      o += ar[a.step] * bf16_to_f32(vs[i * kHeadDim + d]);
      a.o[(size_t)(r0 + i) * a.H + h * kHeadDim + d] = f32_to_bf16_rne(o / rsum[i]);
    }
  }
}

static size_t attention_seq_lds(int n_vis) {
  return (size_t)(3 * kSeqRows * kHeadDim + 8 * kSeqRows * kHeadDim + kSeqRows + kSeqRows * 32 + (size_t)n_vis * kSeqRows) *
         sizeof(float);
}

hipError_t launch_body_attention(const BodyAttnArgs& a, int n_cu, hipStream_t stream) {
  const int n_vis = a.L + a.step + 1;
  // batched rounds with a prompt: one workgroup per (sequence, head), the prompt part on the matrix cores
  if (attention_on_matrix_cores(a.R, a.k, a.L, a.step)) {
    static bool prepared_mf = false;
    if (!prepared_mf) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&body_attention_mfma_kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, kMfLdsMost);
      if (e != hipSuccess) return e;
      prepared_mf = true;
    }
    const int n_seq = (a.step == 0) ? a.R : a.R / a.k;
    hipLaunchKernelGGL(body_attention_mfma_kernel, dim3(n_seq * (a.H / kHeadDim)), dim3(kMfThreads),
                       mf_lds(a.L, a.step).total, stream, a);
    return hipGetLastError();
  }
  // ... with a shorter one or none: the same by ordinary arithmetic
  if (a.R > kBodyRows && a.k <= kSeqRows && attention_seq_lds(n_vis) <= 150 * 1024) {
    static bool prepared = false;
    if (!prepared) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&body_attention_seq_kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024);
      if (e != hipSuccess) return e;
      prepared = true;
    }
    const int n_seq = (a.step == 0) ? a.R : a.R / a.k;
    hipLaunchKernelGGL(body_attention_seq_kernel, dim3(n_seq * (a.H / kHeadDim)), dim3(kSeqThreads),
                       attention_seq_lds(n_vis), stream, a);
    return hipGetLastError();
  }
  // few rows, wider beams, or a prompt too long for the LDS: one workgroup per (row, head)
  // Sixteen waves where a prompt does not fit one pass of eight and the launch has no two workgroups for a CU: 512 keys in flight
  // instead of 256.
  const int n_wg = a.R * (a.H / kHeadDim), tail = ((n_vis + 3) & ~3) + 32;
  // Weights ahead where the attention takes little of the memory itself.  Three calls of one user without and with them: L = 256, H =
  // 4096, ten rows (320 workgroups) 407.2 and 404.1 us; L = 8 400.7 and 397.1; H = 5120, five rows (200) 559.4 and 558.3, ten (400)
  // 584.4 and 585.4; sixteen rows (512) 436.7 and 437.3; sixteen waves, L = 2048, four rows 464.9 and 468.7.
  const bool ahead = a.ahead.W != nullptr && 4 * n_wg <= 5 * n_cu;
  if (a.L > 256 && n_wg <= n_cu)
    hipLaunchKernelGGL(body_attention_kernel<1024>, dim3(n_wg), dim3(1024), (size_t)(kAttnLdsFloats<1024> + tail) * sizeof(float),
                       stream, a);
  else
    hipLaunchKernelGGL(body_attention_kernel<512>, dim3(n_wg + (ahead ? a.ahead.nslice : 0)), dim3(512),
                       (size_t)(kAttnLdsFloats<512> + tail) * sizeof(float), stream, a);
  return hipGetLastError();
}

}  // namespace ddd
