// Streaming-wave building block shared by the weight-stream kernels (LM head, draft-layer
// linears): one 16-row tile of a row-major bf16 matrix against <= 16 resident input rows.
#pragma once
#include "ddd_device.hpp"

namespace ddd {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

constexpr int kStagePitch = 272;               // 256 B of a row group + 16 B pad: conflict-free b128 reads
constexpr int kStageBytes = 16 * kStagePitch;  // one 16x128 bf16 group

__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// One 16-row tile of one streaming wave: drain the register ring group by group through the
// LDS stage into MFMA operands; with REFILL each drained group is reloaded for the next tile.  With RAGGED only the first
// n_cur groups of this tile and the first n_next of the next one exist (wave-uniform).  With REX the next tile belongs to
// another K range: each group's input rows are reloaded too, from xn, behind the MFMAs that
// read them last - requested at the start of the next tile instead, they drained the ring at every range switch.
template <int G, bool REFILL, bool RAGGED = false, bool REX = false>
__device__ __forceinline__ f32x4 stream_tile(u32x4 (&ring)[G][4], bf16x8 (&bfrag)[G][4], unsigned char* mystage,
                                             int wr_off, int rd_off, const uint16_t* wbase, int H, int next_row0,
                                             int vlast, int n_cur = G, int n_next = G, const uint16_t* xn = nullptr) {
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const bool cur = !RAGGED || g < n_cur;
    if (cur) {
#pragma unroll
      for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4*>(mystage + wr_off + i * 4 * kStagePitch) = ring[g][i];
    }
    if (REFILL && (!RAGGED || g < n_next)) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = min(next_row0 + i * 4, vlast);
        ring[g][i] = *reinterpret_cast<const u32x4*>(wbase + (size_t)row * H + g * 128);
      }
    }
    if (cur) {
      wave_lds_fence();
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const u32x4 u = *reinterpret_cast<const u32x4*>(mystage + rd_off + j * 64);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, u), bfrag[g][j], acc, 0, 0, 0);
      }
      wave_lds_fence();
    }
    if (REX) __builtin_amdgcn_sched_barrier(0);   // the group's old operands are dead before the new ones are requested
    if (REX && (!RAGGED || g < n_next)) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        bfrag[g][j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(xn + g * 128 + j * 32));
      }
    }
    if (REX) __builtin_amdgcn_sched_barrier(0);
  }
  return acc;
}

}  // namespace ddd
