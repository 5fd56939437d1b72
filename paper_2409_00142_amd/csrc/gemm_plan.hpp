// How a linear of the draft layer is cut into work units: column tiles and K ranges by the number of active rows.
#pragma once
#include "ddd_device.hpp"
#include "ddd_kernels.hpp"

namespace ddd {

struct GemmPlan {
  int NT;    // column tiles
  int bpt;   // blocks of 32 active rows per column tile
  int S;     // K ranges
};

// What a product costs with NT column tiles and S ranges of K, in ns (fitted to the LM head's launches of
// 32 to 640 rows): a k tile of a unit costs 140 ns times ab * bb / 2 + 2.5 (its MFMAs, and the copies they do not cover), the
// unit's ramp and stores 140 ns times 25 + 6 ab bb, and every partial sum is read once more by whoever adds them up (4 bytes at
// 5 TB/s).  Returns 0 where the combination does not exist.  Integers: the GEMM and every reader of its sums must come to the same
// number of ranges, whatever the compiler fuses in each of them.
__host__ __device__ inline uint32_t plan_price(const SplitShape& g, int n_act, int NT, int S) {
  const int nblk = (n_act + 31) >> 5, nmt = (g.N + 64 * g.ab - 1) / (64 * g.ab);
  const int bpt = (nblk + NT - 1) / NT, bb = (bpt + 1) >> 1;
  const long long sums = (long long)S * n_act * g.N;
  if (NT > nblk || (NT - 1) * bpt >= nblk || S > g.smax || (S > 1 && (g.kt < 4 * S || sums > g.cap))) return 0u;
  const uint32_t waves = (uint32_t)((nmt * NT * S + g.grid - 1) / g.grid), area = (uint32_t)(g.ab * bb);
  const uint32_t ns = 70u * ((area + 5u) * (uint32_t)((g.kt + S - 1) / S) + 50u + 12u * area);   // of one unit
  const uint64_t price = (uint64_t)waves * ns + (((uint64_t)sums * 3498460u) >> 32);              // sums / 1227.7
  return price < 0xFFFFFFFFu ? (uint32_t)price : 0xFFFFFFFEu;
}
__host__ __device__ inline int plan_least_tiles(const SplitShape& g, int n_act) {
  const int nblk = (n_act + 31) >> 5;
  return (nblk + 2 * g.bbmax - 1) / (2 * g.bbmax);
}

// Called by all 64 lanes of a wave, the same result in every wave of every kernel: lane (i, s) prices the least number of
// column tiles + i and s + 1 K ranges, and the cheapest wins.  The products have a few thousand rows of W for 256
// workgroups: a 4096 x 8192 matrix with 640 rows is 64 tiles of 128 x 320, a quarter of the chip, and four ranges of K
// fill it.  Three calls of the draft layer at H = 4096, F = 11008 with 64, 640 and 384 rows: 1519 -> 1184 us a pass (with tiles of
// 192 rows of W where they are cheaper: 1139).
__device__ __forceinline__ GemmPlan gemm_plan(const SplitShape& g, int n_act, int lane) {
  const int nblk = (n_act + 31) >> 5;
  const int S = (lane >> 3) + 1, NT = plan_least_tiles(g, n_act) + (lane & 7), bpt = (nblk + NT - 1) / NT;
  const uint32_t price = plan_price(g, n_act, NT, S);
  const uint32_t key = price != 0u ? ~price : 0u;
  const uint32_t best = wave_max_u32(key);
  const int l = __ffsll((unsigned long long)__ballot(key == best)) - 1;
  GemmPlan p;
  p.NT = __builtin_amdgcn_readlane(NT, l);
  p.bpt = __builtin_amdgcn_readlane(bpt, l);
  p.S = (l >> 3) + 1;
  return p;
}

}  // namespace ddd
