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

// Called by all 64 lanes of a wave, the same result in every wave of every kernel: lane (i, s) prices NTmin + i column
// tiles and s + 1 K ranges, and the cheapest wins.  The products have a few thousand rows of W (32 to 172 row tiles of
// 128) for 256 workgroups: a 4096 x 8192 matrix with 640 rows is 64 tiles of 128 x 320, a quarter of the chip, and four
// ranges of K fill it.  Prices, in steps of 0.14 us (fitted to the LM head's launches of 32 to 640 rows): a k tile costs
// bb + 2.5 (copies of the W rows and of 64 bb hidden rows, MFMAs under them), a unit's ramp and its stores 25 + 12 bb, and
// every partial sum is read once more by whoever adds them up (4 bytes at 5 TB/s).  Three calls of the draft layer at
// H = 4096, F = 11008 with 64, 640 and 384 rows: 1519 -> 1184 us a pass.
__device__ __forceinline__ GemmPlan gemm_plan(const SplitShape& g, int n_act, int lane) {
  const int nblk = (n_act + 31) >> 5;
  const int i = lane & 7, S = (lane >> 3) + 1;
  const int NT = (nblk + 2 * g.bbmax - 1) / (2 * g.bbmax) + i;
  const int bpt = (nblk + NT - 1) / NT, bb = (bpt + 1) >> 1;
  const long long sums = (long long)S * n_act * g.N;
  const bool ok = NT <= nblk && S <= g.smax && (S == 1 || (g.kt >= 4 * S && sums <= g.cap)) && (i == 0 || (NT - 1) * bpt < nblk);
  const int waves = (g.nmt * NT * S + g.grid - 1) / g.grid;
  const float price = (float)waves * (((float)bb + 2.5f) * (float)((g.kt + S - 1) / S) + 25.f + 12.f * (float)bb) +
                      (float)sums * (1.f / 171875.f);
  const uint32_t key = ok ? ~__float_as_uint(price) : 0u;      // prices are positive: their bits order like them
  const uint32_t best = wave_max_u32(key);
  const int l = __ffsll((unsigned long long)__ballot(key == best)) - 1;
  GemmPlan p;
  p.NT = __builtin_amdgcn_readlane(NT, l);
  p.bpt = __builtin_amdgcn_readlane(bpt, l);
  p.S = (l >> 3) + 1;
  return p;
}

}  // namespace ddd
