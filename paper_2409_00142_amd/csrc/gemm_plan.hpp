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

// How the LM head's GEMM is cut: row tiles of 128 or 256 rows of W, NT column tiles.
struct HeadPlan {
  int bm;    // rows of W per tile
  int NT;    // column tiles
  int bpt;   // most blocks of 32 active rows of one
};
struct HeadShape {
  int V, kt, grid;
  int most;     // most blocks of 32 active rows beside a 256-row tile
  float row;    // ns in which the whole chip receives a k tile of one row of W (128 bytes) with 128-row tiles,
  float row2;   // with 256-row tiles
  float once;   // what a cut of one pass costs beside one of several: calls that walk W in opposite directions find in the memory-side
                // cache what the call before read last, but a single pass reads all rows at once, along k
  int once_most;   // ... in calls of up to so many blocks of 32 rows: with more the products take longer than W
};
// In ns, fitted to 900 calls of 20 to 640 rows with V = 4000 to 128256 and H = 1024 to 5120, walking W in one direction and in
// alternating ones, each with up to ten cuts (the chosen cut is 0.65 % slower than the best one on average; with whole passes at the
// chip's rate 2 %, and 37 % at most).  Either the workgroups' passes over the units: a unit's ramp and epilogue are 250 and 210 per
// 32 x 32 products (block columns in twos: two waves share them) or 3600 and 150, a k tile of it 305 and 26 per 32 x 32, or what its
// rows of W take to arrive, 1 us per 256 rows, which the column tiles share.  Or, if that is longer, the stream of W through the chip,
// by the rows that there are - a last pass that is nearly empty streams as little -, and nearly once more for each further column
// tile: 40 rows at V = 100000, H = 4096 take 200 us with one, 227 with two.  Returns 0 where the combination does not exist.
__host__ __device__ inline float head_price(const HeadShape& h, int n_act, int bm, int NT) {
  const int nblk = (n_act + 31) >> 5, bpt = (int)((unsigned)(nblk + NT - 1) / (unsigned)NT);
  if (NT > nblk || bpt > (bm == 256 ? h.most : 10)) return 0.f;                                    // tiles of at most 320 rows
  const int nmt = bm == 256 ? (h.V + 255) >> 8 : (h.V + 127) >> 7, passes = (int)((unsigned)(nmt * NT + h.grid - 1) / (unsigned)h.grid);
  const float area = (float)((bm >> 5) * ((bpt + 1) & ~1));
  const float step = 305.f + 26.f * area, feed = 3.75f * (float)bm / (float)NT;
  const float unit = (bm == 256 ? 3600.f + 150.f * area : 250.f + 210.f * area) + fmaxf(step, feed) * (float)h.kt;
  const float stream = (float)(nmt * bm) * (0.1f + 0.9f * (float)NT) * (bm == 256 ? h.row2 : h.row) * (float)h.kt;
  return fmaxf((float)passes * unit, stream) * (passes == 1 && nblk <= h.once_most ? h.once : 1.f);
}
inline HeadPlan head_plan_host(const HeadShape& h, int n_act) {
  const int nblk = (n_act + 31) >> 5, least = (nblk + 9) / 10;
  HeadPlan p = {0, 0, 0};
  float best = 0.f;
  for (int i = 0; i < 64; ++i) {
    const int bm = i < 32 ? 128 : 256, NT = least + (i & 31);
    const float price = head_price(h, n_act, bm, NT);
    if (price > 0.f && (p.bm == 0 || price < best)) {
      best = price;
      p = HeadPlan{bm, NT, (nblk + NT - 1) / NT};
    }
  }
  return p;
}
// The same by all 64 lanes of a wave, one result in every wave: lanes 0 .. 31 price 128-row tiles, the others 256-row tiles.
__device__ __forceinline__ HeadPlan head_plan(const HeadShape& h, int n_act, int lane) {
  const int nblk = (n_act + 31) >> 5, bm = lane < 32 ? 128 : 256, NT = (nblk + 9) / 10 + (lane & 31);
  const float price = head_price(h, n_act, bm, NT);
  const uint32_t key = price > 0.f ? ~__float_as_uint(price) : 0u;                                 // the order of positive floats
  const int l = __ffsll((unsigned long long)__ballot(key == wave_max_u32(key))) - 1;
  HeadPlan p;
  p.bm = __builtin_amdgcn_readlane(bm, l);
  p.NT = __builtin_amdgcn_readlane(NT, l);
  p.bpt = (nblk + p.NT - 1) / p.NT;
  return p;
}

}  // namespace ddd
