// How tree attention is split over workgroups, and what its workspace holds.
#pragma once

namespace ddd {

constexpr int kQT = 64;         // queries per tile

// Steps of a head: the prompt's whole ones, then the rest of its keys and the tree's (chunks of 32, the last of either ragged).
struct AttnSteps {
  int full, rest_prompt, rest, all;   // whole steps; chunks of the rest from the prompt, in all; steps in all
};
__host__ __device__ inline AttnSteps attn_steps(int L, int T, int nw) {
  AttnSteps n;
  n.full = L / (32 * nw);
  n.rest_prompt = (L - n.full * 32 * nw + 31) / 32;
  n.rest = n.rest_prompt + (T + 31) / 32;
  n.all = n.full + (n.rest + nw - 1) / nw;
  return n;
}

// Waves per workgroup.  Few tiles (one to four users): eight, one workgroup per CU - a step is 256 keys, so a head needs half as many
// splits and partials.  Otherwise four: three workgroups fit a CU, and every value is read by one wave instead of two.
// 32 heads, L = 1999 / 1500 / 700 / 2048 with 1 / 4 / 9 / 64 users, eight against four: 22.8 / 34.9 / 41.9 / 441 us against
// 24.9 / 35.8 / 32.3 / 426 (27.5 / 49.9 / 57.7 / 493 with a whole output tile per wave and merges through LDS); all without the
// weights' low halves, which cost one user 1.6 us and 64 users nothing.
inline int attn_waves(long long tiles, int n_cu) { return 2 * tiles <= n_cu ? 8 : 4; }
inline long long attn_tiles(int B, int n_heads, int T) { return (long long)B * n_heads * ((T + kQT - 1) / kQT); }

// Splits of a head's keys over workgroups that the workspace has room for: one workgroup of eight waves or two of four per CU, a step
// each at least.  Never fewer for a longer prompt, so a program's workspace for its longest prompt serves the shorter ones.
inline int tree_attention_splits(int B, int n_heads, int T, int L, int n_cu) {
  const long long tiles = attn_tiles(B, n_heads, T);
  const int nw = attn_waves(tiles, n_cu), all = attn_steps(L, T, nw).all, most = all < 64 ? all : 64;
  const long long fill = (nw == 8 ? 1 : 2) * n_cu / tiles;
  return fill < 1 ? 1 : fill < most ? (int)fill : most;
}

// What a launch makes of them: `per` chunks of 32 keys per workgroup where one pass over them takes the place of several steps (then
// as few splits as hold all chunks, none without one), or 0.
constexpr int kPassChunks = 16;
struct AttnLaunch {
  int nw, nsplit, per;
};
inline AttnLaunch attn_launch(int B, int n_heads, int T, int L, int n_cu) {
  AttnLaunch p;
  p.nw = attn_waves(attn_tiles(B, n_heads, T), n_cu);
  p.nsplit = tree_attention_splits(B, n_heads, T, L, n_cu);
  const int all = (L + 31) / 32 + (T + 31) / 32, per = (all + p.nsplit - 1) / p.nsplit;
  p.per = p.nw == 8 && p.nsplit > 1 && per > 8 && per <= kPassChunks ? per : 0;
  if (p.per > 0) p.nsplit = (all + per - 1) / per;
  return p;
}

}  // namespace ddd
