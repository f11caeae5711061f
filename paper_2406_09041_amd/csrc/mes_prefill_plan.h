// The plan of the one-product path's launches (mes_prefill.hip): token blocks, row tiles per workgroup, column splits.
// Plain C++ without HIP, so that the host tests compile it.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace mes {

constexpr int kMaxWorkgroups = 256;  // one workgroup per compute unit; launches of fewer split the contraction
constexpr int kMaxSegs = 8;          // long segments (experts) served by one launch
constexpr int kMaxBlocks = 128;      // token blocks of one launch
constexpr int kBlockTiles = 32;      // token tiles (16 tokens) of a full block
constexpr int kTileBytes = 1024;     // a token tile of one k block

constexpr int row_tiles(int d_out) { return (d_out + 63) / 64 * 4; }   // as stored: whole groups of 4

// A token block: its segment, its first token tile (among those of all the launch's segments) and how many it has.
struct TokenBlock { int sg, tile0, tiles; };

// ... as a kernel argument.  The first tile has a word of its own: 2^31 tokens are 2^27 tiles.
struct BlockEntry { int tile0, shape; };
constexpr BlockEntry block_entry(TokenBlock b) { return BlockEntry{b.tile0, b.sg | b.tiles << 3}; }
constexpr TokenBlock token_block(BlockEntry e) { return TokenBlock{e.shape & (kMaxSegs - 1), e.tile0, e.shape >> 3}; }

// Bytes from the first tile of a k block to another.
constexpr uint64_t tile_offset(int tile) { return (uint64_t)(uint32_t)tile * kTileBytes; }

// Time of a workgroup with up to 4, 8, ... 32 token tiles, us, 33 steps at 2 bits on a full chip, by row tiles (7, 8); 11 of
// it do not depend on the steps.
constexpr double kBlockTime[2][8] = {{44, 56, 62, 79, 92, 100, 115, 122}, {44, 59, 68, 82, 106, 109, 130, 136}};
constexpr double kFixedTime = 11;
// A launch of no more workgroups than compute units is not slowed down so much by its bigger blocks (1 bit, 3016 -> 696, 114
// tiles, 25 steps, 4 / 8 / 12 / 16 tiles: 31 / 35 / 39 / 43 us; 4 bits, 1480 -> 2996, 32 tiles, 13 steps: 20 / 22 / 25 / 28).
inline double block_time(int rt, int tiles, int steps, bool alone) {
  if (alone && tiles <= 16) return 7.4 + steps * (rt == 8 ? 0.94 + 0.16 * ((tiles - 1) / 4) : 0.91 + 0.14 * ((tiles - 1) / 4));
  return kFixedTime + (kBlockTime[rt - 7][(tiles - 1) / 4] - kFixedTime) * steps / 33.0;
}

struct Blocks {
  TokenBlock b[kMaxBlocks];
  int n;
};

struct PrefillPlan {
  int rt, n_split, steps_per_split;
  Blocks blocks;
};

// When the compute units are done that take, from a list, every token block's n_rg workgroups, each as soon as one is free.
inline double launch_time(const Blocks& bl, int n_rg, int rt, int steps, int n_split) {
  struct { double at; int units; } pool[48];                   // compute units by the time they are free
  int n = 1;
  pool[0] = {0.0, kMaxWorkgroups};
  double end = 0.0;
  const bool alone = (long)bl.n * n_rg * n_split <= kMaxWorkgroups;
  for (int i = 0; i < bl.n;) {
    int same = i + 1;
    while (same < bl.n && (bl.b[same].tiles - 1) / 4 == (bl.b[i].tiles - 1) / 4) ++same;
    const double t = block_time(rt, bl.b[i].tiles, steps, alone);
    for (long left = (long)(same - i) * n_rg * n_split; left > 0;) {
      int first = 0;
      for (int q = 1; q < n; ++q) first = pool[q].at < pool[first].at ? q : first;
      const int take = left < pool[first].units ? (int)left : pool[first].units;
      const double done = pool[first].at + t;
      end = done > end ? done : end;
      left -= take;
      if (take == pool[first].units || n == (int)(sizeof(pool) / sizeof(pool[0]))) {
        pool[first].at = done;                                 // (no room to tell them apart: all of them)
      } else {
        pool[first].units -= take;
        pool[n++] = {done, take};
      }
    }
    i = same;
  }
  return end;
}

// The segments' tokens as blocks of at most `most` tiles, the longest first.  even: a segment's blocks alike, else full ones
// and what is left.  The last `halved` full blocks become two each.  False: too many for one launch.
inline bool cut_blocks(Blocks& bl, const int* seg_tiles, int n_seg, int most, bool even, int halved) {
  bl.n = 0;
  int tile0 = 0, full = 0;
  if (halved > 0)
    for (int i = 0; i < n_seg; ++i) full += seg_tiles[i] / kBlockTiles;
  for (int i = 0; i < n_seg; ++i) {
    const int r = seg_tiles[i], nb = (r + most - 1) / most;
    for (int b = 0; b < nb; ++b) {
      const int lo = even ? (int)((long)r * b / nb) : b * most, end = even ? (int)((long)r * (b + 1) / nb) : lo + most, hi = end < r ? end : r;
      const bool halve = halved > 0 && hi - lo == kBlockTiles && full-- <= halved;
      if (bl.n + (halve ? 2 : 1) > kMaxBlocks) return false;
      const int mid = halve ? (lo + hi) / 2 : hi;
      bl.b[bl.n++] = {i, tile0 + lo, mid - lo};
      if (halve) bl.b[bl.n++] = {i, tile0 + mid, hi - mid};
    }
    tile0 += r;
  }
  for (int i = 1; i < bl.n; ++i) {                             // insertion: stable, and nearly sorted already
    const TokenBlock v = bl.b[i];
    int j = i;
    for (; j > 0 && (bl.b[j - 1].tiles - 1) / 4 < (v.tiles - 1) / 4; --j) bl.b[j] = bl.b[j - 1];
    bl.b[j] = v;
  }
  return true;
}

// Row tiles per workgroup, token blocks and column splits of a launch: whichever of a few candidates is expected to be done
// first.  A workgroup has a compute unit to itself, so what counts is how the workgroups' times fill the 256 of them.
// seg_tiles: 16-token tiles of every segment; d_out: of every layer.
inline bool prefill_plan(PrefillPlan& best, const int* seg_tiles, int n_seg, const int* d_out, int n_linears, int steps) {
  double best_time = 1e30;
  Blocks bl;
  double elements = 0;
  for (int l = 0; l < n_linears; ++l) elements += d_out[l];
  int tiles = 0;
  for (int i = 0; i < n_seg; ++i) tiles += seg_tiles[i];
  elements *= 16.0 * tiles;
  for (int rt = 8; rt >= 7; --rt) {
    int n_rg = 0;
    for (int l = 0; l < n_linears; ++l) n_rg += (row_tiles(d_out[l]) + rt - 1) / rt;
    auto consider = [&](int most, bool even, int halved) {
      if (!cut_blocks(bl, seg_tiles, n_seg, most, even, halved)) return;
      // fewer workgroups than compute units: share the steps out, at least four to each
      const long wgs = (long)n_rg * bl.n;
      for (int want = 1; want <= 8 && want * wgs <= kMaxWorkgroups && (want == 1 || 4 * want <= steps); ++want) {
        const int per = (steps + want - 1) / want, n_split = (steps + per - 1) / per;
        // (partial sums: written and read at about 9 TB/s, and another launch)
        const double t = launch_time(bl, n_rg, rt, per, n_split) + (n_split > 1 ? 4.0 + n_split * elements * 8.0 / 9e6 : 0.0);
        if (t < 0.99 * best_time) { best_time = t; best.rt = rt; best.n_split = n_split; best.steps_per_split = per; best.blocks = bl; }
      }
      if (wgs > kMaxWorkgroups) {
        const double t = launch_time(bl, n_rg, rt, steps, 1);
        if (t < 0.99 * best_time) { best_time = t; best.rt = rt; best.n_split = 1; best.steps_per_split = steps; best.blocks = bl; }
      }
    };
    consider(32, false, 0);
    int full = 0;
    for (int i = 0; i < n_seg; ++i) full += seg_tiles[i] / kBlockTiles;
    const int over = (int)((long)full * n_rg % kMaxWorkgroups), h = over / n_rg;   // full workgroups of the last round
    if (over > 0 && h > 0) consider(32, false, h);
    if (over > 0 && h < full) consider(32, false, h + 1);
    if (full * (long)n_rg < 4 * kMaxWorkgroups) {
      consider(32, true, 0);
      consider(24, true, 0);
      consider(16, true, 0);
      if (tiles * (long)n_rg < 12 * kMaxWorkgroups) consider(12, true, 0);
      // launches that blocks of 8 or 4 tiles do not make longer than about a round: the chip is idle otherwise, and a block of 4
      // tiles takes 1 us a step where one of 12 takes 1.5 (1648 -> 1920, 702 tokens 27.9 us with at least 11 tiles, now 22.4)
      if (tiles * (long)n_rg < 12 * kMaxWorkgroups) consider(8, true, 0);
      if (tiles * (long)n_rg < 8 * kMaxWorkgroups) consider(4, true, 0);
    }
  }
  return best_time < 1e30;
}

}  // namespace mes
