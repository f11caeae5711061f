// The plan of the one-product path's launches (mes_prefill.hip): token blocks, row tiles per workgroup, column splits.
// Plain C++ without HIP, so that the host tests compile it.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace mes {

constexpr int kMaxWorkgroups = 256;  // one workgroup per compute unit; launches of fewer split the contraction
constexpr int kMaxSegs = 8;          // long segments (experts) served by one launch
constexpr int kMaxBlocks = 128;      // token blocks of a launch that are listed one by one
constexpr int kBlockTiles = 32;      // token tiles (16 tokens) of a full block
constexpr int kTileBytes = 1024;     // a token tile of one k block

constexpr int row_tiles(int d_out) { return (d_out + 63) / 64 * 4; }   // as stored: whole groups of 4

// A token block: its segment, its first token tile (among those of all the launch's segments) and how many it has.
struct TokenBlock { int sg, tile0, tiles; };

// ... as a kernel argument.  The first tile has a word of its own: 2^31 tokens are 2^27 tiles.
struct BlockEntry { int tile0, shape; };
constexpr BlockEntry block_entry(TokenBlock b) { return BlockEntry{b.tile0, b.sg | b.tiles << 3}; }
constexpr TokenBlock token_block(BlockEntry e) { return TokenBlock{e.shape & (kMaxSegs - 1), e.tile0, e.shape >> 3}; }

// The token blocks of a launch: the listed ones, the longest first -- or, of more blocks than the list holds, the listed ones (the
// segments' last, partial blocks), then n_full blocks of full_tiles tiles, one segment's behind the other's, then n_half
// halves of blocks that continue them.  One launch however many they are: launches of 128 blocks each leave part of the chip
// idle at the end of each, all the time where the rows are one row group (80000 tokens of 4 experts on 512 -> 128:
// 102 us, now 70.5).
struct Blocks {
  BlockEntry list[kMaxBlocks];
  int n_list, n_full, n_half, full_tiles;
  int first;                                   // of the blocks that are not listed, those before it are not this launch's
  int full0[kMaxSegs], tile0[kMaxSegs];        // of a segment: its first full block, its first tile
};
constexpr int count(const Blocks& bl) { return bl.n_list + bl.n_full + bl.n_half; }
constexpr int longest(const Blocks& bl) {                       // ... block's tiles
  const int listed = bl.n_list > 0 ? bl.list[0].shape >> 3 : 0;
  return bl.n_full > 0 && bl.full_tiles > listed ? bl.full_tiles : listed;
}
constexpr TokenBlock unlisted_block(const Blocks& bl, int b) {   // b counts from the first one behind the list
  b += bl.first;
  int half = 0, tiles = bl.full_tiles;
  if (b >= bl.n_full) {
    half = (b - bl.n_full) & 1;
    tiles /= 2;
    b = bl.n_full + ((b - bl.n_full) >> 1);
  }
  int sg = 0;
  for (int i = 1; i < kMaxSegs; ++i) sg += b >= bl.full0[i] ? 1 : 0;   // (segments without full blocks start where the next one does)
  return TokenBlock{sg, bl.tile0[sg] + bl.full_tiles * (b - bl.full0[sg]) + half * tiles, tiles};
}
constexpr TokenBlock block_at(const Blocks& bl, int b) {
  return b < bl.n_list ? token_block(bl.list[b]) : unlisted_block(bl, b - bl.n_list);
}

// The blocks behind the first n >= n_list ones (a grid has 65535 at most).
constexpr Blocks behind(Blocks bl, int n) {
  bl.first += n - bl.n_list;
  bl.n_list = 0;
  return bl;
}

// Bytes from the first tile of a k block to another.
constexpr uint64_t tile_offset(int tile) { return (uint64_t)(uint32_t)tile * kTileBytes; }

// Time of a workgroup with up to 4, 8, ... 32 token tiles, us, 33 steps at 2 bits on a full chip, by row tiles (7, 8); 11 of
// it do not depend on the steps.  (Other bit widths use it too: against the better of 7 and 8 row tiles the choice it makes costs
// 0.8 % at 3 and 4 bits, 72 calls, and 1.7 % at 1 and 2, 24 calls.)
constexpr double kBlockTime[2][8] = {{44, 56, 62, 79, 92, 100, 115, 122}, {44, 59, 68, 82, 106, 109, 130, 136}};
constexpr double kFixedTime = 11;
// A launch of no more workgroups than compute units is not slowed down so much by its bigger blocks (1 bit, 3016 -> 696, 114
// tiles, 25 steps, 4 / 8 / 12 / 16 tiles: 31 / 35 / 39 / 43 us; 4 bits, 1480 -> 2996, 32 tiles, 13 steps: 20 / 22 / 25 / 28).
inline double block_time(int rt, int tiles, int steps, bool alone) {
  if (alone && tiles <= 16) return 7.4 + steps * (rt == 8 ? 0.94 + 0.16 * ((tiles - 1) / 4) : 0.91 + 0.14 * ((tiles - 1) / 4));
  return kFixedTime + (kBlockTime[rt - 7][(tiles - 1) / 4] - kFixedTime) * steps / 33.0;
}


struct PrefillPlan {
  int rt, n_split, steps_per_split;
  Blocks blocks;
};

// How a launch's tokens are cut: blocks of at most `most` tiles; even: a segment's blocks alike, else full ones and what is
// left; the last `halved` full blocks (of kBlockTiles) become two each.
struct Cut { int most; bool even; int halved; };

constexpr int size_class(int tiles) { return (tiles - 1) / 4; }
constexpr int kClasses = kBlockTiles / 4;

// What the plan weighs of a cut: how many blocks are listed, by size, and how many are not.  Counted by segments, without
// making the list: a plan weighs up to 18 cuts and takes one, and small calls are as long as the host takes to launch them (128
// -> 368, 1091 + 372 tokens, with a list made per cut 11.7 us of host time, 11.8 a call; now 11.2 and 11.4).
struct Sizes { int listed[kClasses], n_full, n_half, full_tiles, total; bool list_all; };
inline Sizes sizes_of(const int* seg_tiles, int n_seg, Cut c) {
  Sizes z = {};
  z.full_tiles = c.most;
  int full = 0;
  z.total = c.halved;
  for (int i = 0; i < n_seg; ++i) {
    full += seg_tiles[i] / c.most;
    z.total += (seg_tiles[i] + c.most - 1) / c.most;
  }
  z.list_all = z.total <= kMaxBlocks;
  if (!z.list_all) {
    z.n_full = full - c.halved;
    z.n_half = 2 * c.halved;
  }
  for (int i = 0; i < n_seg; ++i) {
    const int r = seg_tiles[i], nb = (r + c.most - 1) / c.most, left = r % c.most;
    if (z.list_all && c.even) {                                // r % nb blocks have a tile more than the others
      z.listed[size_class(r / nb)] += nb - r % nb;
      if (r % nb > 0) z.listed[size_class(r / nb + 1)] += r % nb;
    } else {
      if (z.list_all) z.listed[size_class(c.most)] += r / c.most;
      if (left > 0) ++z.listed[size_class(left)];
    }
  }
  if (z.list_all && c.halved > 0) {
    z.listed[size_class(kBlockTiles)] -= c.halved;
    z.listed[size_class(kBlockTiles / 2)] += 2 * c.halved;
  }
  return z;
}

// When the compute units are done that take, from a list, every token block's n_rg workgroups, each as soon as one is free.
inline double launch_time(const Sizes& z, int n_rg, int rt, int steps, int n_split) {
  struct { double at; int units; } pool[48];                   // compute units by the time they are free
  int n = 1;
  pool[0] = {0.0, kMaxWorkgroups};
  double end = 0.0;
  const bool alone = (long)z.total * n_rg * n_split <= kMaxWorkgroups;
  auto take_blocks = [&](int tiles, long blocks) {
    const double t = block_time(rt, tiles, steps, alone);
    for (long left = blocks * n_rg * n_split; left > 0;) {
      if (n == 1 && left >= kMaxWorkgroups) {                  // whole rounds
        end = pool[0].at += (double)(left / kMaxWorkgroups) * t;
        left %= kMaxWorkgroups;
        continue;
      }
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
  };
  for (int c = kClasses - 1; c >= 0; --c)
    if (z.listed[c] > 0) take_blocks(4 * c + 1, z.listed[c]);
  if (z.n_full > 0) take_blocks(z.full_tiles, z.n_full);
  if (z.n_half > 0) take_blocks(z.full_tiles / 2, z.n_half);
  return end;
}

// The segments' tokens as blocks, the longest first.
inline void cut_blocks(Blocks& bl, const int* seg_tiles, int n_seg, Cut c) {
  const Sizes z = sizes_of(seg_tiles, n_seg, c);
  bl.n_list = bl.first = 0;
  bl.n_full = z.n_full;
  bl.n_half = z.n_half;
  bl.full_tiles = c.most;
  int tile0 = 0, full = 0;
  for (int i = 0; i < kMaxSegs; ++i) {
    bl.full0[i] = full;
    bl.tile0[i] = tile0;
    if (i >= n_seg) continue;
    full += seg_tiles[i] / c.most;
    tile0 += seg_tiles[i];
  }
  for (int i = 0; i < n_seg; ++i) {
    const int r = seg_tiles[i], nb = (r + c.most - 1) / c.most;
    for (int b = z.list_all ? 0 : r / c.most; b < nb; ++b) {
      const bool alike = c.even && z.list_all;
      const int lo = alike ? (int)((long)r * b / nb) : b * c.most, end = alike ? (int)((long)r * (b + 1) / nb) : lo + c.most, hi = end < r ? end : r;
      const bool halve = z.list_all && c.halved > 0 && hi - lo == kBlockTiles && full-- <= c.halved;
      const int mid = halve ? (lo + hi) / 2 : hi;
      bl.list[bl.n_list++] = block_entry({i, bl.tile0[i] + lo, mid - lo});
      if (halve) bl.list[bl.n_list++] = block_entry({i, bl.tile0[i] + mid, hi - mid});
    }
  }
  auto size = [](const BlockEntry& e) { return size_class(e.shape >> 3); };
  for (int i = 1; i < bl.n_list; ++i) {                        // insertion: stable, and nearly sorted already
    const BlockEntry v = bl.list[i];
    int j = i;
    for (; j > 0 && size(bl.list[j - 1]) < size(v); --j) bl.list[j] = bl.list[j - 1];
    bl.list[j] = v;
  }
  for (int i = bl.n_list; i < kMaxBlocks; ++i) bl.list[i] = BlockEntry{0, 0};   // never selected
}

// Row tiles per workgroup, token blocks and column splits of a launch: whichever of a few candidates is expected to be done
// first.  A workgroup has a compute unit to itself, so what counts is how the workgroups' times fill the 256 of them.
// seg_tiles: 16-token tiles of every segment; d_out: of every layer.
inline void prefill_plan(PrefillPlan& best, const int* seg_tiles, int n_seg, const int* d_out, int n_linears, int steps) {
  double best_time = 1e30;
  Cut best_cut = {kBlockTiles, false, 0};
  double elements = 0;
  for (int l = 0; l < n_linears; ++l) elements += d_out[l];
  int tiles = 0, full = 0;
  for (int i = 0; i < n_seg; ++i) {
    tiles += seg_tiles[i];
    full += seg_tiles[i] / kBlockTiles;
  }
  elements *= 16.0 * tiles;
  for (int rt = 8; rt >= 7; --rt) {
    int n_rg = 0;
    for (int l = 0; l < n_linears; ++l) n_rg += (row_tiles(d_out[l]) + rt - 1) / rt;
    auto consider = [&](Cut c) {
      const Sizes z = sizes_of(seg_tiles, n_seg, c);
      auto weigh = [&](int n_split, int per) {
        // (partial sums: written and read at about 9 TB/s, and another launch)
        const double t = launch_time(z, n_rg, rt, per, n_split) + (n_split > 1 ? 4.0 + n_split * elements * 8.0 / 9e6 : 0.0);
        if (t < 0.99 * best_time) { best_time = t; best.rt = rt; best.n_split = n_split; best.steps_per_split = per; best_cut = c; }
      };
      // fewer workgroups than compute units: share the steps out, at least four to each
      const long wgs = (long)n_rg * z.total;
      for (int want = 1; want <= 8 && want * wgs <= kMaxWorkgroups && (want == 1 || 4 * want <= steps); ++want) {
        const int per = (steps + want - 1) / want;
        weigh((steps + per - 1) / per, per);
      }
      if (wgs > kMaxWorkgroups) weigh(1, steps);
    };
    consider({32, false, 0});
    const int over = (int)((long)full * n_rg % kMaxWorkgroups), h = over / n_rg;   // full workgroups of the last round
    if (over > 0 && h > 0) consider({32, false, h});
    if (over > 0 && h < full) consider({32, false, h + 1});
    if (full * (long)n_rg < 4 * kMaxWorkgroups) {
      consider({32, true, 0});
      consider({24, true, 0});
      consider({16, true, 0});
      if (tiles * (long)n_rg < 12 * kMaxWorkgroups) consider({12, true, 0});
      // launches that blocks of 8 or 4 tiles do not make longer than about a round: the chip is idle otherwise, and a block of 4
      // tiles takes 1 us a step where one of 12 takes 1.5 (1648 -> 1920, 702 tokens 27.9 us with at least 11 tiles, now 22.4)
      if (tiles * (long)n_rg < 12 * kMaxWorkgroups) consider({8, true, 0});
      if (tiles * (long)n_rg < 8 * kMaxWorkgroups) consider({4, true, 0});
    }
  }
  cut_blocks(best.blocks, seg_tiles, n_seg, best_cut);
}

}  // namespace mes
