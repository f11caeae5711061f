"""The plan of the one-product path's launches (csrc/mes_prefill_plan.h), compiled for the host: token blocks and the
addresses made from them."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include "mes_prefill_plan.h"
using namespace mes;
extern "C" {
int max_segs() { return kMaxSegs; }
int block_tiles() { return kBlockTiles; }
// what the kernel finds in its arguments for a block: the block, and where its tiles lie in a k block
void through_arguments(int sg, int tile0, int tiles, int* out, uint64_t* at) {
  const TokenBlock b = token_block(block_entry(TokenBlock{sg, tile0, tiles}));
  out[0] = b.sg; out[1] = b.tile0; out[2] = b.tiles;
  for (int t = 0; t < tiles; ++t) at[t] = tile_offset(b.tile0) + tile_offset(t);
}
// a launch's plan: head = row tiles, splits, steps of each, blocks, of these: full ones by arithmetic, halves; and the blocks
int make_plan(const int* seg_tiles, int n_seg, const int* d_out, int n_linears, int steps, int* head, int* blocks, int room) {
  PrefillPlan pl;
  prefill_plan(pl, seg_tiles, n_seg, d_out, n_linears, steps);
  const int n = count(pl.blocks);
  head[0] = pl.rt; head[1] = pl.n_split; head[2] = pl.steps_per_split; head[3] = n; head[4] = pl.blocks.n_full; head[5] = pl.blocks.n_half;
  if (n > room) return 1;
  for (int b = 0; b < n; ++b) {
    const TokenBlock t = b % 3 || b < kMaxBlocks ? block_at(pl.blocks, b) : block_at(behind(behind(pl.blocks, kMaxBlocks), b - kMaxBlocks), 0);
    blocks[3 * b] = t.sg; blocks[3 * b + 1] = t.tile0; blocks[3 * b + 2] = t.tiles;
  }
  return 0;
}
// a cut as the plan weighs it, and as it is made: blocks by size, full and halved ones by arithmetic, all
void weighed_and_made(const int* seg_tiles, int n_seg, int most, int even, int halved, int* weighed, int* made) {
  const Cut c = {most, even != 0, halved};
  const Sizes z = sizes_of(seg_tiles, n_seg, c);
  Blocks bl;
  cut_blocks(bl, seg_tiles, n_seg, c);
  for (int i = 0; i < kClasses; ++i) { weighed[i] = z.listed[i]; made[i] = 0; }
  for (int b = 0; b < bl.n_list; ++b) ++made[size_class(bl.list[b].shape >> 3)];
  weighed[kClasses] = z.n_full; weighed[kClasses + 1] = z.n_half; weighed[kClasses + 2] = z.total;
  made[kClasses] = bl.n_full; made[kClasses + 1] = bl.n_half; made[kClasses + 2] = count(bl);
}
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("prefill_plan")
    src, lib = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-o", str(lib), str(src),
                           "-I" + os.path.join(ROOT, "paper_2406_09041_amd", "csrc")])
    return ctypes.CDLL(str(lib))


@pytest.mark.parametrize("tile0", [0, 1, 4095, (1 << 22) - 32, (1 << 22) - 1, 1 << 22, (1 << 22) + 5, (1 << 23) - 1, 1 << 23, (1 << 27) - 32])
def test_blocks_of_any_tile_reach_the_kernel(plan, tile0):
    """A launch of 2^22 token tiles (67 million tokens) or more: neither the block's place in the kernel's arguments nor the
    byte offset of its tiles wraps."""
    n = plan.block_tiles()
    for sg in range(plan.max_segs()):
        for tiles in (1, 31, n):
            out, at = (ctypes.c_int * 3)(), (ctypes.c_uint64 * n)()
            plan.through_arguments(sg, tile0, tiles, out, at)
            assert list(out) == [sg, tile0, tiles]
            assert list(at)[:tiles] == [(tile0 + t) * 1024 for t in range(tiles)]


def checked_plan(plan, seg_tiles, d_outs, steps):
    head, room = (ctypes.c_int * 6)(), sum(seg_tiles)
    blocks = np.zeros((room, 3), dtype=np.int32)
    st = plan.make_plan((ctypes.c_int * len(seg_tiles))(*seg_tiles), len(seg_tiles), (ctypes.c_int * len(d_outs))(*d_outs), len(d_outs), steps,
                        head, blocks.ctypes.data_as(ctypes.c_void_p), room)
    assert st == 0, "more blocks than tiles"
    rt, n_split, per, n, n_full, n_half = head
    b = blocks[:n]
    b = b[np.argsort(b[:, 1])]
    ends = np.concatenate([[0], np.cumsum(seg_tiles)])
    # every tile of every segment in one block, no block across segments or longer than a workgroup's
    assert (b[:, 1] == np.concatenate([[0], np.cumsum(b[:, 2])[:-1]])).all() and b[:, 2].sum() == ends[-1]
    assert (b[:, 2] >= 1).all() and (b[:, 2] <= plan.block_tiles()).all()
    assert (ends[b[:, 0]] <= b[:, 1]).all() and (b[:, 1] + b[:, 2] <= ends[b[:, 0] + 1]).all()
    # every step in one split, none empty; split sums fit the scratch
    assert rt in (7, 8) and n_split >= 1 and (n_split - 1) * per < steps <= n_split * per
    n_rg = sum((-(-d // 64) * 4 + rt - 1) // rt for d in d_outs)
    assert n_split == 1 or n_split * n_rg * n <= 256
    return rt, n_split, n, n_full, n_half


@pytest.mark.parametrize("seed", range(40))
def test_every_token_is_planned_once(plan, seed):
    rng = np.random.default_rng(seed)
    for _ in range(50):
        lo, hi = (12, 200) if seed % 2 else (12, 20000)
        seg = [int(v) for v in np.exp(rng.uniform(np.log(lo), np.log(hi), rng.integers(1, 9)))]
        d_outs = [int(v) for v in np.exp(rng.uniform(np.log(1), np.log(4000), rng.integers(1, 4)))]
        checked_plan(plan, seg, [4 * d for d in d_outs], int(rng.integers(1, 200)))


@pytest.mark.parametrize("seed", range(20))
def test_cuts_are_weighed_as_they_are_made(plan, seed):
    """The plan counts a cut's blocks by segments; the blocks themselves are made of the cut that is taken only."""
    rng = np.random.default_rng(100 + seed)
    for _ in range(50):
        n, hi = int(rng.integers(1, 9)), (40, 300, 3000)[seed % 3]
        seg = (ctypes.c_int * n)(*[int(v) for v in np.exp(rng.uniform(0, np.log(hi), n))])
        full = sum(t // 32 for t in seg)
        for most, even, halved in [(m, 1, 0) for m in (4, 8, 12, 16, 24, 32)] + [(32, 0, h) for h in {0, full // 2, full}]:
            weighed, made = (ctypes.c_int * 11)(), (ctypes.c_int * 11)()
            plan.weighed_and_made(seg, n, most, even, halved, weighed, made)
            assert list(weighed) == list(made), (list(seg), most, even, halved)


@pytest.mark.parametrize("tokens,d_out,halves", [
    ([69000], 136, True),
    ([23000, 200, 45800], 136, True),         # a segment of less than a full block between two long ones
    ([70000], 72, False),
    ([192, 100, 200000, 300], 128, False),
    ([9000] * 8, 64, False),
    ([80000], 1024, False),
    ([80000], 4096, False),
])
def test_more_blocks_than_the_list_holds_share_one_launch(plan, tokens, d_out, halves):
    """... and only the segments' last, partial blocks are listed."""
    rt, n_split, n, n_full, n_half = checked_plan(plan, [(t + 15) // 16 for t in tokens], [d_out], 5)
    assert n > 128 and n_full > 0 and n - n_full - n_half <= len(tokens)
    assert (n_half > 0) == halves


def test_a_launch_of_as_many_tokens_as_memory_holds(plan):
    """2^30 tokens on a narrow layer: the counts stay within 32 bits, and the plan is made in a moment."""
    head = (ctypes.c_int * 6)()
    seg = [(1 << 26) - 108, 13]
    assert plan.make_plan((ctypes.c_int * 2)(*seg), 2, (ctypes.c_int * 1)(8), 1, 2, head, None, 0) == 1
    assert head[1] == 1 and head[3] >= seg[0] // plan.block_tiles()
