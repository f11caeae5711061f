"""The plan of the one-product path's launches (csrc/mes_prefill_plan.h), compiled for the host: token blocks and the
addresses made from them."""
import ctypes
import os
import subprocess

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
