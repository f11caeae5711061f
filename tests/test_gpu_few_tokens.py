"""Calls of up to 32 tokens, around every edge of the one-launch path's dispatch: tokens per tile, experts per register
set, wavefronts per row tile (row counts), chunks per wavefront, salient pairs.  Bars as for the streaming path: exact
products, fp32 sums, one rounding."""
import ctypes

import numpy as np
import pytest
import torch

import parity_checks as PC

from inputs import synth
from oracle import mes_oracle as O
from test_gpu_parity import gated_case, oracle_experts, rel_fro, run_case, TOL

pytestmark = pytest.mark.gpu
mes = pytest.importorskip("paper_2406_09041_amd")
DEV = "cuda:0"


def segments(tokens, experts, empty=0):
    """`experts` owners of `tokens` tokens (the first ones the surplus), an empty expert before and after them."""
    off = [0] * (1 + empty)
    for e in range(experts):
        off.append(off[-1] + tokens // experts + (1 if e < tokens % experts else 0))
    return off + [off[-1]] * empty


@pytest.mark.parametrize("bits,grid", [(1, 0), (2, 0), (2, 1), (3, 0), (4, 1)])
@pytest.mark.parametrize("tokens,experts", [(1, 1), (15, 4), (16, 5), (16, 8), (16, 9), (16, 16), (17, 1), (32, 4), (31, 5), (32, 8), (32, 9), (33, 2)])
def test_tokens_and_experts(tokens, experts, bits, grid):
    run_case(synth.small_case(520, 76, segments(tokens, experts, 1), 33, bits, seed=tokens + experts), grid)


@pytest.mark.parametrize("d_in,d_out,tokens,experts,k,bits", [
    (8, 4, 1, 1, 0, 2),              # less than one tile of anything
    (128, 16, 2, 2, 2, 2),           # exactly one row tile, one chunk
    (1024, 1024, 3, 3, 64, 2),       # one chunk per wavefront
    (1032, 20, 5, 2, 8, 3),          # a ninth chunk of eight columns; 8 chunks per wavefront at most
    (4096, 2064, 4, 1, 64, 2),       # 129 row tiles: half a round of teams of eight
    (256, 8208, 16, 3, 40, 1),       # 513 row tiles: teams of four
    (136, 16416, 7, 7, 5, 2),        # 1026 row tiles, seven experts: the streaming path
    (136, 16416, 5, 3, 5, 2),        # ... three: teams of one
    (640, 80, 16, 16, 128, 2),       # 64 salient pairs, all there is room for
    (640, 80, 16, 16, 129, 2),       # 80: the streaming path
    (8320, 512, 9, 2, 64, 4),        # 65 chunks: nine for the first wavefront
    (8320, 1024, 9, 2, 64, 4),
    (11144, 332, 2, 2, 8, 2),        # 88 chunks on 21 row tiles: the streaming path
    (2560, 512, 20, 2, 64, 2),       # two token tiles, three chunks
    (4608, 512, 20, 2, 64, 2),       # two token tiles, five chunks: the streaming path
])
def test_shapes(d_in, d_out, tokens, experts, k, bits):
    run_case(synth.small_case(d_in, d_out, segments(tokens, experts), k, bits, seed=d_in % 89 + k))


@pytest.mark.parametrize("d_in,d_out,tokens,experts,k,bits,grid", [(264, 72, 5, 2, 5, 2, 0), (1160, 2080, 16, 9, 24, 3, 1),
                                                                   (520, 4112, 1, 1, 0, 1, 0), (512, 100, 30, 3, 64, 4, 0)])
def test_gated(d_in, d_out, tokens, experts, k, bits, grid):
    seg = segments(tokens, experts, 1)
    wg, wu, _, h = gated_case(d_in, d_out, seg, k, bits, seed=7 + bits, grid=grid)
    h_ref = O.gated_mlp_input(wg.x.double().numpy(), wg.w_base.double().numpy(), oracle_experts(wg, grid),
                              wu.w_base.double().numpy(), oracle_experts(wu, grid), seg)
    assert rel_fro(h, h_ref) <= TOL
    PC.assert_streaming_rows(h.double().cpu().numpy(), h_ref, ("gated", d_in, d_out, bits))


@pytest.mark.parametrize("d_in,d_outs,tokens,experts,k,bits", [(264, (72, 40, 100), 9, 3, 5, 2), (1024, (1040, 16, 1024), 16, 8, 64, 3)])
def test_layers_that_share_their_activations(d_in, d_outs, tokens, experts, k, bits):
    """Bit for bit the single calls (a row tile's sum does not depend on what else is in the launch, as long as the same
    number of wavefronts share it), and the oracle's bars."""
    seg = segments(tokens, experts, 1)
    wls = [synth.small_case(d_in, d, seg, k, bits, seed=50 + i) for i, d in enumerate(d_outs)]
    x = wls[0].x.to(DEV)
    packed = [(mes.mes_pack_base(wl.w_base.to(DEV)), [mes.mes_pack_delta(ex.delta.to(DEV), ex.salient_idx, bits) for ex in wl.experts]) for wl in wls]
    ys = mes.DeltaLinearMulti(packed, max_tokens=tokens)(x, seg)
    for wl, pk, y in zip(wls, packed, ys):
        y_ref = O.delta_linear(wls[0].x.double().numpy(), wl.w_base.double().numpy(), oracle_experts(wl), seg)
        PC.assert_streaming_rows(y.double().cpu().numpy(), y_ref, (d_in, wl.d_out))
        assert torch.equal(y, mes.mes_delta_linear(pk[0], pk[1], x, seg))


def test_same_result_every_time_and_for_any_row_of_the_batch():
    """Run to run the bits are the same; a token's row does not depend on the other rows, non-finite ones included."""
    wl = synth.small_case(1032, 200, [0, 6, 16], 8, 2, seed=3)
    w_t = mes.mes_pack_base(wl.w_base.to(DEV))
    ge = [mes.mes_pack_delta(ex.delta.to(DEV), ex.salient_idx, 2) for ex in wl.experts]
    x = wl.x.to(DEV)
    y = mes.mes_delta_linear(w_t, ge, x, wl.seg_offsets)
    for _ in range(5):
        assert torch.equal(y, mes.mes_delta_linear(w_t, ge, x, wl.seg_offsets))
    bad = x.clone()
    bad[3] = float("inf")
    bad[9, 5] = float("nan")
    yb = mes.mes_delta_linear(w_t, ge, bad, wl.seg_offsets)
    keep = [i for i in range(16) if i not in (3, 9)]
    assert torch.equal(y[keep], yb[keep])
    assert not torch.isfinite(yb[[3, 9]].float()).any()


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("tokens,experts", [(17, 17), (20, 20), (32, 32), (32, 18), (30, 24)])
def test_more_experts_than_a_token_group_holds(tokens, experts, bits):
    """More than 16 experts make several token groups of a call, however few its tokens.  Every entry point, with room for
    one, two and four groups (a server sizes its workspace once, for its largest batch): all rows are written, the oracle's
    bars hold, and the bits do not depend on the workspace."""
    d_in, d_out, k = 392, 76, 9
    seg = segments(tokens, experts)
    wls = [synth.small_case(d_in, d, seg, k, bits, seed=60 + i) for i, d in enumerate((d_out, d_out, 40))]
    x64, x = wls[0].x.double().numpy(), wls[0].x.to(DEV)
    packed = [(mes.mes_pack_base(wl.w_base.to(DEV)), [mes.mes_pack_delta(ex.delta.to(DEV), ex.salient_idx, bits) for ex in wl.experts]) for wl in wls]
    oes = [oracle_experts(wl) for wl in wls]
    w64 = [wl.w_base.double().numpy() for wl in wls]
    refs = [O.delta_linear(x64, w, oe, seg) for w, oe in zip(w64, oes)]
    refs.append(O.gated_mlp_input(x64, w64[0], oes[0], w64[1], oes[1], seg))

    def unwritten(d):
        return torch.full((tokens, d), float("nan"), dtype=torch.bfloat16, device=DEV)

    runs = []
    for room in (1, 128, 256):
        one = mes.DeltaLinear(*packed[0], max_tokens=room)(x, seg, unwritten(d_out))
        ys = mes.DeltaLinearMulti(packed, max_tokens=room)(x, seg, [unwritten(wl.d_out) for wl in wls])
        h = mes.DeltaLinearGated(*packed[0], *packed[1], max_tokens=room)(x, seg, unwritten(d_out))
        runs.append([one, *ys, h])
    y = unwritten(d_out)
    mes.mes_delta_linear_noalloc(*packed[0], x, seg, y)
    for got, ref in zip([*runs[0], y], [refs[0], *refs, refs[0]]):
        PC.assert_streaming_rows(got.double().cpu().numpy(), ref, (tokens, experts, bits))
    for run in runs[1:]:
        assert all(torch.equal(a, b) for a, b in zip(run, runs[0]))
    assert torch.equal(y, runs[0][0])


def blank_expert(d_in, d_out, k, bits):
    """A packed delta of zeros: right sizes, no numbers (for calls that are recorded and not run)."""
    def zeros(n, dtype=torch.uint8):
        return torch.zeros(n, dtype=dtype, device=DEV)
    lib = mes.binding.lib
    return mes.PackedDelta(d_in, d_out, k, bits, 0, zeros(lib.mes_codes_bytes(d_in, d_out, bits)), zeros(d_out, torch.float32),
                           zeros(lib.mes_salient_bytes(d_out, k)), torch.arange(k, dtype=torch.int32, device=DEV))


@pytest.mark.parametrize("d_in,d_outs,gated,counts,bits,k,one_launch", [
    # measured us per call, streaming path / one launch
    (4096, [4096], False, [1], 2, 64, True),                        # 22.8 / 14.1
    (4096, [4096], False, [1] * 16, 2, 64, True),                   # 42.8 / 34.4
    (1024, [1024], False, [1], 2, 64, True),                        # 17.4 / 8.6
    (14336, [4096], False, [1], 2, 64, True),                       # 42.0 / 31.7
    (4096, [14336, 14336], True, [1], 2, 64, True),                 # 67.7 / 56.4
    (4096, [14336], False, [2] * 7 + [1] * 2, 3, 64, True),         # 94.9 / 78.8
    (5120, [11008, 11008], True, [2] * 3, 1, 64, False),            # 70.3 / 83.0
    (4096, [14336, 14336], True, [2] * 7 + [1] * 2, 1, 64, False),  # 88.5 / 96.3
    (6152, [1112, 1112], True, [2, 2, 2, 1], 2, 64, False),         # 25.8 / 30.9
    (14336, [5120], False, [2] + [1] * 8, 2, 33, False),            # 77.3 / 91.5
    (6672, [2328, 5160, 10424], False, [4], 2, 64, False),          # 74.5 / 82.7
    (4096, [4096], False, [1] * 24, 2, 64, True),                   # two groups: 63.0 / 55.9
    (2048, [1024, 1024], True, [1] * 21, 2, 64, False),             # two groups: 30.6 / 51.2
    (4832, [444], False, [1] * 25, 2, 8, False),                    # two groups: 33 / 41
    (1024, [1024], False, [2] * 12 + [1] * 8, 2, 64, False),        # two groups, the first of two tiles: 34.6 / 41.3 mixed
])
def test_the_faster_path_is_taken(d_in, d_outs, gated, counts, bits, k, one_launch):
    """The launches of a call (recorded in a graph that is never run): one per token group, or the streaming path's two or
    three.  Lines are far from the rule's edge."""
    layers = [(torch.zeros(mes.binding.base_bytes(d_in, d) // 2, dtype=torch.bfloat16, device=DEV),
               [blank_expert(d_in, d, k, bits) for _ in counts]) for d in d_outs]
    seg = [sum(counts[:e]) for e in range(len(counts) + 1)]
    x = torch.zeros((seg[-1], d_in), dtype=torch.bfloat16, device=DEV)
    ys = [torch.empty((seg[-1], d), dtype=torch.bfloat16, device=DEV) for d in d_outs]
    call = mes.DeltaLinearGated(*layers[0], *layers[1], max_tokens=256) if gated else mes.DeltaLinearMulti(layers, max_tokens=256)
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call(x, seg, ys[0] if gated else ys)
    n = ctypes.c_size_t()
    get_nodes = mes.binding.lib.hipGraphGetNodes      # (of the HIP runtime that the library is linked to)
    get_nodes.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.POINTER(ctypes.c_size_t)]
    assert get_nodes(graph.raw_cuda_graph(), None, ctypes.byref(n)) == 0
    groups = -(-len(counts) // 16)
    assert (n.value == groups) if one_launch else (2 <= n.value <= 3)
