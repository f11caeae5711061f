"""The streaming kernel's bodies by number of experts (4, 8 or as many slots as a bit width has room for; two sweeps
beyond): every count around the edges, and launches whose token groups take different bodies."""
import pytest
import torch

from inputs import synth
from oracle import mes_oracle as O
from test_gpu_parity import check_rows, oracle_experts, run_case

pytestmark = pytest.mark.gpu
mes = pytest.importorskip("paper_2406_09041_amd")
DEV = "cuda:0"


def offsets(counts):
    off = [0]
    for c in counts:
        off.append(off[-1] + c)
    return off


@pytest.mark.parametrize("bits,experts", [(1, 5), (1, 9), (2, 4), (2, 8), (2, 16), (3, 8), (3, 9), (3, 13), (3, 14), (3, 16),
                                          (4, 8), (4, 9), (4, 10), (4, 11), (4, 16)])
def test_expert_counts(bits, experts):
    """64 tokens (the streaming path at any count), five column chunks, enough salient pairs to ride along all of them."""
    counts = [64 // experts + (1 if e < 64 % experts else 0) for e in range(experts)]
    run_case(synth.small_case(584, 200, offsets(counts), 40, bits, seed=experts))


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("counts", [[64, 30, 34] + [11] * 5 + [9] + [5] * 10 + [14], [20, 20, 24] + [8] * 8, [8] * 8 + [5] * 12 + [4]])
def test_groups_with_different_bodies_in_one_launch(bits, counts):
    """Bit for bit the result of one launch per token group: a group's body depends on its own experts only."""
    wl = synth.small_case(1160, 328, offsets(counts), 24, bits, seed=5, device=DEV)
    w_t = mes.mes_pack_base(wl.w_base)
    ge = [mes.mes_pack_delta(ex.delta, ex.salient_idx, bits) for ex in wl.experts]
    y = mes.mes_delta_linear(w_t, ge, wl.x, wl.seg_offsets)
    y1 = mes.mes_delta_linear(w_t, ge, wl.x, wl.seg_offsets, workspace=mes.make_workspace(wl.d_in, wl.d_out, 64, torch.device(DEV)))
    assert torch.equal(y, y1)
    run_case(synth.small_case(1160, 328, offsets(counts), 24, bits, seed=5))


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("counts", [[1] * 41, [1] * 42, [1] * 40, [2] * 16 + [1] * 13, [2] * 16 + [1] * 10, [2] * 16 + [1] * 7, [1] * 32 + [7, 2]])
def test_small_groups_with_different_bodies_in_one_launch(counts, bits):
    """Nearly as many experts as tokens: groups of 16 experts and one or two token tiles, the experts left in one more group.
    One launch for all of them gives bit for bit what a launch per group does, and the oracle's bars hold."""
    wl = synth.small_case(1160, 328, offsets(counts), 24, bits, seed=6, device=DEV)
    w_t = mes.mes_pack_base(wl.w_base)
    ge = [mes.mes_pack_delta(ex.delta, ex.salient_idx, bits) for ex in wl.experts]
    ys = []
    for room in (64, 256):
        y = torch.full((wl.x.shape[0], wl.d_out), float("nan"), dtype=torch.bfloat16, device=DEV)
        ys.append(mes.DeltaLinear(w_t, ge, max_tokens=room)(wl.x, wl.seg_offsets, y))
    assert torch.equal(ys[0], ys[1])
    oe = oracle_experts(wl)
    w64 = wl.w_base.double().cpu().numpy()
    check_rows(wl, ys[1], O.delta_linear(wl.x.double().cpu().numpy(), w64, oe, wl.seg_offsets), oe, w64)


@pytest.mark.parametrize("d_in,d_out", [(2184, 1096), (648, 72), (1032, 2184)])
@pytest.mark.parametrize("counts", [[37], [5] * 13, [64, 64, 3], [64] + [16] * 4 + [4] * 16 + [21]])
def test_every_row_group_and_split_is_computed_once(d_in, d_out, counts):
    """Numbers of (row group, split) pairs that are no multiple of the 8 dies they are dealt to, with one to four token groups
    in a launch: the oracle's bars, and bit for bit the result of one launch per group."""
    wl = synth.small_case(d_in, d_out, offsets(counts), 24, 2, seed=7, device=DEV)
    w_t = mes.mes_pack_base(wl.w_base)
    ge = [mes.mes_pack_delta(ex.delta, ex.salient_idx, 2) for ex in wl.experts]
    ys = []
    for room in (64, 191):
        y = torch.full((wl.x.shape[0], wl.d_out), float("nan"), dtype=torch.bfloat16, device=DEV)
        ys.append(mes.DeltaLinear(w_t, ge, max_tokens=room)(wl.x, wl.seg_offsets, y))
    assert torch.equal(ys[0], ys[1])
    oe = oracle_experts(wl)
    w64 = wl.w_base.double().cpu().numpy()
    check_rows(wl, ys[1], O.delta_linear(wl.x.double().cpu().numpy(), w64, oe, wl.seg_offsets), oe, w64)
