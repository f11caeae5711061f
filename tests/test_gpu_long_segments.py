"""Long segments on the one-product path: calls of more token blocks than a launch lists one by one, short
contractions, layers that share their activations."""
import pytest
import torch

from inputs import synth
from oracle import mes_oracle as O
from test_gpu_parity import TOL, check_rows, gpu_experts, oracle_experts, run_case, sampled_rows_check

pytestmark = pytest.mark.gpu
mes = pytest.importorskip("paper_2406_09041_amd")
DEV = "cuda:0"


def offsets(lengths):
    off = [0]
    for n in lengths:
        off.append(off[-1] + n)
    return off


@pytest.mark.parametrize("d_in,d_out,k,bits,lengths", [
    (264, 136, 8, 2, [23000, 200, 45800]),   # 32-tile blocks, the last ones as halves, three partial ones
    (136, 72, 0, 3, [70000]),                # one row group: 24-tile blocks
    (72, 40, 5, 4, [9000] * 7 + [5, 9000]),  # eight long segments and a streamed one
])
def test_more_blocks_than_the_list_holds(d_in, d_out, k, bits, lengths):
    run_case(synth.small_case(d_in, d_out, offsets(lengths), k, bits, seed=len(lengths)))


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("d_in,d_out,k,lengths", [
    (264, 7448, 8, [784]),                   # 8 row tiles; blocks of 13 tiles (the last column of wavefronts has one) and of 12
    (648, 9000, 0, [220, 205]),              # 7 row tiles; 14 tiles (the last column has none) and 13
    (264, 9000, 33, [256, 272, 200]),        # 16 tiles, and halves of 17
])
def test_short_contractions(d_in, d_out, k, lengths, bits):
    """Blocks of 13 to 16 token tiles in launches of few steps: eight columns of wavefronts instead of four.  Every tile of
    16 x 16 results within the path's Frobenius tolerance (256 errors of about 1.4 sigma = 2.3e-3 each; 16 rows' share of the norm
    varies by a few times 1 / 16, hence twice the tolerance), and the element-wise bars on 512 channels (6 sigma of a sum of
    d_in rounding errors, whose tails are a little heavier than normal, is exceeded about once in 4 million elements)."""
    wl = synth.small_case(d_in, d_out, offsets(lengths), k, bits, seed=len(lengths), device=DEV)
    w_t = mes.mes_pack_base(wl.w_base)
    ge = [mes.mes_pack_delta(ex.delta, ex.salient_idx.to(DEV), bits) for ex in wl.experts]
    y = torch.full((wl.x.shape[0], d_out), float("nan"), dtype=torch.bfloat16, device=DEV)
    mes.DeltaLinear(w_t, ge, max_tokens=wl.x.shape[0])(wl.x, wl.seg_offsets, y)
    torch.cuda.synchronize()
    for p, lo, hi in zip(ge, wl.seg_offsets, wl.seg_offsets[1:]):
        w = wl.w_base.double() + mes.mes_unpack_delta(p, want_codes=False)[0].double()
        ref = wl.x[lo:hi].double() @ w.t()

        def tiles(v):                        # sums of squares of the 16 x 16 tiles
            v = torch.nn.functional.pad(v * v, (0, -d_out % 16, 0, -(hi - lo) % 16))
            return v.reshape(-(-(hi - lo) // 16), 16, -(-d_out // 16), 16).sum((1, 3))
        assert (tiles(y[lo:hi].double() - ref) <= (2 * TOL) ** 2 * tiles(ref)).all(), (lo, hi)
    assert sampled_rows_check(wl, y, 512, 3 + bits) <= TOL


def test_short_contractions_of_more_blocks_than_the_list_holds():
    """16-tile blocks and partial ones of 4 tiles in one launch."""
    run_case(synth.small_case(136, 64, offsets([8000] * 8), 8, 2, seed=4))


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("d_in,d_outs,k,lengths", [
    (248, [136, 72, 200], 40, [300, 5, 210]),     # one launch per layer: the scratch has no room for three layers' gathered channels
    (120, [72, 328], 8, [193, 450]),              # ... nor for two beside one chunk
    (1024, [72, 136], 512, [200]),                # one launch, three splits: the last one has nothing but salient steps
    (2048, [72, 136, 64], 600, [200, 3]),         # five: one goes over to the salient steps of its layer, one begins in them
    (520, [72, 264, 136], 33, [449]),             # one salient step per layer
])
def test_long_segments_of_layers_that_share_their_activations(d_in, d_outs, k, lengths, bits):
    """Each layer has salient channels of its own, gathered behind the shared input channels or, where they do not fit, in the
    same place one layer after the other."""
    off = offsets(lengths)
    wls = [synth.small_case(d_in, d, off, k, bits, seed=70 + i) for i, d in enumerate(d_outs)]
    x = wls[0].x
    layers = [(mes.mes_pack_base(w.w_base.to(DEV)), gpu_experts(w)) for w in wls]
    ys = [torch.full((off[-1], d), float("nan"), dtype=torch.bfloat16, device=DEV) for d in d_outs]
    mes.DeltaLinearMulti(layers, off[-1])(x.to(DEV), off, ys)
    torch.cuda.synchronize()
    for w, y in zip(wls, ys):
        w.x = x
        oe, w64 = oracle_experts(w), w.w_base.double().numpy()
        check_rows(w, y, O.delta_linear(x.double().numpy(), w64, oe, off), oe, w64, what=w.d_out)


@pytest.mark.parametrize("bits", [3, 4])
@pytest.mark.parametrize("d_out,lengths", [(9488, [265, 405])])
def test_blocks_of_17_to_24_tiles_with_8_row_tiles(d_out, lengths, bits):
    """... keep three sets of activation fragments at 3 and 4 bits, where full blocks have two; 9 chunks and a salient step."""
    run_case(synth.small_case(1032, d_out, offsets(lengths), 33, bits, seed=bits))
