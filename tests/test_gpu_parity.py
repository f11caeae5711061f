"""GPU parity: the HIP path (through the C ABI) against the fp64 CPU oracle, same seeded inputs.

Bars: packed code words, step bits, fp16 salient bits, salient indices and routing are bit-exact.
y is compared element by element (tests/parity_checks.py): rows of the streaming path within 1 bf16 ulp of
bf16_rne(y_oracle) on at least 99.9 % of the elements and within 2 ulp on all; rows of the one-product path
(segments of mes_long_segment_tokens() tokens or more) within 6 sigma of the operand rounding plus 1 ulp.  The
stated bar, relative Frobenius error <= 5e-3, is checked as well; it is dominated by the final rounding of y to
bf16 (half an ulp is up to 2^-8 relative: about 1.6e-3 in the norm).
"""
import numpy as np
import pytest
import torch

import paper_2406_09041_amd as mes
import parity_checks as PC
from inputs import synth
from oracle import mes_oracle as O

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 5e-3


def oracle_experts(wl, grid=O.GRID_SYM, policy=O.STEP_MAXABS, rows=None):
    out = []
    for ex in wl.experts:
        d = ex.delta.cpu().numpy() if rows is None else ex.delta[rows].cpu().numpy()
        c, s, sal = O.quantize(d, ex.salient_idx.numpy(), wl.bits, grid, policy)
        out.append(dict(codes=c, step=s, salient=sal, salient_idx=ex.salient_idx.numpy(), bits=wl.bits, grid=grid))
    return out


def gpu_experts(wl, grid=mes.GRID_SYM, policy=mes.STEP_MAXABS):
    return [mes.mes_pack_delta(ex.delta.to(DEV), ex.salient_idx, wl.bits, grid, policy) for ex in wl.experts]


def rel_fro(y_gpu, y_ref):
    y = y_gpu.double().cpu().numpy()
    return float(np.linalg.norm(y - y_ref) / max(np.linalg.norm(y_ref), 1e-300))


LONG = mes.binding.lib.mes_long_segment_tokens()


def check_rows(wl, y, y_ref, oe, w64, one_product=True, what=""):
    """The element-wise bars.  y: the HIP output (all tokens; the output channels the oracle computed), y_ref the
    oracle's, oe the oracle's experts and w64 the base weight for the same output channels.  one_product: the call
    had a workspace sized for its tokens, so segments of LONG tokens or more took the one-product path."""
    yg = y.double().cpu().numpy()
    x64 = wl.x.double().cpu().numpy()
    seg = wl.seg_offsets
    short = np.ones(yg.shape[0], dtype=bool)
    out = {}
    for e, ex in enumerate(oe):
        lo, hi = seg[e], seg[e + 1]
        if one_product and hi - lo >= LONG:
            short[lo:hi] = False
            w_eff = w64 + O.compressed_delta(ex["codes"], ex["step"], ex["salient"], ex["salient_idx"], ex["bits"], ex["grid"])
            out[f"one_product[{e}]"] = PC.assert_one_product_rows(yg[lo:hi], y_ref[lo:hi], x64[lo:hi], w_eff, (what, e))
    if short.any():
        out["streaming"] = PC.assert_streaming_rows(yg[short], y_ref[short], what)
    assert rel_fro(y, y_ref) <= TOL, what
    return out


def check_pack(packed, ora, d_out, d_in, k, bits):
    got = packed.codes.cpu().numpy().view(np.uint32)
    want = O.pack_codes(ora["codes"], bits).reshape(-1)
    assert np.array_equal(got[: want.size], want), "packed code words differ"
    assert np.array_equal(packed.step.cpu().numpy().view(np.uint32), ora["step"].view(np.uint32)), "step bits differ"
    if k:
        gs = packed.salient.cpu().numpy().view(np.uint16)
        assert np.array_equal(gs, O.pack_salient(ora["salient"]).reshape(-1)), "fp16 salient bits differ"


# ------------------------------------------------------------------ offline calls: bit-exact

@pytest.mark.parametrize("d_out,d_in", [(64, 512), (72, 264), (256, 256), (4, 8), (200, 1032)])
def test_pack_base_matches_oracle_layout(d_out, d_in):
    w = synth.normal((d_out, d_in), 0.02, 11 + d_in, dtype=torch.bfloat16)
    t = mes.mes_pack_base(w.to(DEV))
    want = O.pack_base(w.view(torch.int16).numpy().view(np.uint16)).reshape(-1)
    assert np.array_equal(t.cpu().numpy().view(np.uint16), want)
    back = mes.mes_unpack_base(t, d_in, d_out)
    assert torch.equal(back.cpu().view(torch.int16), w.view(torch.int16))


@pytest.mark.parametrize("bits,grid,policy", [(2, 0, 1), (1, 0, 1), (3, 0, 1), (4, 0, 1), (2, 1, 1), (3, 1, 1), (4, 1, 1), (1, 0, 2)])
@pytest.mark.parametrize("d_out,d_in,k", [(256, 256, 8), (72, 264, 5), (64, 1032, 33), (132, 520, 0)])
def test_pack_delta_bit_exact(bits, grid, policy, d_out, d_in, k):
    ex = synth.make_delta(d_in, d_out, k, 0.003, 15.0, 5000 + bits * 7 + d_in)
    c, s, sal = O.quantize(ex.delta.numpy(), ex.salient_idx.numpy(), bits, grid, policy)
    p = mes.mes_pack_delta(ex.delta.to(DEV), ex.salient_idx if k else None, bits, grid, policy)
    check_pack(p, dict(codes=c, step=s, salient=sal), d_out, d_in, k, bits)
    # unpack: codes with 0xFF at salient columns, and the compressed delta rounded once to fp32
    dh, cd = mes.mes_unpack_delta(p)
    assert np.array_equal(cd.cpu().numpy(), c)
    want = O.compressed_delta(c, s, sal, ex.salient_idx.numpy(), bits, grid).astype(np.float32)
    assert np.array_equal(dh.cpu().numpy().view(np.uint32), want.view(np.uint32))
    if k:   # salient columns reproduce fp16(delta) exactly
        got = dh[:, ex.salient_idx.long().to(DEV)].cpu()
        assert torch.equal(got, ex.delta[:, ex.salient_idx.long()].to(torch.float16).float())


def test_pack_delta_given_step_and_zero_rows():
    ex = synth.make_delta(256, 64, 4, 0.003, 15.0, 77)
    step_in = torch.full((64,), 2e-3)
    step_in[3] = 0.0
    step_in[9] = -1.0
    ex.delta[20] = 0.0
    c, s, sal = O.quantize(ex.delta.numpy(), ex.salient_idx.numpy(), 2, 0, O.STEP_GIVEN, step_in.numpy())
    p = mes.mes_pack_delta(ex.delta.to(DEV), ex.salient_idx, 2, 0, mes.STEP_GIVEN, step_in)
    check_pack(p, dict(codes=c, step=s, salient=sal), 64, 256, 4, 2)
    c2, s2, sal2 = O.quantize(ex.delta.numpy(), ex.salient_idx.numpy(), 2, 0, O.STEP_MAXABS)
    p2 = mes.mes_pack_delta(ex.delta.to(DEV), ex.salient_idx, 2)
    assert s2[20] == 0 and float(p2.step[20]) == 0
    check_pack(p2, dict(codes=c2, step=s2, salient=sal2), 64, 256, 4, 2)


def test_pack_delta_rejects_bad_salient_indices():
    d = synth.normal((64, 256), 0.003, 1).to(DEV)
    for bad in ([5, 5, 9], [9, 5], [0, 256], [-1, 3]):
        with pytest.raises(mes.MesError) as e:
            mes.mes_pack_delta(d, torch.tensor(bad, dtype=torch.int32), 2)
        assert e.value.status == 4


@pytest.mark.parametrize("bits,grid", [(2, 0), (2, 1), (3, 0), (1, 0), (4, 1)])
def test_select_salient_indices_bit_exact(bits, grid):
    d_out, d_in, n, k = 96, 264, 40, 8
    ex = synth.make_delta(d_in, d_out, k, 0.003, 15.0, 900 + bits)
    xc = synth.normal((n, d_in), 1.0, 31 + bits)
    idx_o, score_o = O.select_salient(ex.delta.numpy(), xc.numpy(), bits, grid, k)
    idx_g, score_g = mes.mes_select_salient(ex.delta.to(DEV), xc.to(DEV), bits, grid, k, want_scores=True)
    assert np.allclose(score_g.cpu().numpy(), score_o, rtol=1e-11)
    srt = np.sort(score_o)[::-1]
    assert (srt[k - 1] - srt[k]) / srt[k - 1] > 1e-9          # the k-th and (k+1)-th score are not tied
    assert idx_g.cpu().numpy().tolist() == idx_o.tolist()
    assert idx_g.dtype == torch.int32


# ------------------------------------------------------------------ the hot path

def run_case(wl, grid=0, policy=1):
    w_t = mes.mes_pack_base(wl.w_base.to(DEV))
    ge = gpu_experts(wl, grid, policy)
    oe = oracle_experts(wl, grid, policy)
    for p, o in zip(ge, oe):
        check_pack(p, o, wl.d_out, wl.d_in, wl.k, wl.bits)
    y = mes.mes_delta_linear(w_t, ge, wl.x.to(DEV), wl.seg_offsets)
    # ... and in a workspace for a larger batch than this one: every element written, the same bits
    roomy = torch.full_like(y, float("nan"))
    mes.DeltaLinear(w_t, ge, max_tokens=max(256, 2 * y.shape[0]))(wl.x.to(DEV), wl.seg_offsets, roomy)
    torch.cuda.synchronize()
    assert torch.equal(roomy, y), (wl.d_in, wl.d_out, wl.bits, grid, wl.seg_offsets)
    w64 = wl.w_base.double().numpy()
    y_ref = O.delta_linear(wl.x.double().numpy(), w64, oe, wl.seg_offsets)
    check_rows(wl, y, y_ref, oe, w64, what=(wl.d_in, wl.d_out, wl.bits, grid, wl.seg_offsets))
    return y, y_ref


def test_config1():
    y, y_ref = run_case(synth.config1())
    assert y.shape == (4, 256) and y.dtype == torch.bfloat16
    assert rel_fro(y, y_ref) <= TOL


@pytest.mark.parametrize("bits,grid,policy", [(2, 0, 1), (1, 0, 1), (1, 0, 2), (3, 0, 1), (2, 1, 1), (3, 1, 1), (4, 0, 1), (4, 1, 1)])
def test_config1_all_bit_widths_and_grids(bits, grid, policy):
    wl = synth.config1()
    wl.bits = bits
    y, y_ref = run_case(wl, grid, policy)
    assert rel_fro(y, y_ref) <= TOL


@pytest.mark.parametrize("d_in,d_out,seg,k,bits", [
    (264, 72, [0, 3, 3, 20, 37], 5, 2),          # ragged everything, an empty segment, tile-straddling segments
    (1032, 132, [0, 1, 2, 3, 64], 33, 3),        # one-token segments, 64 tokens exactly
    (520, 64, [0, 70, 70, 150], 0, 1),           # more than one 64-token group, no salient channels
    (2048, 320, [0, 0, 0, 5], 16, 2),            # leading empty experts
    (512, 64, [0, 16, 32, 48, 64], 32, 2),       # tile-aligned segments
    (4096, 192, [0, 7, 30, 31, 50, 61], 64, 2),  # several column splits, ragged token tail
    (1160, 200, [0, 5, 5, 21, 40, 64], 24, 4),   # 4-bit codes, ragged shape
])
def test_ragged_shapes_and_segments(d_in, d_out, seg, k, bits):
    wl = synth.small_case(d_in, d_out, seg, k, bits, seed=d_in % 97)
    y, y_ref = run_case(wl)
    assert rel_fro(y, y_ref) <= TOL
    # per-row check too: no single token may be far off
    yg = y.double().cpu().numpy()
    row_err = np.linalg.norm(yg - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)
    assert row_err.max() <= 2 * TOL


def test_routing_is_exact():
    """Experts differ by large, distinct constants: a mis-routed row is off by far more than the tolerance."""
    d_in, d_out = 512, 128
    seg = [0, 1, 1, 18, 33, 47]
    wl = synth.small_case(d_in, d_out, seg, 8, 2, seed=5)
    for e, ex in enumerate(wl.experts):
        ex.delta += 0.01 * (e + 1)
    wl.x = wl.x.abs()
    y, y_ref = run_case(wl)
    yg = y.double().cpu().numpy()
    oe = oracle_experts(wl)
    x64 = wl.x.double().numpy()
    w64 = wl.w_base.double().numpy()
    for t in range(seg[-1]):
        e_true = max(e for e in range(5) if seg[e] <= t)
        errs = []
        for e in range(5):
            alt = O.delta_linear(x64[t:t + 1], w64, [oe[e]], [0, 1])
            errs.append(np.linalg.norm(yg[t] - alt[0]) / np.linalg.norm(alt[0]))
        assert int(np.argmin(errs)) == e_true and errs[e_true] <= TOL and min(errs[:e_true] + errs[e_true + 1:]) > 10 * TOL


def test_empty_batch_and_determinism():
    wl = synth.small_case(1024, 128, [0, 9, 21, 40], 16, 2, seed=8)
    w_t = mes.mes_pack_base(wl.w_base.to(DEV))
    ge = gpu_experts(wl)
    lin = mes.DeltaLinear(w_t, ge, 64)
    y0 = lin(wl.x.to(DEV)[:0], [0, 0, 0, 0])
    assert y0.shape == (0, 128)
    x = wl.x.to(DEV)
    guard = torch.full((42, 128), 7.0, dtype=torch.bfloat16, device=DEV)     # canary rows after y
    y1 = lin(x, wl.seg_offsets, guard[:40])
    torch.cuda.synchronize()
    assert torch.all(guard[40:] == 7.0)
    y2 = lin(x, wl.seg_offsets)
    torch.cuda.synchronize()
    assert torch.equal(y1.view(torch.int16), y2.view(torch.int16))           # run-to-run bitwise equal


def test_special_cases_reduce_to_dense_products():
    wl = synth.small_case(512, 64, [0, 10, 25], 8, 2, seed=12)
    dev_x = wl.x.to(DEV)
    w_t = mes.mes_pack_base(wl.w_base.to(DEV))
    # zero step, no salient channels: the base product alone
    ge = [mes.mes_pack_delta(ex.delta.to(DEV), None, 2, 0, mes.STEP_GIVEN, torch.zeros(64)) for ex in wl.experts]
    y = mes.mes_delta_linear(w_t, ge, dev_x, wl.seg_offsets)
    ref = wl.x.double().numpy() @ wl.w_base.double().numpy().T
    assert rel_fro(y, ref) <= TOL
    PC.assert_streaming_rows(y.double().cpu().numpy(), ref, "base product alone")
    # zero base: the delta term alone
    z_t = mes.mes_pack_base(torch.zeros_like(wl.w_base).to(DEV))
    ge = gpu_experts(wl)
    y = mes.mes_delta_linear(z_t, ge, dev_x, wl.seg_offsets)
    oe = oracle_experts(wl)
    ref = O.delta_linear(wl.x.double().numpy(), np.zeros((64, 512)), oe, wl.seg_offsets)
    assert rel_fro(y, ref) <= TOL
    PC.assert_streaming_rows(y.double().cpu().numpy(), ref, "delta term alone")


@pytest.mark.parametrize("d_in,d_outs,seg,k,bits", [
    (512, [128, 64, 72], [0, 9, 21, 40], 8, 2),          # three layers of different widths, one launch
    (1032, [132, 256], [0, 1, 2, 3, 64], 33, 3),          # ragged widths, 3-bit, 64 tokens
    (4096, [320, 192, 64], [0, 7, 30, 31, 50, 61], 64, 2),   # column splits across the fused row groups
])
def test_fused_layers_match_the_oracle_and_the_single_calls(d_in, d_outs, seg, k, bits):
    """Several layers reading the same activations through one mes_delta_linear_multi call: every layer within
    tolerance of the oracle, and as close to its own single-layer call as two fp32 summation orders can be."""
    wls = [synth.small_case(d_in, d, seg, k, bits, seed=100 + 7 * i + d_in % 97) for i, d in enumerate(d_outs)]
    x = wls[0].x
    layers, oes = [], []
    for wl in wls:
        wl.x = x                                           # the same activations for every layer
        layers.append((mes.mes_pack_base(wl.w_base.to(DEV)), gpu_experts(wl)))
        oes.append(oracle_experts(wl))
    fused = mes.DeltaLinearMulti(layers, 64)
    ys = fused(x.to(DEV), seg)
    torch.cuda.synchronize()
    for wl, (w_t, ge), oe, y in zip(wls, layers, oes, ys):
        y_ref = O.delta_linear(x.double().numpy(), wl.w_base.double().numpy(), oe, seg)
        assert y.shape == (seg[-1], wl.d_out)
        check_rows(wl, y, y_ref, oe, wl.w_base.double().numpy(), one_product=False)
        y_single = mes.mes_delta_linear(w_t, ge, x.to(DEV), seg)
        assert rel_fro(y, y_single.double().cpu().numpy()) <= 4e-3   # both are one bf16 rounding away from the same sum


def test_copy_probe_copies():
    src = torch.arange(1 << 20, dtype=torch.int32, device=DEV)
    dst = torch.zeros_like(src)
    mes.mes_copy_probe(dst, src)
    torch.cuda.synchronize()
    assert torch.equal(dst, src)


def test_config2_full_size():
    """Mistral-7B q_proj shape, 3 experts, 16/16/16 decode tokens; full output against the oracle."""
    y, y_ref = run_case(synth.config2())
    assert rel_fro(y, y_ref) <= TOL


def test_config4_sampled_rows_at_full_size():
    """16 experts, Zipf routing, 64 tokens, gate_proj shape (4096 -> 14336): the HIP path runs at full size in
    the launch configuration the benchmark times; the oracle recomputes a seeded sample of output channels."""
    wl = synth.config4_linear("gate_proj", device=DEV)
    w_t = mes.mes_pack_base(wl.w_base)
    ge = [mes.mes_pack_delta(ex.delta, ex.salient_idx, wl.bits) for ex in wl.experts]
    y = mes.mes_delta_linear(w_t, ge, wl.x, wl.seg_offsets)
    torch.cuda.synchronize()
    g = torch.Generator().manual_seed(99)
    rows = torch.sort(torch.randperm(wl.d_out, generator=g)[:192]).values
    oe = oracle_experts(wl, rows=rows.to(DEV))
    w64 = wl.w_base[rows.to(DEV)].double().cpu().numpy()
    y_ref = O.delta_linear(wl.x.double().cpu().numpy(), w64, oe, wl.seg_offsets)
    check_rows(wl, y[:, rows.to(DEV)], y_ref, oe, w64)
    assert sum(1 for e in range(16) if wl.seg_offsets[e + 1] > wl.seg_offsets[e]) >= 8


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
def test_more_experts_than_one_pass_holds(bits):
    """40 experts, most with one or two tokens, in one 64-token batch: the token group has to be cut where the
    kernel's expert slots run out (16; at 3 and 4 bits in two sweeps), with empty experts sprinkled in."""
    seg = [0]
    for e in range(40):
        seg.append(seg[-1] + (1, 2, 0, 1, 3, 1, 2, 1)[e % 8])      # 55 tokens, 35 experts with tokens
    wl = synth.small_case(640, 80, seg, 24, bits, seed=40 + bits)
    y, y_ref = run_case(wl)
    assert rel_fro(y, y_ref) <= TOL
    yg = y.double().cpu().numpy()
    row_err = np.linalg.norm(yg - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)
    assert row_err.max() <= 2 * TOL


def sampled_rows_check(wl, y, n_rows, seed, grid=0, one_product=True, zero_base=False):
    """The oracle recomputes a seeded sample of output channels for all tokens; element-wise bars on those, the
    relative Frobenius error returned."""
    g = torch.Generator().manual_seed(seed)
    rows = torch.sort(torch.randperm(wl.d_out, generator=g)[:n_rows]).values.to(DEV)
    oe = oracle_experts(wl, grid=grid, rows=rows)
    w64 = wl.w_base[rows].double().cpu().numpy()
    if zero_base:
        w64 = np.zeros_like(w64)
    y_ref = O.delta_linear(wl.x.double().cpu().numpy(), w64, oe, wl.seg_offsets)
    rep = check_rows(wl, y[:, rows], y_ref, oe, w64, one_product=one_product, what=(wl.name, wl.bits, grid))
    print(wl.name, wl.bits, {k: {a: float(f"{b:.4g}") for a, b in v.items()} for k, v in rep.items()})
    return rel_fro(y[:, rows], y_ref)


@pytest.mark.parametrize("bits,which", [(1, "down_proj"), (3, "down_proj"), (3, "q_proj"), (4, "down_proj"), (4, "q_proj")])
def test_config4_other_bit_widths_at_full_size(bits, which):
    """The 1- and 3-bit code paths at a full Mistral-7B shape with 16 experts (the 14336-wide input of
    down_proj is the longest reduction any config has)."""
    wl = synth.config4_linear(which, device=DEV, bits=bits)
    w_t = mes.mes_pack_base(wl.w_base)
    ge = [mes.mes_pack_delta(ex.delta, ex.salient_idx, wl.bits) for ex in wl.experts]
    y = mes.mes_delta_linear(w_t, ge, wl.x, wl.seg_offsets)
    torch.cuda.synchronize()
    assert sampled_rows_check(wl, y, 96, 5 + bits) <= TOL


def test_config4_fused_calls_at_full_size():
    """The launch configuration the benchmark times: q+k+v in one call and gate+up in one call, 16 experts,
    64 Zipf-routed tokens, every layer checked on sampled output channels."""
    for names in (["q_proj", "k_proj", "v_proj"], ["gate_proj", "up_proj"]):
        wls = [synth.config4_linear(n, device=DEV) for n in names]
        assert all(torch.equal(w.x, wls[0].x) for w in wls)
        layers = [(mes.mes_pack_base(w.w_base), [mes.mes_pack_delta(ex.delta, ex.salient_idx, w.bits) for ex in w.experts])
                  for w in wls]
        ys = mes.DeltaLinearMulti(layers, 64)(wls[0].x, wls[0].seg_offsets)
        torch.cuda.synchronize()
        for i, (w, y) in enumerate(zip(wls, ys)):
            assert y.shape == (64, w.d_out)
            assert sampled_rows_check(w, y, 64, 300 + i) <= TOL
        del wls, layers, ys
        torch.cuda.empty_cache()


@pytest.mark.parametrize("which,n_tokens,bits", [("q_proj", 256, 2), ("down_proj", 200, 2), ("gate_proj", 130, 3),
                                                  ("down_proj", 256, 4), ("o_proj", 65, 1)])
def test_config4_several_token_groups_in_one_launch(which, n_tokens, bits):
    """65 .. 256 decode tokens at full size: one launch serves up to four 64-token groups (its workgroups share the
    base weights through L2).  Element-wise bars against the oracle on sampled channels, and bit-for-bit the result
    of the same call made with a workspace that only has room for one group per launch."""
    wl = synth.config4_linear(which, device=DEV, n_tokens=n_tokens, bits=bits)
    assert max(b - a for a, b in zip(wl.seg_offsets, wl.seg_offsets[1:])) < LONG
    w_t = mes.mes_pack_base(wl.w_base)
    ge = [mes.mes_pack_delta(ex.delta, ex.salient_idx, wl.bits) for ex in wl.experts]
    y = mes.mes_delta_linear(w_t, ge, wl.x, wl.seg_offsets)
    ws1 = mes.make_workspace(wl.d_in, wl.d_out, 64, torch.device(DEV))
    y1 = mes.mes_delta_linear(w_t, ge, wl.x, wl.seg_offsets, workspace=ws1)
    torch.cuda.synchronize()
    assert torch.equal(y, y1)
    assert sampled_rows_check(wl, y, 96, seed=7 + n_tokens, one_product=False) <= TOL


@pytest.mark.parametrize("which", ["gate_proj", "up_proj", "down_proj"])
@pytest.mark.parametrize("bits", [2, 3])
def test_config3_prefill_sampled_rows(bits, which):
    """Three experts with one 512-token sequence each (24 token groups over the same weights), 128 salient
    channels; the oracle recomputes sampled output channels for all 1536 tokens."""
    wl = synth.config3(which, bits=bits, device=DEV)
    w_t = mes.mes_pack_base(wl.w_base)
    ge = [mes.mes_pack_delta(ex.delta, ex.salient_idx, wl.bits) for ex in wl.experts]
    y = mes.mes_delta_linear(w_t, ge, wl.x, wl.seg_offsets)
    torch.cuda.synchronize()
    assert y.shape == (1536, wl.d_out)
    assert sampled_rows_check(wl, y, 64, 11 + bits) <= TOL


@pytest.mark.parametrize("k,bits,grid", [(8, 2, 1), (32, 2, 0), (16, 4, 1), (0, 2, 0)])
def test_config4_salient_counts_and_eq1_grid_at_full_size(k, bits, grid):
    """The paper's sweep of the number of fp16 channels (8 to 64) and the Eq. 1 grid, at the o_proj shape with 16
    experts; k = 0 is the fixed-precision baseline of the paper's comparison."""
    wl = synth.config4_linear("o_proj", device=DEV, bits=bits, k=k)
    w_t = mes.mes_pack_base(wl.w_base)
    ge = [mes.mes_pack_delta(ex.delta, ex.salient_idx if k else None, wl.bits, grid) for ex in wl.experts]
    y = mes.mes_delta_linear(w_t, ge, wl.x, wl.seg_offsets)
    torch.cuda.synchronize()
    g = torch.Generator().manual_seed(17 + k)
    rows = torch.sort(torch.randperm(wl.d_out, generator=g)[:96]).values.to(DEV)
    oe = oracle_experts(wl, grid=grid, rows=rows)
    w64 = wl.w_base[rows].double().cpu().numpy()
    y_ref = O.delta_linear(wl.x.double().cpu().numpy(), w64, oe, wl.seg_offsets)
    check_rows(wl, y[:, rows], y_ref, oe, w64)


def test_on_demand_swapping_gives_the_resident_result():
    """20 experts registered in pinned host memory, 6 device slots.  Every batch acquires the experts it routes to
    (least recently used slots are overwritten) and must give, bit for bit, what the same call gives on the
    always-resident packed deltas; one batch is also checked against the oracle, and the hit / miss counts
    against the policy oracle."""
    from oracle.pool_oracle import LruPool
    d_in, d_out, k, bits, n_experts, n_slots = 520, 136, 16, 2, 20, 6
    wl = synth.small_case(d_in, d_out, [0] + [3 * (e + 1) for e in range(n_experts)], k, bits, seed=61)   # only the experts are used
    w_t = mes.mes_pack_base(wl.w_base.to(DEV))
    ge = gpu_experts(wl)
    pool = mes.ExpertPool(d_in, d_out, k, bits, 0, n_slots, n_experts, device=DEV)
    for e, pk in enumerate(ge):
        pool.register(e, pk)
    ws = mes.make_workspace(d_in, d_out, 64, torch.device(DEV))
    ref = LruPool(n_slots)
    rng = np.random.default_rng(5)
    oe = oracle_experts(wl)
    for step in range(12):
        ids = sorted(rng.choice(n_experts, size=int(rng.integers(1, n_slots + 1)), replace=False).tolist())
        counts = rng.integers(1, 9, size=len(ids))
        seg = [0] + np.cumsum(counts).tolist()
        x = synth.normal((seg[-1], d_in), 1.0, 700 + step, DEV, torch.bfloat16)
        ref.acquire(ids)
        desc = pool.acquire(ids)
        y_pool = mes.mes_delta_linear_descriptors(w_t, desc, x, seg, ws)
        y_res = mes.mes_delta_linear(w_t, [ge[e] for e in ids], x, seg)
        torch.cuda.synchronize()
        assert torch.equal(y_pool.view(torch.int16), y_res.view(torch.int16)), f"batch {step}"
        if step == 7:
            y_ref = O.delta_linear(x.double().cpu().numpy(), wl.w_base.double().numpy(), [oe[e] for e in ids], seg)
            assert rel_fro(y_pool, y_ref) <= TOL
            PC.assert_streaming_rows(y_pool.double().cpu().numpy(), y_ref, "swapped-in experts")
    hits, misses, nbytes = pool.stats()
    assert (hits, misses) == (ref.hits, ref.misses) and misses > n_slots          # slots were really recycled
    assert nbytes == misses * (mes.codes_bytes(d_in, d_out, bits) + 4 * d_out + mes.salient_bytes(d_out, k) + 4 * k)


def gated_case(d_in, d_out, seg, k, bits, seed, device="cpu", grid=0):
    """Two layers over the same activations and routing (gate, up), oracle result and HIP result of the gated call."""
    wg = synth.small_case(d_in, d_out, seg, k, bits, seed=seed, device=device)
    wu = synth.small_case(d_in, d_out, seg, k, bits, seed=seed + 1, device=device)
    x = wg.x.to(DEV)
    packed = []
    for wl in (wg, wu):
        packed.append((mes.mes_pack_base(wl.w_base.to(DEV)),
                       [mes.mes_pack_delta(ex.delta.to(DEV), ex.salient_idx if k else None, bits, grid) for ex in wl.experts]))
    lin = mes.DeltaLinearGated(packed[0][0], packed[0][1], packed[1][0], packed[1][1], max_tokens=seg[-1])
    h = lin(x, seg)
    torch.cuda.synchronize()
    return wg, wu, packed, h


@pytest.mark.parametrize("d_in,d_out,seg,k,bits,grid", [
    (264, 72, [0, 3, 3, 20, 37], 5, 2, 0),               # ragged shape, an empty segment, one row group half empty
    (4096, 192, [0, 7, 30, 31, 50, 61], 64, 2, 0),       # the columns are split over workgroups: the reduction applies the gate
    (1160, 200, [0, 5, 5, 21, 40, 64, 150], 24, 4, 1),   # 4-bit codes, Eq. 1 grid, three token groups
    (520, 1024, [0, 300], 16, 3, 0),                     # a long segment: the gated call streams it all the same
    (640, 80, [0] + [i + 1 for i in range(20)], 24, 1, 0),   # 20 experts with one token each, 1 bit
])
def test_gated_mlp_input_matches_the_oracle(d_in, d_out, seg, k, bits, grid):
    """h = SiLU(y_gate) * y_up in one pass: against the fp64 oracle (which rounds nothing on the way) on every
    element, within one bf16 ulp on all but a few per thousand (streaming arithmetic: exact products, fp32 sums, one
    rounding)."""
    wg, wu, packed, h = gated_case(d_in, d_out, seg, k, bits, seed=31 + bits, grid=grid)
    x64 = wg.x.double().numpy()
    h_ref = O.gated_mlp_input(x64, wg.w_base.double().numpy(), oracle_experts(wg, grid), wu.w_base.double().numpy(),
                              oracle_experts(wu, grid), seg)
    assert rel_fro(h, h_ref) <= TOL
    PC.assert_streaming_rows(h.double().cpu().numpy(), h_ref, ("gated", d_in, d_out, bits))
    # and the two layers alone, combined on the host in fp64 from their bf16 outputs, agree to bf16 accuracy
    yg = mes.mes_delta_linear(packed[0][0], packed[0][1], wg.x.to(DEV), seg).double().cpu().numpy()
    yu = mes.mes_delta_linear(packed[1][0], packed[1][1], wg.x.to(DEV), seg).double().cpu().numpy()
    assert rel_fro(h, O.silu(yg) * yu) <= 2 * TOL


def test_gated_mlp_input_at_full_size():
    """gate_proj and up_proj of the 16-expert decode batch (4096 -> 14336, 64 tokens, Zipf routing) through the gated
    call; the oracle recomputes a seeded sample of output channels."""
    wg = synth.config4_linear("gate_proj", device=DEV)
    wu = synth.config4_linear("up_proj", device=DEV)
    assert torch.equal(wg.x, wu.x) and wg.seg_offsets == wu.seg_offsets
    packed = [(mes.mes_pack_base(wl.w_base), [mes.mes_pack_delta(ex.delta, ex.salient_idx, wl.bits) for ex in wl.experts]) for wl in (wg, wu)]
    h = mes.DeltaLinearGated(packed[0][0], packed[0][1], packed[1][0], packed[1][1], 64)(wg.x, wg.seg_offsets)
    torch.cuda.synchronize()
    g = torch.Generator().manual_seed(123)
    rows = torch.sort(torch.randperm(wg.d_out, generator=g)[:128]).values.to(DEV)
    x64 = wg.x.double().cpu().numpy()
    h_ref = O.gated_mlp_input(x64, wg.w_base[rows].double().cpu().numpy(), oracle_experts(wg, rows=rows),
                              wu.w_base[rows].double().cpu().numpy(), oracle_experts(wu, rows=rows), wg.seg_offsets)
    assert rel_fro(h[:, rows], h_ref) <= TOL
    PC.assert_streaming_rows(h[:, rows].double().cpu().numpy(), h_ref, "gated gate+up at full size")


def test_layer_spanning_pool_with_prefetch_gives_the_resident_result():
    """A pool whose slots hold an expert's deltas of three linear layers (two of them read the same activations and go
    through one fused call), one pinned blob and one copy per expert.  After every acquire the next batch's experts
    are prefetched -- those copies run under the current batch's kernels and may only go to slots the current batch
    does not use.  Every batch must give, bit for bit, what the always-resident packed deltas give; residency and
    counters must follow the policy oracle."""
    from oracle.pool_oracle import LruPool
    shapes = [(520, 136, 16), (520, 72, 16), (264, 200, 8)]            # (d_in, d_out, k)
    bits, n_experts, n_slots = 2, 18, 8
    wls = [synth.small_case(di, do, [0] + [e + 1 for e in range(n_experts)], k, bits, seed=70 + i) for i, (di, do, k) in enumerate(shapes)]
    w_t = [mes.mes_pack_base(wl.w_base.to(DEV)) for wl in wls]
    ge = [gpu_experts(wl) for wl in wls]
    pool = mes.ExpertPool([s[0] for s in shapes], [s[1] for s in shapes], [s[2] for s in shapes], bits, 0, n_slots, n_experts, device=DEV)
    for e in range(n_experts):
        pool.register(e, [ge[l][e] for l in range(3)])
    ws_a = torch.empty(mes.DeltaLinearMulti.workspace_bytes(520, [136, 72], 64), dtype=torch.uint8, device=DEV)
    ws_b = mes.make_workspace(264, 200, 64, torch.device(DEV))
    ref = LruPool(n_slots)
    rng = np.random.default_rng(9)
    batches = []
    for step in range(14):
        ids = sorted(rng.choice(n_experts, size=int(rng.integers(1, 5)), replace=False).tolist())
        batches.append((ids, [0] + np.cumsum(rng.integers(1, 12, size=len(ids))).tolist()))
    for step, (ids, seg) in enumerate(batches):
        xa = synth.normal((seg[-1], 520), 1.0, 800 + step, DEV, torch.bfloat16)
        xb = synth.normal((seg[-1], 264), 1.0, 900 + step, DEV, torch.bfloat16)
        ref.acquire(ids)
        desc = pool.acquire(ids)
        ya = mes.mes_delta_linear_multi_descriptors(w_t[:2], desc[:2], xa, seg, ws_a)
        yb = mes.mes_delta_linear_descriptors(w_t[2], desc[2], xb, seg, ws_b)
        if step + 1 < len(batches):
            assert pool.prefetch(batches[step + 1][0]) == len(ref.prefetch(batches[step + 1][0]))
        # the same calls on the resident deltas (the fused one included: its column split differs from a single call's)
        res = mes.DeltaLinearMulti([(w_t[l], [ge[l][e] for e in ids]) for l in range(2)], 64)(xa, seg)
        res.append(mes.mes_delta_linear(w_t[2], [ge[2][e] for e in ids], xb, seg))
        torch.cuda.synchronize()
        for l, y in enumerate(ya + [yb]):
            assert torch.equal(y.view(torch.int16), res[l].view(torch.int16)), f"batch {step}, layer {l}"
        for e in range(n_experts):
            assert pool.slot_of(e) == ref.slot_of(e)
    hits, misses, _ = pool.stats()
    assert (hits, misses, pool.prefetched()) == (ref.hits, ref.misses, ref.prefetched)
    assert pool.prefetched() > n_slots and misses < pool.prefetched()       # slots recycled by prefetches; most loads were ahead of need


@pytest.mark.parametrize("d_in,d_out,seg,k,bits,grid", [
    (520, 136, [0, 5, 305, 310, 330, 560], 16, 2, 0),     # long segments (300 and 230 tokens) between short ones
    (1032, 72, [0, 200], 33, 3, 1),                        # one long segment only, Eq. 1 grid, 3 bits
    (264, 200, [0, 0, 192, 400, 401], 0, 4, 0),            # exactly at the threshold, no salient channels, 4 bits
    (512, 64, [0, 250, 260], 8, 1, 0),                     # 1 bit
    (640, 136, [0, 3, 703, 710], 136, 2, 0),               # 700 tokens: 3 token blocks; 136 salient channels: 2 salient
                                                           # steps; 136 rows: the second row group is half padding
    (1280, 72, [0, 300, 600], 40, 3, 1),                   # two long segments, few rows: the contraction is split 3 ways
    (2048, 520, [0, 513], 64, 4, 0),                       # 513 tokens (a ragged third token block), 4 bits
    (264, 72, [0, 200, 205, 405, 605, 805, 1005, 1205, 1405, 1605, 1805, 1810, 2010, 2300], 5, 2, 0),
                                                           # 11 long segments: two launches of the fused kernel (8 + 3)
    (264, 5504, [0, 512, 1000, 1536], 16, 2, 0),           # 344 row tiles x 7 token blocks: the plan takes 7 row tiles
                                                           # per workgroup, and the last group has one tile of its own
    (264, 5504, [0, 512, 1000, 1536], 16, 1, 0),           # the same plan at 1, 3 and 4 bits
    (264, 5504, [0, 512, 1000, 1536], 40, 3, 1),
    (264, 5504, [0, 512, 1000, 1536], 0, 4, 0),
])
def test_long_segments_take_the_one_product_path(d_in, d_out, seg, k, bits, grid):
    """Expert segments of 192 tokens or more are computed as x (W + Delta~)^T by the fused one-product kernel (the
    effective weight formed in registers); the rest of the batch streams as usual.  Every row against the oracle."""
    wl = synth.small_case(d_in, d_out, seg, k, bits, seed=300 + bits)
    y, y_ref = run_case(wl, grid)
    assert rel_fro(y, y_ref) <= TOL
    yg = y.double().cpu().numpy()
    row_err = np.linalg.norm(yg - y_ref, axis=1) / np.linalg.norm(y_ref, axis=1)
    assert row_err.max() <= 2 * TOL
    # a workspace without the extra room keeps the whole batch on the streaming path: same result within rounding
    w_t = mes.mes_pack_base(wl.w_base.to(DEV))
    ge = gpu_experts(wl, grid)
    small_ws = mes.make_workspace(d_in, d_out, 64, torch.device(DEV))
    y_stream = mes.mes_delta_linear(w_t, ge, wl.x.to(DEV), wl.seg_offsets, workspace=small_ws)
    torch.cuda.synchronize()
    check_rows(wl, y_stream, y_ref, oracle_experts(wl, grid), wl.w_base.double().numpy(), one_product=False)
    assert rel_fro(y, y_stream.double().cpu().numpy()) <= 4e-3


def test_long_segments_with_a_workspace_sized_for_fewer_tokens():
    """All long segments of a call are re-tiled into the scratch together.  A workspace sized for 512 tokens serves a
    call with one 300-token segment on the one-product path and keeps a call with three of them (900 tokens of long
    segments) on the streaming path; both must match the oracle."""
    d_in, d_out = 392, 136
    ws = mes.make_workspace(d_in, d_out, 512, torch.device(DEV))
    for seg in ([0, 5, 305, 330], [0, 300, 600, 900, 910]):
        wl = synth.small_case(d_in, d_out, seg, 6, 2, seed=600 + len(seg))
        w_t = mes.mes_pack_base(wl.w_base.to(DEV))
        y = mes.mes_delta_linear(w_t, gpu_experts(wl), wl.x.to(DEV), wl.seg_offsets, workspace=ws)
        torch.cuda.synchronize()
        oe = oracle_experts(wl)
        y_ref = O.delta_linear(wl.x.double().numpy(), wl.w_base.double().numpy(), oe, wl.seg_offsets)
        check_rows(wl, y, y_ref, oe, wl.w_base.double().numpy(), one_product=(len(seg) == 4))


def test_long_segments_in_a_fused_call():
    d_in, seg = 512, [0, 4, 210, 230]
    wls = [synth.small_case(d_in, d, seg, 8, 2, seed=400 + i) for i, d in enumerate([128, 72])]
    x = wls[0].x
    layers = [(mes.mes_pack_base(w.w_base.to(DEV)), gpu_experts(w)) for w in wls]
    ys = mes.DeltaLinearMulti(layers, seg[-1])(x.to(DEV), seg)
    torch.cuda.synchronize()
    for w, y in zip(wls, ys):
        oe = oracle_experts(w)
        y_ref = O.delta_linear(x.double().numpy(), w.w_base.double().numpy(), oe, seg)
        w.x = x
        check_rows(w, y, y_ref, oe, w.w_base.double().numpy())


@pytest.mark.parametrize("seed", range(12))
def test_random_shapes_routing_and_settings(seed):
    """Seeded random cases: shapes that are no multiple of any tile size, random routing with empty experts, every
    bit width, both grids, any number of salient channels; batches of up to 300 tokens so that token groups, slot
    sweeps and (sometimes) the long-segment path all occur."""
    rng = np.random.default_rng(1000 + seed)
    d_in = int(rng.integers(1, 160)) * 8
    d_out = int(rng.integers(1, 70)) * 4
    bits = int(rng.integers(1, 5))
    grid = int(rng.integers(0, 2)) if bits > 1 else 0
    k = int(rng.integers(0, min(d_in, 48) + 1))
    n_experts = int(rng.integers(1, 25))
    sizes = rng.choice([0, 0, 1, 2, 3, 5, 9, 17, 40, 70, 200], size=n_experts)
    seg = [0] + np.cumsum(sizes).tolist()
    if seg[-1] == 0:
        seg[-1] = 3
    wl = synth.small_case(d_in, d_out, seg, k, bits, seed=50 + seed)
    y, y_ref = run_case(wl, grid)
    assert y.shape == (seg[-1], d_out)
    assert rel_fro(y, y_ref) <= TOL, (d_in, d_out, bits, grid, k, seg)
    yg = y.double().cpu().numpy()
    row_err = np.linalg.norm(yg - y_ref, axis=1) / np.maximum(np.linalg.norm(y_ref, axis=1), 1e-30)
    assert row_err.max() <= 2.5 * TOL, (d_in, d_out, bits, grid, k, seg)


# ------------------------------------------------------------------ the delta term alone, at a full shape

@pytest.mark.parametrize("bits", [1, 2, 3, 4])
def test_zero_base_streaming_path_at_full_size(bits):
    """Eq. 4's second term alone (W = 0) at the o_proj shape, 16 experts, 64 Zipf-routed tokens: nothing of the
    base product is there to hide an error of the low-bit or the salient product."""
    wl = synth.config4_linear("o_proj", device=DEV, bits=bits)
    z_t = mes.mes_pack_base(torch.zeros_like(wl.w_base))
    ge = [mes.mes_pack_delta(ex.delta, ex.salient_idx, wl.bits) for ex in wl.experts]
    y = mes.mes_delta_linear(z_t, ge, wl.x, wl.seg_offsets)
    torch.cuda.synchronize()
    assert sampled_rows_check(wl, y, 128, 700 + bits, zero_base=True) <= TOL


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
def test_zero_base_one_product_path_at_full_size(bits):
    """The same on the one-product path: three 512-token segments at the q_proj shape; the operand is bf16(Delta~)."""
    wl = synth.make_linear("zero_base_long", 4096, 4096, 3, [0, 512, 1024, 1536], 128, bits, 31, device=DEV)
    z_t = mes.mes_pack_base(torch.zeros_like(wl.w_base))
    ge = [mes.mes_pack_delta(ex.delta, ex.salient_idx, wl.bits) for ex in wl.experts]
    y = mes.mes_delta_linear(z_t, ge, wl.x, wl.seg_offsets)
    torch.cuda.synchronize()
    assert sampled_rows_check(wl, y, 96, 800 + bits, zero_base=True) <= TOL


# ------------------------------------------------------------------ the mixed batch of the 32-layer configuration

@pytest.mark.parametrize("bits", [1, 2, 3])
@pytest.mark.parametrize("which", ["gate_proj", "down_proj"])
def test_config5_mixed_batch_one_layer(which, bits):
    """One layer's gate_proj / down_proj of the 32-layer configuration: 16 experts, 256 Zipf-routed decode tokens and
    4 x 1024 prompt tokens in ONE call (4352 tokens: long segments on the one-product path, everything else streaming),
    sampled output channels against the oracle."""
    wl = synth.config5_linear(which, layer=1, bits=bits, device=DEV)
    assert wl.x.shape[0] == 4352 and max(b - a for a, b in zip(wl.seg_offsets[:-1], wl.seg_offsets[1:])) >= 1024
    w_t = mes.mes_pack_base(wl.w_base)
    ge = [mes.mes_pack_delta(ex.delta, ex.salient_idx, wl.bits) for ex in wl.experts]
    y = mes.mes_delta_linear(w_t, ge, wl.x, wl.seg_offsets)
    torch.cuda.synchronize()
    assert y.shape == (4352, wl.d_out)
    assert sampled_rows_check(wl, y, 48, 900 + bits) <= TOL


# ------------------------------------------------------------------ offline calls at the widest shape

def test_select_and_pack_at_the_widest_shape():
    """mes_select_salient and mes_pack_delta on a 4096 x 14336 delta (down_proj): indices, code words, steps and
    fp16 bits against the oracle."""
    d_out, d_in, k, bits, n = 4096, 14336, 64, 2, 6
    ex = synth.make_delta(d_in, d_out, k, 0.003, 15.0, 4321, DEV)
    xc = synth.normal((n, d_in), 1.0, 77, DEV)
    d_host = ex.delta.cpu().numpy()
    idx_g, score_g = mes.mes_select_salient(ex.delta, xc, bits, mes.GRID_EQ1, k, want_scores=True)
    idx_o, score_o = O.select_salient(d_host, xc.cpu().numpy(), bits, O.GRID_EQ1, k)
    assert np.allclose(score_g.cpu().numpy(), score_o, rtol=1e-11)
    srt = np.sort(score_o)[::-1]
    assert (srt[k - 1] - srt[k]) / srt[k - 1] > 1e-9
    assert idx_g.cpu().numpy().tolist() == idx_o.tolist()
    assert idx_o.tolist() == ex.salient_idx.tolist()            # Eq. 1's grid finds the planted outlier channels
    p = mes.mes_pack_delta(ex.delta, idx_g.cpu(), bits)
    c, s, sal = O.quantize(d_host, idx_o, bits)
    check_pack(p, dict(codes=c, step=s, salient=sal), d_out, d_in, k, bits)
