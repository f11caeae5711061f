"""Packing and salient selection at the sizes where their kernels change: row lengths around the block's register
capacity, matrices that are only 4-byte aligned, weights planted on and next to the grid's decision boundaries, steps at
both ends of fp32's range.  Everything that is stored is compared bit for bit with the oracle."""
import numpy as np
import pytest
import torch

from oracle import mes_oracle as O

pytestmark = pytest.mark.gpu
mes = pytest.importorskip("paper_2406_09041_amd")
DEV = "cuda:0"


def on_gpu(a, aligned=True):
    """A contiguous GPU copy of a; with aligned=False it starts 4 bytes past a 16-byte boundary."""
    t = torch.from_numpy(a)
    if aligned:
        return t.to(DEV)
    room = torch.empty(t.numel() + 4, dtype=t.dtype, device=DEV)
    out = room[1:1 + t.numel()].view(t.shape)
    out.copy_(t)
    assert out.data_ptr() % 16 == 4
    return out


def planted(d_out, d_in, bits, step, rng):
    """Weights at (half) integer multiples of the row's step, one float above and below them, and random ones."""
    with np.errstate(over="ignore", under="ignore"):
        m = rng.integers(-2 ** bits - 2, 2 ** bits + 3, (d_out, d_in)) * 0.5
        w = (m * step.astype(np.float64)[:, None]).astype(np.float32)
        kind = rng.integers(0, 4, (d_out, d_in))
        w = np.where(kind == 1, np.nextafter(w, np.float32(np.inf)), w)
        w = np.where(kind == 2, np.nextafter(w, np.float32(-np.inf)), w)
        noise = (rng.standard_normal((d_out, d_in)) * 2 ** (bits - 1) * np.where(step > 0, step, 1).astype(np.float64)[:, None]).astype(np.float32)
        w = np.where(kind == 3, noise, w).astype(np.float32)
    return np.where(np.isfinite(w), w, np.float32(0.0))


def check(p, codes, step, sal, bits, k):
    want = O.pack_codes(codes, bits).reshape(-1)
    assert np.array_equal(p.codes.cpu().numpy().view(np.uint32)[: want.size], want)
    assert np.array_equal(p.step.cpu().numpy().view(np.uint32), step.view(np.uint32))
    if k:
        assert np.array_equal(p.salient.cpu().numpy().view(np.uint16), O.pack_salient(sal).reshape(-1))


@pytest.mark.parametrize("bits,grid", [(1, 0), (2, 0), (2, 1), (3, 0), (3, 1), (4, 0), (4, 1)])
@pytest.mark.parametrize("d_in", [8, 1024, 1032, 4096, 4104, 8200, 16384, 16392])
def test_codes_at_the_decision_boundaries(d_in, bits, grid):
    d_out, k = 20, min(33, d_in // 2)
    rng = np.random.default_rng(d_in + 10 * bits + grid)
    step = (10.0 ** rng.uniform(-4, 1, d_out)).astype(np.float32)
    step[:8] = [2.0 ** -10, 2.0 ** -101, 1e-38, 2.0 ** 101, 0.0, -1.0, 3e38, 1e-44]
    w = planted(d_out, d_in, bits, np.maximum(step, 0), rng)
    w[9, :4] = [0.0, -0.0, 1e-45, -1e-45]
    sidx = np.sort(rng.choice(d_in, k, replace=False)).astype(np.int32)
    with np.errstate(over="ignore"):
        codes, s, sal = O.quantize(w, sidx, bits, grid, O.STEP_GIVEN, step)
    for aligned in (True, False):
        p = mes.mes_pack_delta(on_gpu(w, aligned), torch.from_numpy(sidx), bits, grid, mes.STEP_GIVEN, torch.from_numpy(step))
        check(p, codes, s, sal, bits, k)


@pytest.mark.parametrize("bits,policy", [(1, 1), (1, 2), (2, 1)])
@pytest.mark.parametrize("d_out,d_in,k", [(4, 8, 8), (60, 1000, 3), (68, 1032, 64), (132, 72, 40), (64, 16392, 5)])
def test_initial_steps_are_the_oracles_bits(d_out, d_in, k, bits, policy):
    rng = np.random.default_rng(d_in + d_out)
    w = (rng.standard_normal((d_out, d_in)) * 10.0 ** rng.uniform(-6, 0, (d_out, d_in))).astype(np.float32)
    w[1] = 0.0
    sidx = np.sort(rng.choice(d_in, k, replace=False)).astype(np.int32)
    codes, s, sal = O.quantize(w, sidx, bits, 0, policy)
    check(mes.mes_pack_delta(on_gpu(w, False), torch.from_numpy(sidx), bits, 0, policy), codes, s, sal, bits, k)


@pytest.mark.parametrize("d_out,d_in,n,k,bits,grid", [(4, 8, 1, 8, 2, 0), (300, 24, 7, 1, 1, 0), (260, 1032, 257, 64, 3, 1),
                                                      (12, 2056, 3, 2000, 4, 0), (1000, 136, 300, 17, 2, 1)])
def test_selection_with_equal_scores(d_out, d_in, n, k, bits, grid):
    """Columns 1 and 5 are copies of columns 0 and 4, activations included: their scores are equal and the lower index
    wins.  A score is the product of two fp64 sums of terms of one sign, n squares and d_out squares of differences: kernel
    and oracle may take the terms in any order and round each a few times, at most (n + d_out + 8) 2^-53 relative each."""
    rng = np.random.default_rng(d_in)
    w = (rng.standard_normal((d_out, d_in)) * 0.003 * 10.0 ** rng.uniform(0, 1, d_in)).astype(np.float32)
    x = rng.standard_normal((n, d_in)).astype(np.float32)
    for a in (w, x):
        a[:, 1], a[:, 5] = a[:, 0], a[:, 4]
    idx_o, score_o = O.select_salient(w, x, bits, grid, k)
    for aligned in (True, False):
        idx, score = mes.mes_select_salient(on_gpu(w, aligned), on_gpu(x, aligned), bits, grid, k, want_scores=True)
        got = score.cpu().numpy()
        rtol = 2 * (n + d_out + 8) * 2.0 ** -53
        assert np.allclose(got, score_o, rtol=rtol, atol=0)
        assert got[0] == got[1] and got[4] == got[5]
        order = np.lexsort((np.arange(d_in), -got))[:k]
        assert idx.cpu().numpy().tolist() == np.sort(order).tolist()
        # the oracle's own choice: no other score is so close to the k-th that the sums' order could decide (equal columns
        # apart, which both sides give to the lower index)
        kth = np.sort(score_o)[::-1][k - 1]
        other = np.delete(score_o, np.flatnonzero(score_o == kth))
        assert (np.abs(other - kth) > 2 * rtol * kth).all()
        assert idx.cpu().numpy().tolist() == idx_o.tolist()
