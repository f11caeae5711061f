"""The last step of every path, fp32 sum -> bf16: to nearest, ties to even, over to infinity where the format ends, NaN stays
NaN.  Outputs are sums of two weights that fp32 holds exactly, planted on and next to the middle between two bf16 numbers."""
import pytest
import torch

pytestmark = pytest.mark.gpu
mes = pytest.importorskip("paper_2406_09041_amd")
DEV = "cuda:0"


def planted(n):
    """(a, b), bf16: b is half a spacing of a, a little more or less than that, or some other part of one; both signs."""
    g = torch.Generator().manual_seed(17)
    m = torch.randint(128, 256, (n,), generator=g).float()
    e = torch.randint(-60, 60, (n,), generator=g).float()
    e[:16] = 120.0                                                       # the largest exponent: 2^127
    m[:8] = 255.0                                                        # ... and the largest number of the format
    part = torch.tensor([0.5, 0.50390625, 0.498046875, 0.25, 0.75, 0.996, 1.5, 0.0])[torch.arange(n) % 8]
    part[:16] = part[:16].clamp(max=0.996)                               # (fp32 ends there as well)
    a = m * 2.0 ** e * torch.where(torch.arange(n) // 8 % 2 == 0, 1.0, -1.0)
    b = part * 2.0 ** e * torch.where(torch.rand(n, generator=g) < 0.5, a.sign(), -a.sign())
    b[:8] = b[:8].abs()                                                  # from the middle on: infinity
    a[-4:] = torch.tensor([float("inf"), float("-inf"), float("nan"), 0.0])
    return a.bfloat16(), b.bfloat16()


@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("tokens", [1, 17, 40, 200])
def test_results_are_rounded_to_nearest_even(tokens, gated):
    """1 and 17 tokens: one launch; 40: the streaming path; 200: the one-product path (the gated pair streams).  d_in of 1032
    splits the columns of the streaming path over workgroups.  Gated: up = 1 in one column and gate so large that SiLU(gate) = gate
    up to a sign of zero, where positive."""
    d_in, d_out = 1032, 512
    a, b = planted(d_out)
    w = torch.zeros((d_out, d_in), dtype=torch.bfloat16)
    w[:, 3], w[:, 1000] = a, b
    want = a.float() + b.float()
    assert torch.equal(want[:-4].double(), a[:-4].double() + b[:-4].double())
    x = torch.zeros((tokens, d_in), dtype=torch.bfloat16)
    x[:, 3] = x[:, 1000] = 1.0
    blank = mes.mes_pack_delta(torch.zeros((d_out, d_in), device=DEV), None, 2)
    w_t = mes.mes_pack_base(w.to(DEV))
    if gated:
        up = torch.zeros_like(w)
        up[:, 3] = 1.0
        y = mes.DeltaLinearGated(w_t, [blank], mes.mes_pack_base(up.to(DEV)), [blank], max_tokens=tokens)(x.to(DEV), [0, tokens])
        rows = (want > 2.0 ** 8) & torch.isfinite(want)                 # SiLU(v) = v / (1 + e^-v) = v exactly
    else:
        y = mes.mes_delta_linear(w_t, [blank], x.to(DEV), [0, tokens])
        rows = torch.ones(d_out, dtype=torch.bool)
    got, want = y.cpu()[:, rows], want.bfloat16()[rows].expand(tokens, -1)
    assert torch.equal(got.isnan(), want.isnan())
    assert torch.equal(got[~got.isnan()], want[~want.isnan()])
    assert gated or (got[0, :8].isinf().any() and got.isnan().any())
