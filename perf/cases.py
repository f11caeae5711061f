"""The calls whose speed and outputs are measured: what a user of this package has it do, through its public entry
points, from one decoded token on one linear layer to a mixed batch through a whole transformer block, and the offline
work on one expert's delta (salient selection, step-size learning, packing).

Matrix shapes are those of a Mistral-7B block (4096 wide, key / value 1024, MLP 14336), or generic odd ones.  Inputs
are synthetic: activations N(0, 1), base weights N(0, 0.02), deltas N(0, 0.003) with k input channels scaled by 15.

A case of kind
  linear  is one call of one layer, of up to three layers that read the same activations, or of a gated pair;
          `segs` are the tokens of each expert (rows of x are sorted by expert)
  block   is the seven linears of a block in four calls: [q, k, v], [o], [gate, up], [down]
  step    is loss and gradient of the step sizes of one matrix on calibration tokens
  pack    is the compression of one expert's delta of one matrix
  select  is the choice of the salient input channels of one matrix on calibration tokens
"""
import math

import torch

import paper_2406_09041_amd as mes

SYM, EQ1 = 0, 1
DEV = "cuda"

# 64 decoding sequences on 16 experts, Zipf(1.1)
DECODE_64 = "25,8,6,3,3,5,4,1,3,1,0,3,1,1,0,0"
# 256 decoding sequences, the same law
DECODE_256 = "93,40,25,16,8,10,8,13,7,7,3,7,0,4,8,7"
# ... together with four prompts of 1024 tokens
MIXED = "2141,1064,25,16,8,10,8,13,7,7,1027,7,0,4,8,7"

BLOCK = ((4096, "4096,1024,1024"), (4096, "4096"), (4096, "14336,14336"), (14336, "4096"))


def _linear(name, d_in, d_outs, segs, bits, k=64, grid=SYM, gated=False):
    c = {"kind": "linear", "d_in": d_in, "d_outs": d_outs, "segs": segs, "bits": bits, "k": k, "grid": grid, "gated": gated}
    return {"name": name, **c} if name else c


def listed():
    return [
        # one sequence being decoded on one expert: the smallest call, all latency
        _linear("one_token_q", 4096, "4096", "1", 2),
        # a decode batch through the projections that share their input
        _linear("decode_qkv_64", 4096, "4096,1024,1024", DECODE_64, 2),
        # ... through the gated MLP input, the largest weights of a block
        _linear("decode_gated_64", 4096, "14336,14336", DECODE_64, 2, gated=True),
        # ... through the MLP output, deltas kept at three bits
        _linear("decode_down_b3_64", 14336, "4096", DECODE_64, 3),
        # a layer whose sizes fit no tile, few experts, four bits on the grid of the paper's Eq. 1
        _linear("decode_ragged_b4", 5128, "3204", "11,0,1,17,5,0,3", 4, k=40, grid=EQ1),
        # a large decode batch
        _linear("decode_gate_up_256", 4096, "14336,14336", DECODE_256, 2),
        # three prompts of equal length on three experts
        _linear("prefill_gate_3x512", 4096, "14336", "512,512,512", 2, k=128),
        # prompts of odd lengths, deltas kept at three bits
        _linear("prefill_o_ragged_b3", 4096, "4096", "200,333,0,770", 3),
        # decoding sequences and prompts in one batch, all of a block
        {"name": "mixed_block", "kind": "block", "segs": MIXED, "bits": 2, "k": 64, "grid": SYM},
        # one step of learning the step sizes of the largest matrix
        {"name": "step_gate_512", "kind": "step", "d_in": 4096, "d_out": 14336, "tokens": 512, "bits": 2, "k": 8, "grid": SYM},
        # a fine-tuned expert's largest matrix being compressed
        {"name": "pack_gate", "kind": "pack", "d_in": 4096, "d_out": 14336, "bits": 2, "k": 64, "grid": SYM, "policy": mes.STEP_MAXABS},
        # its salient channels being chosen
        {"name": "select_q", "kind": "select", "d_in": 4096, "d_out": 4096, "tokens": 512, "bits": 2, "k": 64, "grid": SYM},
    ]


def _log_int(rng, lo, hi, multiple=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi, max(lo, int(round(v / multiple)) * multiple))


def _zipf(rng, tokens, experts):
    counts = [0] * experts
    for e in rng.choices(range(experts), [r ** -1.1 for r in range(1, experts + 1)], k=tokens):
        counts[e] += 1
    return ",".join(map(str, counts))


def draw(rng):
    bits = rng.choice([1, 2, 2, 3, 4])
    grid = rng.choice([SYM, EQ1]) if bits > 1 else SYM
    k = rng.choice([0, 8, 33, 64, 128])
    d_in, d_out = _log_int(rng, 256, 14336, 8), _log_int(rng, 256, 14336, 4)
    kind = rng.choice(["decode"] * 5 + ["prefill"] * 2 + ["step", "pack", "select"])
    if kind == "decode":
        segs = _zipf(rng, _log_int(rng, 1, 256), rng.randint(1, 24))
        form = rng.choice(["one", "multi", "gated"])
        if form == "one":
            return _linear("", d_in, str(d_out), segs, bits, k, grid)
        if form == "gated":
            return _linear("", d_in, "%d,%d" % (d_out, d_out), segs, bits, k, grid, gated=True)
        return _linear("", d_in, ",".join(str(_log_int(rng, 256, 14336, 4)) for _ in range(rng.randint(2, 3))), segs, bits, k, grid)
    if kind == "prefill":
        return _linear("", d_in, str(d_out), ",".join(str(_log_int(rng, 100, 1200)) for _ in range(rng.randint(1, 4))), bits, k, grid)
    if kind == "step":
        return {"kind": "step", "d_in": d_in, "d_out": d_out, "tokens": _log_int(rng, 64, 1024), "bits": bits, "k": k, "grid": grid}
    if kind == "pack":
        policy = rng.choice([mes.STEP_MAXABS, mes.STEP_MEANABS]) if bits == 1 else mes.STEP_MAXABS
        d_out = min(d_out, 4096 * 14336 // d_in // 4 * 4)
        return {"kind": "pack", "d_in": d_in, "d_out": d_out, "bits": bits, "k": k, "grid": grid, "policy": policy}
    d_out = min(d_out, 4096 * 4096 // d_in // 4 * 4)
    return {"kind": "select", "d_in": d_in, "d_out": d_out, "tokens": _log_int(rng, 64, 1024), "bits": bits, "k": k, "grid": grid}


# ---- inputs -----------------------------------------------------------------------------------------------------

def _normal(shape, std, seed, *which, dtype=torch.float32):
    g = torch.Generator(device=DEV)
    n = seed
    for w in which:
        n = (n * 1000003 + w + 1) % (1 << 62)
    g.manual_seed(n)
    return torch.empty(shape, device=DEV).normal_(0.0, std, generator=g).to(dtype)


def _salient(d_in, k, seed, *which):
    if not k:
        return torch.empty(0, dtype=torch.int32, device=DEV)
    return torch.sort(torch.topk(_normal((d_in,), 1.0, seed, 77, *which), k).indices).values.to(torch.int32)


def _delta(d_in, d_out, k, seed, *which):
    d, idx = _normal((d_out, d_in), 0.003, seed, 78, *which), _salient(d_in, k, seed, *which)
    if k:
        d[:, idx.long()] *= 15.0
    return d, idx


def _base(d_in, d_out, seed, *which):
    return _normal((d_out, d_in), 0.02, seed, 79, *which, dtype=torch.bfloat16)


def _segs(case):
    n = [int(v) for v in case["segs"].split(",")]
    off = [0]
    for v in n:
        off.append(off[-1] + v)
    return n, off


def _calls(case):
    """(d_in, [d_out ...], gated, number of its activations) of every call of a pass; calls of one width share x."""
    if case["kind"] == "linear":
        return [(case["d_in"], [int(v) for v in case["d_outs"].split(",")], case["gated"], 0)]
    return [(d_in, [int(v) for v in d.split(",")], False, d_in) for d_in, d in BLOCK]


def _given_step(case, d, idx):
    """Step sizes part of the way through their training: some weights already clamp."""
    m = d.clone()
    m[:, idx.long()] = 0
    return (0.6 * m.abs().amax(1) / max(0.5, 2 ** (case["bits"] - 1) - 0.5)).contiguous()


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("linear", "block"):
        counts, off = _segs(case)
        layers = []
        for ci, (d_in, d_outs, gated, xi) in enumerate(_calls(case)):
            parts = []
            for li, d_out in enumerate(d_outs):
                w = mes.mes_pack_base(_base(d_in, d_out, seed, ci, li))
                ex = []
                for e in range(len(counts)):
                    d, idx = _delta(d_in, d_out, case["k"], seed, ci, li, e)
                    ex.append(mes.mes_pack_delta(d, idx, case["bits"], case["grid"]))
                parts.append((w, ex))
            x = _normal((off[-1], d_in), 1.0, seed, 80, xi, dtype=torch.bfloat16)
            n_out = 1 if gated else len(d_outs)
            ys = [torch.empty((off[-1], d), dtype=torch.bfloat16, device=DEV) for d in d_outs[:n_out]]
            if gated:
                call = mes.DeltaLinearGated(*parts[0], *parts[1], max_tokens=off[-1])
            elif len(parts) == 1:
                call = mes.DeltaLinear(*parts[0], max_tokens=off[-1])
            else:
                call = mes.DeltaLinearMulti(parts, max_tokens=off[-1])
            layers.append((call, x, ys if len(d_outs) > 1 and not gated else ys[0]))
        return {"kind": kind, "layers": layers, "off": off}
    d, idx = _delta(case["d_in"], case["d_out"], case["k"], seed)
    if kind == "step":
        x = _normal((case["tokens"], case["d_in"]), 1.0, seed, 80, dtype=torch.bfloat16)
        return {"kind": kind, "fn": mes.StepGrad(d, idx, case["bits"], case["grid"], max_tokens=case["tokens"]),
                "step": _given_step(case, d, idx), "x": x}
    if kind == "pack":
        return {"kind": kind, "args": (d, idx, case["bits"], case["grid"], case["policy"])}
    x = _normal((case["tokens"], case["d_in"]), 1.0, seed, 80)
    return {"kind": kind, "args": (d, x, case["bits"], case["grid"], case["k"])}


def run(state):
    kind = state["kind"]
    if kind in ("linear", "block"):
        return [call(x, state["off"], y) for call, x, y in state["layers"]]
    if kind == "step":
        return state["fn"](state["step"], state["x"])
    if kind == "pack":
        p = mes.mes_pack_delta(*state["args"])
        return [t for t in (p.codes, p.step, p.salient) if t is not None]
    return mes.mes_select_salient(*state["args"], want_scores=True)


# ---- what a pass cannot do without ------------------------------------------------------------------------------

def work(case):
    kind, b, k = case["kind"], case["bits"], case["k"]
    if kind in ("linear", "block"):
        counts, off = _segs(case)
        active, T = sum(1 for n in counts if n), off[-1]
        nbytes = flops = 0
        for d_in, d_outs, gated, _ in _calls(case):
            nbytes += 2 * T * d_in
            for i, d_out in enumerate(d_outs):
                nbytes += 2 * d_out * d_in + active * (d_out * (d_in - k) * b // 8 + 2 * d_out * k + 4 * d_out + 4 * k)
                nbytes += 0 if gated and i else 2 * T * d_out
                flops += 2 * T * d_out * d_in
        return {"bytes": nbytes, "flops": flops}
    d_in, d_out = case["d_in"], case["d_out"]
    if kind == "step":   # two products: x E^T and x D^T
        return {"bytes": 4 * d_in * d_out + 2 * case["tokens"] * d_in + 12 * d_out + 4 * k, "flops": 4 * case["tokens"] * d_in * d_out}
    if kind == "pack":
        return {"bytes": 4 * d_in * d_out + d_out * (d_in - k) * b // 8 + 2 * d_out * k + 4 * d_out + 4 * k, "flops": 0}
    return {"bytes": 4 * d_in * d_out + 4 * case["tokens"] * d_in + 8 * d_in + 4 * k, "flops": 0}


def tolerance(case):
    """About four times what a pass differs from the same sums in 64 bits (2-norm, largest element)."""
    kind = case["kind"]
    if kind in ("linear", "block"):
        if max(_segs(case)[0]) < 192:
            return {"rel": 7e-3, "max": 0.016}   # exact products, results rounded to bf16: 1.7e-3, 3.9e-3
        return {"rel": 0.01, "max": 0.05}        # long segments round W + delta to bf16 as well: 2.4e-3, 1.3e-2
    if kind == "step":
        return {"rel": 2e-3, "max": 8e-3}        # operands rounded to bf16, squares summed over tokens: 3.7e-4, 6.5e-4
    if kind == "pack":
        return "exact"
    return {"rel": 1e-13, "max": 1e-12, "differ": 0.0}   # sums in 64 bits, 2e-15


# ---- the same in 64 bits, from the definitions ------------------------------------------------------------------

def _max_div(bits, grid):
    return 2 ** (bits - 1) - (0.5 if grid == SYM else 1.0)


def _init_step(w, bits, grid, policy):
    """w: the row with nothing but its quantised columns (a 2-d fp64 tensor)."""
    if policy == mes.STEP_MEANABS:
        return 2.0 * w.abs().mean(1)
    return w.abs().amax(1) / _max_div(bits, grid)


def _codes(w, step, bits, grid):
    """Unclamped and clamped signed codes of fp64 weights (SYM: cell index, EQ1: nearest level)."""
    s = step.double()[:, None]
    t = torch.where(s > 0, w / torch.where(s > 0, s, 1.0), 0.0)
    m = torch.floor(t) if grid == SYM else torch.round(t)
    return m, m.clamp(-2 ** (bits - 1), 2 ** (bits - 1) - 1)


def _shift(grid):
    return 0.5 if grid == SYM else 0.0


def _compress(d, idx, bits, grid, policy):
    """(step in 64 bits, step as stored, clamped codes, weights of the compressed delta)."""
    w, sal = d.double(), idx.long()
    keep = torch.ones(d.shape[1], dtype=torch.bool, device=d.device)
    keep[sal] = False
    exact = _init_step(w[:, keep], bits, grid, policy)
    step = exact.float()
    _, m = _codes(w, step, bits, grid)
    hat = (m + _shift(grid)) * step.double()[:, None]
    hat[:, sal] = d[:, sal].half().double()
    return exact, step, m, hat


def _pack_codes(m, idx, bits):
    """Signed codes [d_out, d_in] -> the stored bytes: blocks of 128 columns x 16 rows, 4-bit fields."""
    d_out, d_in = m.shape
    po, pi = -(-d_out // 64) * 64, -(-d_in // 128) * 128
    u = torch.zeros((po, pi), dtype=torch.int64, device=m.device)
    u[:d_out, :d_in] = (m + 2 ** (bits - 1)).long()
    u[:, idx.long()] = 0
    u = u.view(po // 16, 16, pi // 128, 4, 4, 8).permute(2, 0, 3, 1, 4, 5)   # [chunk][row tile][g][row][q][p]
    p4 = 4 * torch.arange(8, device=m.device)

    def plane1(bit):                       # one word a lane: code (q, p) at bit 4 p + q
        q = torch.arange(4, device=m.device)[:, None]
        return (((u >> bit) & 1) << (p4 + q)).sum((-2, -1))[..., None]

    def plane2(low):                       # two words a lane: code (q, p) in word q / 2 at bit 4 p + 2 (q % 2)
        v = ((u >> low) & 3).unflatten(-2, (2, 2))
        q = 2 * torch.arange(2, device=m.device)[:, None]
        return (v << (p4 + q)).sum((-2, -1))

    planes = {1: [plane1(0)], 2: [plane2(0)], 3: [plane2(0), plane1(2)], 4: [plane2(0), plane2(2)]}[bits]
    words = torch.cat([v.flatten(2) for v in planes], -1)
    words = torch.where(words >= 2 ** 31, words - 2 ** 32, words).to(torch.int32)
    return words.contiguous().view(torch.uint8).reshape(-1)


def _pack_salient(d, idx):
    d_out, k = d.shape[0], idx.numel()
    po, kp = -(-d_out // 64) * 64, -(-k // 32) * 32
    v = torch.zeros((po, kp), dtype=torch.float16, device=d.device)
    v[:d_out, :k] = d[:, idx.long()].half()
    return v.view(po // 16, 16, kp // 32, 4, 8).permute(0, 2, 3, 1, 4).contiguous().view(torch.uint8).reshape(-1)


def exact(case, seed):
    kind, bits, grid, k = case["kind"], case["bits"], case["grid"], case["k"]
    if kind in ("linear", "block"):
        counts, off = _segs(case)
        out = []
        for ci, (d_in, d_outs, gated, xi) in enumerate(_calls(case)):
            x = _normal((off[-1], d_in), 1.0, seed, 80, xi, dtype=torch.bfloat16).double()
            ys = []
            for li, d_out in enumerate(d_outs):
                w, y = _base(d_in, d_out, seed, ci, li).double(), torch.empty((off[-1], d_out), dtype=torch.float64, device=DEV)
                for e, n in enumerate(counts):
                    if n:
                        d, idx = _delta(d_in, d_out, k, seed, ci, li, e)
                        y[off[e]:off[e + 1]] = x[off[e]:off[e + 1]] @ (w + _compress(d, idx, bits, grid, mes.STEP_MAXABS)[3]).t()
                ys.append(y)
            if gated:
                out.append(torch.nn.functional.silu(ys[0]) * ys[1])
            else:
                out.append(ys if len(ys) > 1 else ys[0])
        return out
    d, idx = _delta(case["d_in"], case["d_out"], k, seed)
    if kind == "pack":
        step, _, m, _ = _compress(d, idx, bits, grid, case["policy"])
        return [_pack_codes(m, idx, bits), step] + ([_pack_salient(d, idx)] if k else [])
    w, sal = d.double(), idx.long()
    if kind == "select":
        x = _normal((case["tokens"], case["d_in"]), 1.0, seed, 80).double()
        step = _init_step(w, bits, grid, mes.STEP_MAXABS).float()
        hat = (_codes(w, step, bits, grid)[1] + _shift(grid)) * step.double()[:, None]
        score = (x * x).sum(0) * ((w - hat) ** 2).sum(0)
        order = torch.sort(score, descending=True, stable=True).indices[:k]
        return torch.sort(order).values.to(torch.int32), score
    x = _normal((case["tokens"], case["d_in"]), 1.0, seed, 80, dtype=torch.bfloat16).double()
    step = _given_step(case, d, idx)
    s = step.double()[:, None]
    m, mc = _codes(w, step, bits, grid)
    level = mc + _shift(grid)
    diff = level * s - w
    diff[:, sal] = d[:, sal].half().double() - w[:, sal]
    slope = level if bits == 1 else torch.where(m == mc, level - w / s, level)
    slope[:, sal] = 0.0
    r, p = x @ diff.t(), x @ slope.t()
    return 0.5 * (r * r).sum(0), (r * p).sum(0)
