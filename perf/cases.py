"""The work that this library's performance is judged on, as cases that a measuring program can prepare, run and check.

A case is one of four kinds of call sequence through the public entry points:

  layer   the seven projections of a decoder layer against one batch of m token rows, as a serving or prefill
          loop issues them: {q,k,v} and {gate,up} as grouped calls, o and down as single ones, all four marshalled
          once per weight copy (prepare_linear*) and re-issued
  linear  one projection through razer_linear with nothing prepared (output and workspace come with the call)
  codec   offline quantisation of one weight matrix and its decoding to bf16
  w4a4    a batch of bf16 activations encoded on the fly, then multiplied with an encoded weight

Weights are Student-t(4) with std 0.02 and 0.1 % of the input channels x20; activations N(0, 1), in the w4a4
kind with 0.5 % of the channels x50.  Everything is drawn on the GPU from the seed.
"""
import math

import torch

import paper_2501_04052_amd as razer

WEIGHT_SV = (5.0, 8.0)
ACT_SV = (5.0,)
FORMATS = {"byte": razer.WEIGHT, "f16": razer.WEIGHT_F16}


def listed():
    return [
        # latency of one small call at batch 1, host side included: the o projection of a 7B-class layer
        dict(name="linear_m1", kind="linear", n=4096, k=4096, m=1, format="byte", block=16),
        # one decode step of a 7B-class layer for one sequence
        dict(name="layer7b_m1", kind="layer", hidden=4096, kv=4096, inter=11008, m=1, format="byte", block=16),
        # the same for a few sequences, and for ordinary serving batches
        dict(name="layer7b_m4", kind="layer", hidden=4096, kv=4096, inter=11008, m=4, format="byte", block=16),
        dict(name="layer7b_m16", kind="layer", hidden=4096, kv=4096, inter=11008, m=16, format="byte", block=16),
        dict(name="layer7b_m64", kind="layer", hidden=4096, kv=4096, inter=11008, m=64, format="byte", block=16),
        # prefill of a short and of a long prompt
        dict(name="layer7b_m512", kind="layer", hidden=4096, kv=4096, inter=11008, m=512, format="byte", block=16),
        dict(name="layer7b_m2048", kind="layer", hidden=4096, kv=4096, inter=11008, m=2048, format="byte", block=16),
        # the format with 128-element blocks and FP16 scales, a small serving batch
        dict(name="layer7b_f16_m8", kind="layer", hidden=4096, kv=4096, inter=11008, m=8, format="f16", block=128),
        # a 70B-class layer (grouped-query attention), a small serving batch
        dict(name="layer70b_m8", kind="layer", hidden=8192, kv=1024, inter=28672, m=8, format="byte", block=16),
        # sizes that fit no tile, blocks of 32, an odd batch
        dict(name="ragged_m37", kind="linear", n=5003, k=3360, m=37, format="byte", block=32),
        # offline quantisation of a gate projection and a look at what it decodes to
        dict(name="codec_weight", kind="codec", n=11008, k=4096, format="byte", block=16),
        # weight-activation mode at prefill size
        dict(name="w4a4_m4096", kind="w4a4", n=11008, k=4096, m=4096, format="byte", block=16),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "linear", "linear", "codec", "w4a4"])
    block = rng.choice([16, 16, 16, 32, 64, 128])
    fmt = "byte"
    if kind != "w4a4" and rng.random() < 0.2:
        fmt, block = "f16", 128
    step = max(32, block)
    if kind == "layer":
        hidden = step * _log_int(rng, 1024 // step, 6144 // step)
        heads = rng.choice([1, 2, 4, 8])
        kv = max(step, hidden // heads // step * step)
        inter = step * int(hidden * rng.uniform(2.0, 3.6) / step)
        m = _log_int(rng, 1, 2048)
        case = dict(kind=kind, hidden=hidden, kv=kv, inter=inter, m=m, format=fmt, block=block)
    elif kind == "linear":
        case = dict(kind=kind, n=_log_int(rng, 512, 14336), k=step * _log_int(rng, 1024 // step, 12288 // step),
                    m=_log_int(rng, 1, 2048), format=fmt, block=block)
    elif kind == "codec":
        case = dict(kind=kind, n=_log_int(rng, 512, 14336), k=step * _log_int(rng, 1024 // step, 12288 // step),
                    format=fmt, block=block)
    else:
        case = dict(kind=kind, n=_log_int(rng, 512, 11008), k=step * _log_int(rng, 1024 // step, 8192 // step),
                    m=_log_int(rng, 1, 4096), format=fmt, block=block)
    # nothing drawn costs more than the largest listed cases (a 7B-class layer at 2048 rows; 480 MB of weights)
    while work(case)["flops"] > 8.2e11:
        case["m"] = max(1, case["m"] // 2 - 1)
    return case


# ------------------------------------------------------------------------------------------------ inputs
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + 17)
    return g


def _weight(n, k, gen):
    z = torch.randn((n, k), generator=gen, device="cuda")
    chi = torch.zeros((n, k), device="cuda")
    for _ in range(4):
        chi += torch.randn((n, k), generator=gen, device="cuda").square_()
    w = z.div_(chi.div_(4.0).sqrt_()).mul_(0.02 / 2.0 ** 0.5)
    outliers = max(1, round(0.001 * k))
    w[:, torch.randperm(k, generator=gen, device="cuda")[:outliers]] *= 20.0
    return w


def _activation(m, k, gen, outlier_frac=0.0):
    a = torch.randn((m, k), generator=gen, device="cuda")
    if outlier_frac:
        a[:, torch.randperm(k, generator=gen, device="cuda")[:max(1, round(outlier_frac * k))]] *= 50.0
    return a.to(torch.bfloat16)


def _layer_rows(case):
    h, kv, inter = case["hidden"], case["kv"], case["inter"]
    return [[(h, h), (kv, h), (kv, h)], [(h, h)], [(inter, h), (inter, h)], [(h, inter)]]


def _inputs(case, seed):
    """Unencoded operands in a fixed order, one at a time: ("w" | "a", tensor)."""
    gen = _generator(seed)
    if case["kind"] == "layer":
        for group in _layer_rows(case):
            for n, k in group:
                yield "w", _weight(n, k, gen)
            yield "a", _activation(case["m"], group[0][1], gen)
    else:
        yield "w", _weight(case["n"], case["k"], gen)
        if case["kind"] == "linear":
            yield "a", _activation(case["m"], case["k"], gen)
        elif case["kind"] == "w4a4":
            yield "a", _activation(case["m"], case["k"], gen, 0.005)


def prepare(case, seed):
    fmt, block = FORMATS[case["format"]], case["block"]
    if case["kind"] == "codec":
        (_, w), = _inputs(case, seed)
        return dict(kind="codec", w=w, fmt=fmt, block=block)
    encode = lambda w: razer.razer_quantize(w, fmt, WEIGHT_SV, block=block)  # noqa: E731
    if case["kind"] == "layer":
        calls, outs, ws = [], [], []
        for kind, t in _inputs(case, seed):
            if kind == "w":
                ws.append(encode(t))
                continue
            ys = [torch.empty((case["m"], w.rows), dtype=torch.bfloat16, device="cuda") for w in ws]
            calls.append(razer.prepare_linear_grouped(ws, t, ys) if len(ws) > 1 else razer.prepare_linear(ws[0], t, ys[0]))
            outs += ys
            ws = []
        return dict(kind="layer", calls=calls, outs=outs)
    (_, w), (_, a) = _inputs(case, seed)
    return dict(kind=case["kind"], w=encode(w), a=a)


def run(state):
    if state["kind"] == "layer":
        for call in state["calls"]:
            call()
        return state["outs"]
    if state["kind"] == "linear":
        return razer.razer_linear(state["w"], state["a"])
    if state["kind"] == "codec":
        t = razer.razer_quantize(state["w"], state["fmt"], WEIGHT_SV, block=state["block"])
        return dict(codes=t.codes, scales=t.scales, tensor_scale=t.tensor_scale,
                    decoded=razer.razer_dequant(t, torch.bfloat16))
    t = razer.razer_quantize(state["a"], razer.ACT, ACT_SV)
    return dict(codes=t.codes, scales=t.scales, tensor_scale=t.tensor_scale, y=razer.razer_linear(state["w"], t))


# ------------------------------------------------------------------------------------------------ what a pass needs
def _packed(n, k, case):
    return n * k / 2 + n * k / case["block"] * (2 if case["format"] == "f16" else 1) + 4


def work(case):
    """Each operand read once, each result written once; 2 m n k operations per product (none counted for the encoder)."""
    if case["kind"] == "layer":
        m, nbytes, flops = case["m"], 0.0, 0.0
        for group in _layer_rows(case):
            nbytes += 2.0 * m * group[0][1]
            for n, k in group:
                nbytes += _packed(n, k, case) + 2.0 * m * n
                flops += 2.0 * m * n * k
        return dict(bytes=nbytes, flops=flops)
    n, k = case["n"], case["k"]
    if case["kind"] == "codec":        # fp32 in, packed out, packed in, bf16 out
        return dict(bytes=4.0 * n * k + 2 * _packed(n, k, case) + 2.0 * n * k, flops=0.0)
    m = case["m"]
    nbytes = _packed(n, k, case) + 2.0 * m * k + 2.0 * m * n
    if case["kind"] == "w4a4":         # and the encoded activations, written and read
        nbytes += 2 * (m * k / 2 + m * k / 16 + 4)
    return dict(bytes=nbytes, flops=2.0 * m * n * k)


def tolerance(case):
    if case["kind"] == "codec":
        return "exact"                 # codes, scales and a decoder with one rounding: the format fixes every bit
    # bf16 results of fp32 sums: against 64 bits one sees the bf16 rounding, 1.7e-3 in the 2-norm and half a unit in the
    # last place (2^-8 of the value) at most; two summation orders differ in a few roundings, by one unit each
    return {"rel": 7e-3, "max": 1.6e-2, "differ": 0.0}


# ------------------------------------------------------------------------------------------------ 64-bit results
_FP4 = (0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0)
_FP4_MID = (0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0)


def _scale_grid(fmt):
    """Values of the block-scale codes in ascending order (the code is the index)."""
    if fmt == "f16":
        return torch.arange(0x4000, dtype=torch.int16).view(torch.float16).double()
    bias, top = (3, 64) if fmt == "byte" else (7, 127)
    c = torch.arange(top)
    e, mant = c >> 3, (c & 7).double()
    return torch.where(e > 0, 2.0 ** (e - bias).double() * (1 + mant / 8), 2.0 ** (1 - bias) * mant / 8)


def _f32(x):
    return x.float().double()


def _nearest_even(x, grid):
    """Index of the nearest grid value, ties to the even index, saturating."""
    hi = torch.searchsorted(grid, x).clamp_(1, grid.numel() - 1)
    lo = hi - 1
    down, up = x - grid[lo], grid[hi] - x
    take = (up < down) | ((up == down) & (hi % 2 == 0))
    return torch.where(take, hi, lo)


def _encode(x, fmt, block, specials):
    """Codes (packed), scale bytes / words, tensor scale and decoded values (64 bits, without the last rounding) of x
    as the format defines them: fp32 scale arithmetic, special value by the 64-bit error sum in index order."""
    grid = _scale_grid(fmt).to(x.device)
    fp4 = torch.tensor(_FP4, dtype=torch.float64, device=x.device)
    mid = torch.tensor(_FP4_MID, dtype=torch.float64, device=x.device)
    absmax = x.abs().max().double()
    delta = _f32(absmax / float(grid[-1] * 6)) if float(absmax) else torch.ones_like(absmax)
    n, k = x.shape
    codes, scales, values = [], [], []
    rows = max(1, (1 << 24) // k)
    for r in range(0, n, rows):
        b = x[r:r + rows].double().reshape(-1, k // block, block)
        sc = _nearest_even(_f32(b.abs().amax(-1) / _f32(delta * 6)), grid)
        s = grid[sc]
        live = (s > 0).unsqueeze(-1)
        xs = torch.where(live, _f32(b / _f32(delta * s).unsqueeze(-1).clamp_min(1e-300)), torch.zeros_like(b))
        mag = torch.searchsorted(mid, xs.abs())
        on_tie = (mag < 7) & (xs.abs() == mid[mag.clamp_max(6)]) & (mag % 2 == 1)
        mag = mag + on_tie
        base = (xs - torch.sign(xs) * fp4[mag])
        best = meta = None
        for i, v in enumerate(specials):
            e = torch.where((xs - v).abs() < base.abs(), xs - v, base).square()
            total = torch.zeros_like(e[..., 0])
            for j in range(block):
                total = total + e[..., j]
            better = torch.ones_like(total, dtype=torch.bool) if i == 0 else total < best
            best = total if i == 0 else torch.where(better, total, best)
            meta = torch.zeros_like(sc) if i == 0 else torch.where(better, torch.full_like(sc, i), meta)
        meta = torch.where(live[..., 0], meta, torch.zeros_like(meta))
        special = torch.tensor(specials, dtype=torch.float64, device=x.device)[meta].unsqueeze(-1)
        took = live & ((xs - special).abs() < base.abs())
        nib = torch.where(took, torch.full_like(mag, 8), mag + torch.where((xs < 0) & (mag > 0), 8, 0)).reshape(-1, k)
        values.append((s.unsqueeze(-1) * torch.where(took, special, torch.sign(xs) * fp4[mag])).reshape(-1, k))
        codes.append((nib[:, 0::2] | (nib[:, 1::2] << 4)).to(torch.uint8))
        word = sc | (meta << (14 if fmt == "f16" else 6 if fmt == "byte" else 7))
        scales.append(word.to(torch.int32).to(torch.int16) if fmt == "f16" else word.to(torch.uint8))
    return torch.cat(codes), torch.cat(scales), delta, torch.cat(values)


def _encode_weight(w, case):
    a, b = WEIGHT_SV
    return _encode(w, case["format"], case["block"], (a, b, -a, -b))


def exact(case, seed):
    if case["kind"] == "codec":
        (_, w), = _inputs(case, seed)
        codes, scales, delta, values = _encode_weight(w, case)
        return dict(codes=codes, scales=scales, tensor_scale=delta.reshape(1), decoded=values * delta)
    if case["kind"] == "w4a4":
        (_, w), (_, a) = _inputs(case, seed)
        _, _, dw, vw = _encode_weight(w, case)
        codes, scales, da, va = _encode(a.float(), "act", 16, (ACT_SV[0], -ACT_SV[0]))
        return dict(codes=codes, scales=scales, tensor_scale=da.reshape(1), y=(va @ vw.t()) * (da * dw))
    ys, ws = [], []
    for kind, t in _inputs(case, seed):
        if kind == "w":
            _, _, delta, values = _encode_weight(t, case)
            ws.append(values.mul_(delta))
            continue
        ys += [t.double() @ w.t() for w in ws]
        ws = []
    return ys if case["kind"] == "layer" else ys[0]
