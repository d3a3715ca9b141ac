"""The work that a user of this framework has it do, as cases that can be timed and checked.

One pass of a case is what a post-training quantization run executes over and over, through the
public calls of `paper_2302_01382_amd`:

  layer    one linear layer from its fp32 input: max calibration, error sweep, quantizer, quantized
           GEMM, squared distance to the reference output
  linear   the quantized GEMM alone, on operands that are already codes
  ffn      a BERT feed-forward block under one candidate bit configuration
  tensor   calibration, error sweep and quantizer of one tensor, scales per tensor / row / column
  sweep    the sensitivity sweep over a model's whole set of weight tensors
  noise    the noise perturbation of a weight tensor, one level or all seven
  adjust   one step of the scale adjustment: forward, gradients of the two scales, descent step
  hessian  the quadratic forms of the Hessian trace estimate
  search   one evaluation of a stack of layers, as the configuration searches ask for it

Inputs have the distributions of `workloads.py`: activations N(0, 1) or |N(0, 1)| after a ReLU,
weights N(0, sigma^2) with a few outliers.
"""
import math

import torch

from paper_2302_01382_amd import mpq
from paper_2302_01382_amd.stack import QuantStack

GRAN = {"tensor": mpq.PER_TENSOR, "row": mpq.PER_ROW, "col": mpq.PER_COL}
WIDTHS = (8, 4, 2)
LAMBDA = 0.28867513


def listed():
    return [
        # a small linear layer (configuration 1): every launch is latency
        {"name": "layer_small", "kind": "layer", "M": 64, "K": 256, "N": 256, "bits": 8, "w_bits": 8},
        # ResNet-50 stage 3, 3x3 convolution as a GEMM at batch 32 (configuration 2), int4 weights
        {"name": "layer_conv", "kind": "layer", "M": 6272, "K": 2304, "N": 256, "bits": 8, "w_bits": 4},
        # ResNet-50 stage 4, 3x3 convolution at inference batch 1: the latency table's long-K layer
        {"name": "linear_batch1", "kind": "linear", "M": 49, "K": 4608, "N": 512, "w_bits": 8},
        # BERT-large FFN2 at M = 16384 (configuration 5): the largest GEMM
        {"name": "linear_large", "kind": "linear", "M": 16384, "K": 4096, "N": 1024, "w_bits": 8},
        # a layer whose sizes fit no tile and no vector load
        {"name": "linear_ragged", "kind": "linear", "M": 2999, "K": 1155, "N": 1021, "w_bits": 8},
        # one candidate of configuration 5: the BERT-large FFN block, int4 weights in its second layer
        {"name": "ffn_candidate", "kind": "ffn", "M": 16384, "K": 1024, "H": 4096, "bits": 8, "w_bits": 8, "w2_bits": 4},
        # a tensor with odd sizes, scales per row: calibration, sensitivity, codes and dequantized values
        {"name": "tensor_ragged", "kind": "tensor", "rows": 3001, "cols": 1147, "gran": "row", "bits": 6},
        # the 96 weight tensors of BERT-large (configuration 4), both granularities
        {"name": "sweep_model", "kind": "sweep", "layers": 24, "width": 1024, "ffn": 4096},
        # the seven noise levels on one weight tensor, scales per output channel
        {"name": "noise_levels", "kind": "noise", "rows": 4096, "cols": 1024, "gran": "row", "b_lo": 2, "b_hi": 8},
        # the adjustment step on one layer's activations under an upstream gradient
        {"name": "adjust_step", "kind": "adjust", "rows": 12288, "cols": 768, "gran": "row", "bits": 4, "upstream": True},
        # 32 sign probes on the hidden activations of configuration 5
        {"name": "hessian_probe", "kind": "hessian", "M": 16384, "K": 4096, "probes": 32},
        # one evaluation of the search benchmark's stack, widths mixed
        {"name": "search_eval", "kind": "search", "layers": 24, "width": 1024, "M": 4096},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _odd_or_multiple(rng, v, of):
    """v itself (odd as often as not), or the multiple of `of` next to it."""
    return v if rng.random() < 0.4 else max(of, v // of * of)


def draw(rng):
    kind = rng.choice(["layer", "linear", "linear", "ffn", "tensor", "tensor", "sweep", "noise", "adjust", "hessian", "search"])
    bits, w_bits = rng.randint(2, 8), rng.choice([8, 4])
    if kind in ("layer", "linear"):
        while True:
            M, K, N = (_odd_or_multiple(rng, _log(rng, *r), 64) for r in ((1, 16384), (32, 4608), (16, 4096)))
            K += K & 1 if w_bits == 4 else 0  # packed pairs
            if M * N * K <= 2 ** (36 if K % 64 == 0 else 31):
                break
        c = {"kind": kind, "M": M, "K": K, "N": N, "w_bits": w_bits}
        return dict(c, bits=bits) if kind == "layer" else c
    if kind == "ffn":
        K = 64 * _log(rng, 1, 16)
        return {"kind": kind, "M": _log(rng, 16, 16384), "K": K, "H": 4 * K, "bits": rng.choice([4, 8]), "w_bits": w_bits,
                "w2_bits": rng.choice([8, 4])}
    if kind in ("tensor", "noise", "adjust"):
        rows, cols = _odd_or_multiple(rng, _log(rng, 16, 16384), 16), _odd_or_multiple(rng, _log(rng, 16, 4096), 16)
        if kind == "tensor":
            return {"kind": kind, "rows": rows, "cols": cols, "gran": rng.choice(["tensor", "row", "col"]), "bits": bits}
        if kind == "noise":
            rows = min(rows, 2 ** 22 // cols + 1)
            lo = rng.randint(2, 8)
            return {"kind": kind, "rows": rows, "cols": cols, "gran": rng.choice(["tensor", "row"]), "b_lo": lo,
                    "b_hi": rng.choice([lo, 8])}
        return {"kind": kind, "rows": rows, "cols": cols, "gran": rng.choice(["tensor", "row"]), "bits": bits,
                "upstream": rng.random() < 0.5}
    if kind == "sweep":
        width = 4 * _log(rng, 8, 256)
        return {"kind": kind, "layers": _log(rng, 1, 24), "width": width, "ffn": 4 * width}
    if kind == "hessian":
        return {"kind": kind, "M": _log(rng, 64, 16384), "K": 16 * _log(rng, 4, 256), "probes": _log(rng, 4, 64)}
    return {"kind": kind, "layers": _log(rng, 2, 24), "width": 32 * _log(rng, 2, 32), "M": _log(rng, 32, 4096)}


# ---- inputs -------------------------------------------------------------------------------------
def _gen(seed, *path):
    g = torch.Generator(device="cuda")
    for p in path:
        seed = (seed * 1000003 + 7919 * (p + 1)) & (2 ** 62 - 1)
    g.manual_seed(seed)
    return g


def _acts(g, rows, cols, relu=False):
    x = torch.randn((rows, cols), generator=g, device="cuda")
    return x.abs_() if relu else x


def _weight(g, rows, cols, sigma=None, share=0.0005, k=10.0):
    """N(0, sigma^2) with a share of the entries at +-k sigma."""
    sigma = sigma or math.sqrt(2.0 / cols)
    w = torch.randn((rows, cols), generator=g, device="cuda")
    u = torch.rand((rows, cols), generator=g, device="cuda")
    w = torch.where(u < share, torch.where(w < 0, -k, k), w)
    return w.mul_(sigma)


def _linear_inputs(c, seed):
    g = _gen(seed, 1)
    return _acts(g, c["M"], c["K"], relu=True), _weight(g, c["N"], c["K"])


def _ffn_inputs(c, seed):
    g = _gen(seed, 2)
    x, w1, w2 = _acts(g, c["M"], c["K"]), _weight(g, c["H"], c["K"]), _weight(g, c["K"], c["H"])
    ref = torch.randn((c["M"], c["K"]), generator=g, device="cuda")  # stands for the unquantized model's output
    return x, w1, w2, ref


def _tensor_input(c, seed):
    return _weight(_gen(seed, 3), c["rows"], c["cols"], 0.02)


def _sweep_inputs(c, seed):
    g = _gen(seed, 4)
    w, f = c["width"], c["ffn"]
    return [_weight(g, r, k, 0.02) for _ in range(c["layers"]) for r, k in ((3 * w, w), (w, w), (f, w), (w, f))]


def _adjust_inputs(c, seed):
    g = _gen(seed, 5)
    x = _acts(g, c["rows"], c["cols"])
    up = torch.randn((c["rows"], c["cols"]), generator=g, device="cuda") if c["upstream"] else None
    # scales that max calibration gives, moved by a few earlier steps so that some elements are clipped
    qmax = float(2 ** (c["bits"] - 1) - 1)
    m = x.abs().amax(dim=1) if c["gran"] == "row" else x.abs().amax().reshape(1)
    inv = qmax / m * (1.0 + 0.2 * torch.rand(m.shape, generator=g, device="cuda"))
    scale = m / qmax * (1.0 - 0.1 * torch.rand(m.shape, generator=g, device="cuda"))
    return x, up, inv, scale


def _search_inputs(c, seed):
    g = _gen(seed, 6)
    x = _acts(g, c["M"], c["width"])
    # layers of different sensitivity: the larger the outliers, the coarser the grid for the rest
    k = (3.0 + 9.0 * torch.rand(c["layers"], generator=g, device="cuda")).tolist()
    return x, [_weight(g, c["width"], c["width"], None, 0.002, k[l]) for l in range(c["layers"])]


def _search_bits(c):
    return [WIDTHS[(5 * l // 3) % 3] for l in range(c["layers"])]


# ---- the framework's side -----------------------------------------------------------------------
def _weight_codes(w, bits):
    """A layer's weights as a program keeps them: codes (packed up to 4 bits), step sizes, storage."""
    m = mpq.calibrate_absmax(w, mpq.PER_ROW)
    _, codes, packed = mpq.fake_quant(w, m, bits, mpq.PER_ROW, want_y=False, want_codes=bits > 4, want_packed4=bits <= 4)
    return (packed if bits <= 4 else codes), mpq.scale_from_absmax(m, bits), 4 if bits <= 4 else 8


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = {"case": c, "ws": mpq.Workspace()}
    if kind in ("layer", "linear"):
        x, w = _linear_inputs(c, seed)
        s["wq"], s["sw"], s["store"] = _weight_codes(w, c["w_bits"])
        if kind == "layer":
            s["x"] = x
            s["ref"] = x @ w.t()
        else:
            m = mpq.calibrate_absmax(x)
            s["aq"] = mpq.fake_quant(x, m, 8, want_y=False, want_codes=True)[1]
            s["sa"] = mpq.scale_from_absmax(m, 8)
    elif kind == "ffn":
        s["x"], w1, w2, s["ref"] = _ffn_inputs(c, seed)
        s["w1"], s["w2"] = _weight_codes(w1, c["w_bits"]), _weight_codes(w2, c["w2_bits"])
        s["mx"] = mpq.calibrate_absmax(s["x"])
    elif kind in ("tensor", "noise"):
        s["x"] = _tensor_input(c, seed)
        if kind == "noise":
            s["m"] = mpq.calibrate_absmax(s["x"], GRAN[c["gran"]])
            s["seed"] = seed
    elif kind == "sweep":
        s["plan"] = mpq.sweep_plan_build(_sweep_inputs(c, seed))
    elif kind == "adjust":
        s["x"], s["g"], s["inv"], s["scale"] = _adjust_inputs(c, seed)
    elif kind == "hessian":
        s["x"] = _acts(_gen(seed, 7), c["M"], c["K"])
        s["seed"] = seed
    else:
        x, weights = _search_inputs(c, seed)
        s["stack"] = QuantStack(x, weights, WIDTHS)
        s["bits"] = _search_bits(c)
    return s


def run(state):
    s, c, ws = state, state["case"], state["ws"]
    kind = c["kind"]
    if kind == "layer":
        m = mpq.calibrate_absmax(s["x"], ws=ws)
        sse = mpq.quant_error(s["x"], m, 2, 8, ws=ws)
        _, codes, _ = mpq.fake_quant(s["x"], m, c["bits"], want_y=False, want_codes=True)
        y, _ = mpq.qgemm(codes, s["wq"], mpq.scale_from_absmax(m, c["bits"]), s["sw"], s["store"], mpq.PER_ROW, ws=ws)
        return {"absmax": m, "sse": sse, "codes": codes, "y": y, "score": mpq.sse_pair(y, s["ref"], ws=ws)}
    if kind == "linear":
        return mpq.qgemm(s["aq"], s["wq"], s["sa"], s["sw"], s["store"], mpq.PER_ROW, ws=ws)[0]
    if kind == "ffn":
        _, a1, _, s1 = mpq.fake_quant_step(s["x"], s["mx"], c["bits"], want_y=False, want_codes=True)
        h, mh = mpq.qgemm_act(a1, s["w1"][0], s1, s["w1"][1], mpq.ACT_GELU, s["w1"][2], mpq.PER_ROW)
        _, a2, _, s2 = mpq.fake_quant_step(h, mh, c["bits"], want_y=False, want_codes=True)
        score, _ = mpq.qgemm_score(a2, s["w2"][0], s2, s["w2"][1], s["ref"], s["w2"][2], mpq.PER_ROW, ws=ws)
        return {"hidden": h, "absmax": mh, "score": score}
    if kind == "tensor":
        gran = GRAN[c["gran"]]
        m = mpq.calibrate_absmax(s["x"], gran, ws=ws)
        sse = mpq.quant_error(s["x"], m, 2, 8, gran, ws=ws)
        packed = c["bits"] <= 4 and c["cols"] % 2 == 0
        y, codes, p4 = mpq.fake_quant(s["x"], m, c["bits"], gran, want_codes=not packed, want_packed4=packed)
        return {"absmax": m, "sse": sse, "y": y, "codes": p4 if packed else codes}
    if kind == "noise":
        gran = GRAN[c["gran"]]
        if c["b_lo"] == c["b_hi"]:
            return mpq.noise_inject(s["x"], s["m"], c["b_lo"], LAMBDA, s["seed"], 3, gran)
        return mpq.noise_inject_sweep(s["x"], s["m"], c["b_lo"], c["b_hi"], LAMBDA, s["seed"], 3, gran)
    if kind == "sweep":
        p = s["plan"]
        mpq.calibrate_absmax_batch(p)
        mpq.quant_error_batch(p, mpq.PER_TENSOR)
        mpq.quant_error_batch(p, mpq.PER_ROW)
        return {"absmax_row": p.absmax_row_all, "absmax": p.absmax_tensor_all, "sse": p.sse_tensor_all, "sse_row": p.sse_row_all}
    if kind == "adjust":
        gran = GRAN[c["gran"]]
        inv, scale = s["inv"].clone(), s["scale"].clone()
        y, _ = mpq.fake_quant_scales(s["x"], inv, scale, c["bits"], gran)
        dinv, dscale, loss = mpq.scale_grad(s["x"], inv, scale, c["bits"], s["g"], gran, ws=ws)
        mpq.scale_sgd_step(inv, scale, dinv, dscale, 1e-5)
        return {"y": y, "dinv": dinv, "dscale": dscale, "loss": loss, "inv": inv, "scale": scale}
    if kind == "hessian":
        return mpq.hutchinson_quad_signs(s["x"], s["seed"], 0, c["probes"], ws=ws)
    return {"accuracy": s["stack"].evaluate(s["bits"]), "absmax": s["stack"].a_absmax_all}


# ---- what a pass cannot do without --------------------------------------------------------------
def _gemm_bytes(M, N, K, w_bits):
    return M * K + N * K * w_bits // 8 + 4 * N


def work(case):
    c, kind = case, case["kind"]
    if kind in ("layer", "linear"):
        M, N, K = c["M"], c["N"], c["K"]
        flops = 2 * M * N * K
        if kind == "linear":
            return {"bytes": _gemm_bytes(M, N, K, c["w_bits"]) + 4 * M * N, "flops": flops}
        # the fp32 input is read once, its codes are an output, the reference is read, the result written
        return {"bytes": 4 * M * K + _gemm_bytes(M, N, K, c["w_bits"]) + 8 * M * N, "flops": flops + 28 * M * K}
    if kind == "ffn":
        M, K, H = c["M"], c["K"], c["H"]
        return {"bytes": 4 * M * K + 4 * M * H + 4 * M * K + H * K * (c["w_bits"] + c["w2_bits"]) // 8, "flops": 4 * M * K * H}
    if kind == "tensor":
        n = c["rows"] * c["cols"]
        nch = {"tensor": 1, "row": c["rows"], "col": c["cols"]}[c["gran"]]
        out = 0.5 if c["bits"] <= 4 and c["cols"] % 2 == 0 else 1
        return {"bytes": (8 + out) * n + (4 + 56) * nch, "flops": 34 * n}
    if kind == "noise":
        n = c["rows"] * c["cols"]
        return {"bytes": 4 * n * (1 + c["b_hi"] - c["b_lo"] + 1), "flops": 70 * n}
    if kind == "sweep":
        w, f = c["width"], c["ffn"]
        n, rows = c["layers"] * (4 * w * w + 2 * w * f), c["layers"] * (5 * w + f)
        return {"bytes": 4 * n + 60 * rows, "flops": 57 * n}
    if kind == "adjust":
        n = c["rows"] * c["cols"]
        return {"bytes": (12 if c["upstream"] else 8) * n, "flops": 17 * n}
    if kind == "hessian":
        return {"bytes": 4 * c["M"] * c["K"], "flops": 2 * c["M"] * c["K"] * c["probes"]}
    M, D, L = c["M"], c["width"], c["layers"]
    weights = sum(D * D * (8 if b > 4 else 4) // 8 for b in _search_bits(c))
    return {"bytes": M * D + weights + 4 * M * D, "flops": 2 * M * D * D * L}


def tolerance(case):
    # Codes, maxima, noise and dequantized values have fixed 32-bit recipes; the error sums are
    # 32-bit sums in an order of the implementation's choosing.
    return {
        "layer": {"rel": 1e-5},
        "linear": {"rel": 1e-6},
        "ffn": {"rel": 1e-5},       # GELU from a fitted form in 32 bits
        "tensor": {"rel": 1e-5},
        "sweep": {"rel": 1e-5},
        "noise": {"rel": 1e-6},
        "adjust": {"rel": 2e-5, "max": 1e-3},  # sums of either sign: the scale gradients cancel
        "hessian": {"rel": 1e-5},
        "search": {"rel": 1e-5},
    }[case["kind"]]


# ---- the same in 64 bits, without this repository's code -------------------------------------------
def _along(m, gran):
    return m[:, None] if gran == "row" else m[None, :] if gran == "col" else m


def _absmax(x, gran):
    a = x.abs()
    return a.amax(dim=1) if gran == "row" else a.amax(dim=0) if gran == "col" else a.amax().reshape(1)


def _codes64(x, m, bits, gran):
    """Codes from the 32-bit factor qmax / m and the exact product with it, and the 32-bit step size."""
    qmax = float(2 ** (bits - 1) - 1)
    q = torch.full_like(m, qmax)  # a tensor: torch divides by (and into) a number through a rounded reciprocal
    inv = torch.where(m > 0, q / m, torch.zeros_like(m))
    code = torch.round(x.double() * _along(inv, gran).double()).clamp_(-qmax, qmax)
    return code, m / q


def _chunks(n, size):
    return [slice(i, min(n, i + size)) for i in range(0, n, size)]


def _sse64(x, m, gran):
    total = 0.0 if gran != "row" else []
    for r in _chunks(x.shape[0], max(1, 2 ** 24 // x.shape[1])):
        mr, v = (m[r] if gran == "row" else m), x[r]
        per_b = []
        for b in range(2, 9):
            code, step = _codes64(v, mr, b, gran)
            e = (code * _along(step, gran).double() - v.double()).square_()
            per_b.append(e.sum(dim=1) if gran == "row" else e.sum(dim=0) if gran == "col" else e.sum().reshape(1))
        part = torch.stack(per_b, dim=1)
        if gran == "row":
            total.append(part)
        else:
            total = total + part
    return torch.cat(total) if gran == "row" else total


def _weight_codes64(w, bits):
    return _codes64(w, _absmax(w, "row"), bits, "row")


def _product64(codes, step, wc, sw):
    return (codes @ wc.t()) * step.double() * sw.double()[None, :]


def _philox(counter_lo, stream, key_hi_tag, seed):
    """Philox-4x32-10 in 64-bit integers; counter (counter_lo < 2^32, 0, stream, 0)."""
    mask = 0xFFFFFFFF
    c0, zero = counter_lo, torch.zeros_like(counter_lo)
    c1, c2, c3 = zero, zero + stream, zero
    k0, k1 = seed & mask, ((seed >> 32) & mask) ^ key_hi_tag
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = ((p1 >> 32) & mask) ^ c1 ^ k0, p1 & mask, ((p0 >> 32) & mask) ^ c3 ^ k1, p0 & mask
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return c0, c1, c2, c3


def _normals64(n, seed, stream):
    w = _philox(torch.arange((n + 3) // 4, device="cuda", dtype=torch.int64), stream, 0, seed)
    z = []
    for a, b in ((w[0], w[1]), (w[2], w[3])):
        r = torch.sqrt(-2.0 * torch.log(((a >> 8) + 1).double() * 2.0 ** -24))
        t = (b >> 8).double() * (2.0 * math.pi * 2.0 ** -24)
        z += [r * torch.cos(t), r * torch.sin(t)]
    return torch.stack(z, dim=1).reshape(-1)[:n]


def _signs64(rows, cols, seed):
    n = rows * cols
    w = torch.stack(_philox(torch.arange((n + 127) // 128, device="cuda", dtype=torch.int64), 0, 0x5241444D, seed), dim=1)
    bit = (w.reshape(-1, 1) >> torch.arange(32, device="cuda")) & 1
    return (1.0 - 2.0 * bit.reshape(-1)[:n].double()).reshape(rows, cols)


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("layer", "linear"):
        x, w = _linear_inputs(c, seed)
        wc, sw = _weight_codes64(w, c["w_bits"])
        m = _absmax(x, "tensor")
        code, step = _codes64(x, m, c.get("bits", 8), "tensor")
        y = _product64(code, step, wc, sw)
        if kind == "linear":
            return y
        return {"absmax": m.double(), "sse": _sse64(x, m, "tensor"), "codes": None, "y": y,
                "score": (y - (x @ w.t()).double()).square().sum().reshape(1)}
    if kind == "ffn":
        x, w1, w2, ref = _ffn_inputs(c, seed)
        code, step = _codes64(x, _absmax(x, "tensor"), c["bits"], "tensor")
        wc, sw = _weight_codes64(w1, c["w_bits"])
        h = _product64(code, step, wc, sw)
        h = 0.5 * h * torch.erfc(h * -math.sqrt(0.5))
        code, step = _codes64(h.float(), _absmax(h.float(), "tensor"), c["bits"], "tensor")
        wc, sw = _weight_codes64(w2, c["w2_bits"])
        y = _product64(code, step, wc, sw)
        return {"hidden": h, "absmax": _absmax(h, "tensor"), "score": (y - ref.double()).square_().sum().reshape(1)}
    if kind == "tensor":
        x = _tensor_input(c, seed)
        m = _absmax(x, c["gran"])
        code, step = _codes64(x, m, c["bits"], c["gran"])
        return {"absmax": m.double(), "sse": _sse64(x, m, c["gran"]), "y": code * _along(step, c["gran"]).double(), "codes": None}
    if kind == "noise":
        x = _tensor_input(c, seed)
        m = _absmax(x, c["gran"])
        z = _normals64(x.numel(), seed, 3).reshape(x.shape)
        planes = []
        for b in range(c["b_lo"], c["b_hi"] + 1):
            sigma = torch.tensor(LAMBDA, dtype=torch.float32, device="cuda") * (m / torch.full_like(m, 2 ** (b - 1) - 1))
            planes.append(x.double() + _along(sigma, c["gran"]).double() * z)
        return planes[0] if c["b_lo"] == c["b_hi"] else torch.stack(planes)
    if kind == "sweep":
        ts = _sweep_inputs(c, seed)
        rows, whole = [_absmax(t, "row") for t in ts], [_absmax(t, "tensor") for t in ts]
        return {"absmax_row": torch.cat(rows).double(), "absmax": torch.cat(whole).double(),
                "sse": torch.cat([_sse64(t, m, "tensor") for t, m in zip(ts, whole)]),
                "sse_row": torch.cat([_sse64(t, m, "row") for t, m in zip(ts, rows)])}
    if kind == "adjust":
        x, up, inv, scale = _adjust_inputs(c, seed)
        qmax = float(2 ** (c["bits"] - 1) - 1)
        x, i64, s64 = x.double(), _along(inv, c["gran"]).double(), _along(scale, c["gran"]).double()
        r = torch.round(x * i64)
        q = r.clamp(-qmax, qmax)
        e = q * s64 - x
        g = up.double() if up is not None else 2.0 * e

        def total(v):
            return v.sum(dim=1) if c["gran"] == "row" else v.sum().reshape(1)

        dscale, dinv = total(g * q), scale.double() * total(torch.where(r == q, g * x, torch.zeros_like(x)))
        return {"y": q * s64, "dinv": dinv, "dscale": dscale, "loss": total(e * e),
                "inv": inv.double() - 1e-5 * dinv, "scale": scale.double() - 1e-5 * dscale}
    if kind == "hessian":
        x = _acts(_gen(seed, 7), c["M"], c["K"])
        return (x.double() @ _signs64(c["probes"], c["K"], seed).t()).square_().sum(dim=0)
    x, weights = _search_inputs(c, seed)
    h, ref, maxima, last = x, x, [], len(weights) - 1
    for l, (w, b) in enumerate(zip(weights, _search_bits(c))):
        m = _absmax(h, "tensor")
        maxima.append(m)
        code, step = _codes64(h, m, 8, "tensor")
        wc, sw = _weight_codes64(w, b)
        ref = ref @ w.t()
        if l < last:
            # a layer's output is a 32-bit tensor, two products rounded once each: with unrounded ones
            # codes would flip, and the layers behind would follow another trajectory
            h, ref = torch.relu((code @ wc.t()).float() * step * sw[None, :]), torch.relu(ref)
        else:
            h = _product64(code, step, wc, sw)
    ref = ref.double()
    return {"accuracy": 1.0 - float((h - ref).square().sum()) / float(ref.square().sum()), "absmax": torch.cat(maxima).double()}
