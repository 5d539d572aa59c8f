"""The performance cases of the Sigma-Delta linear layer: what a program does with the library.

Decode (1-16 activation rows: token generation, alone or in small batches), batched and prefill
linears (17 rows and more), the weight encoder, and the calibration behind the compensated encoder
(Hessian, its factor, the block-compensated encoding).  Shapes are those of OPT-125m, LLaMA-7B and
LLaMA-70B layers; code storage, level counts, OSRs and activation types are the ones a model is
encoded and run with.

The linear cases need codes before the call.  They are made here from seeded weights by a plain
torch form of Algorithm 1 (block Hadamard, band-limited upsampling, row scale, first-order
Sigma-Delta scan) and packed in the documented storage format, so that the 64-bit results of
``exact`` rest on no code of the library.
"""
import math

import torch

import paper_2510_03275_amd as sdq

DEV = "cuda"
_TYPES = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}

# LLaMA-7B decoder layer: the four groups of linears that share an input, as (k, rows of each
# linear, OSR).  The OSRs are what MultiOSR gives such a layer at a mean of 2.5 (grid 1/8).
_LAYER_7B = [(4096, [4096, 4096, 4096], 2.25), (4096, [4096], 2.125),
             (4096, [11008, 11008], 2.75), (11008, [4096], 2.5)]


def _linear(kind, groups, m, levels, dtype, base3=False, **more):
    return {"kind": kind, "groups": groups, "m": m, "levels": levels, "dtype": dtype, "base3": base3,
            **more}


def _groups(text):
    """'k:n,n:osr;...' -> [(k, [n, ...], osr), ...] (cases hold plain values only)."""
    out = []
    for g in text.split(";"):
        k, ns, osr = g.split(":")
        out.append((int(k), [int(n) for n in ns.split(",")], float(osr)))
    return out


def _text(groups):
    return ";".join("%d:%s:%g" % (k, ",".join(map(str, ns)), osr) for k, ns, osr in groups)


def listed():
    return [
        # One token through the smallest projection (OPT-125m q_proj): two short launches.
        _linear("linear", "768:768:2", 1, 3, "f16", name="decode_opt125m_q_m1"),
        # One token through a binary LLaMA-7B down_proj (fractional OSR 1.5).
        _linear("linear", "11008:4096:1.5", 1, 2, "f16", name="decode_7b_down_binary_m1"),
        # A whole LLaMA-7B decoder layer's seven linears for a batch of 16 sequences.
        _linear("linear", _text(_LAYER_7B), 16, 3, "f16", name="decode_7b_layer_m16"),
        # One token through LLaMA-70B gate/up (one input, two linears: one group call).
        _linear("linear", "8192:28672,28672:2.5", 1, 3, "bf16", name="decode_70b_gateup_m1"),
        # A batch of eight through LLaMA-70B down_proj.
        _linear("linear", "28672:8192:2.5", 8, 3, "f16", name="decode_70b_down_m8"),
        # The smallest storage (1.6 bits per ternary code) at a batch of three.
        _linear("linear", "8192:8192:2", 3, 3, "f16", True, name="decode_70b_o_base3_m3"),
        # A batch of 64 sequences (or a short prompt) through LLaMA-7B gate/up.
        _linear("linear", "4096:11008,11008:2.5", 64, 3, "f16", name="batch_7b_gateup_m64"),
        # A prompt of ragged length through a binary down_proj.
        _linear("linear", "11008:4096:1.5", 333, 2, "f16", name="prefill_7b_down_binary_m333"),
        # A long prompt through LLaMA-70B up_proj: the largest contraction.
        _linear("linear", "8192:28672:2", 2048, 3, "bf16", name="prefill_70b_up_m2048"),
        # Encoding a LLaMA-7B down_proj (the step that a user runs over every weight of a model).
        {"kind": "encode", "n": 4096, "k": 11008, "osr": 1.5, "levels": 2, "block": 256, "base3": False,
         "name": "encode_7b_down_binary"},
        # Calibration of one input: H += 2 X^T X over 2048 token rows, and the factor of its inverse.
        {"kind": "calibrate", "k": 4096, "rows": 2048, "name": "calibrate_7b_k4096"},
        # The compensated encoding of a LLaMA-7B q_proj against such a factor.
        {"kind": "compensate", "n": 4096, "k": 4096, "osr": 2.0, "levels": 3, "block": 256,
         "name": "compensate_7b_q"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: sizes over their logarithm, odd row counts among them."""
    kind = rng.choice(["decode", "decode", "decode", "prefill", "prefill", "encode", "calibrate", "compensate"])
    osr = rng.randint(8, 24) / 8.0                       # 1 .. 3 on the grid of 1/8
    levels = rng.choice([2, 3, 3])
    if kind in ("decode", "prefill"):
        m = rng.randint(1, 16) if kind == "decode" else _log(rng, 17, 2048)
        k = 256 * _log(rng, 3, 112 if kind == "decode" else 43)
        ns = [_log(rng, 500, 29000 if kind == "decode" else 12000) for _ in range(rng.choice([1, 1, 2, 3]))]
        return _linear("linear", _text([(k, ns, osr)]), m, levels, rng.choice(["f16", "bf16", "bf16", "f32"]),
                       levels == 3 and rng.random() < 0.2)
    if kind == "encode":
        block = rng.choice([64, 128, 256, 256])
        if block == 64:
            osr = max(1.0, round(osr * 2) / 2)           # M a multiple of 32
        elif block == 128:
            osr = max(1.0, round(osr * 4) / 4)
        return {"kind": "encode", "n": _log(rng, 500, 12000), "k": 256 * _log(rng, 3, 43), "osr": osr,
                "levels": levels, "block": block, "base3": levels == 3 and rng.random() < 0.25}
    if kind == "calibrate":
        return {"kind": "calibrate", "k": 64 * _log(rng, 12, 64), "rows": _log(rng, 100, 4096)}
    return {"kind": "compensate", "n": _log(rng, 500, 5000), "k": 256 * _log(rng, 3, 16), "osr": osr,
            "levels": levels, "block": 256}


# ---------------------------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------------------------

def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((seed * 1000003 + stream * 7919 + 17) % (1 << 62))
    return g


def _weights(g, n, k, sigma=0.015):
    """Gaussian weights with 0.1 % of the entries ten times as large."""
    w = torch.randn(n, k, generator=g, device=DEV).mul_(sigma)
    return torch.where(torch.rand(n, k, generator=g, device=DEV) < 0.001, w * 10, w)


def _sylvester(b):
    h = torch.ones(1, 1, dtype=torch.float64, device=DEV)
    while h.shape[0] < b:
        h = torch.cat([torch.cat([h, h], 1), torch.cat([h, -h], 1)], 0)
    return h / math.sqrt(b)


def _upsample(b, m):
    """U [B x M]: sample j of the upsampled block is sum_t v[t] U[t, j]."""
    p = (torch.arange(m, device=DEV)[None, :] * b - torch.arange(b, device=DEV)[:, None] * m) % (b * m)
    tau = p.double() / m
    u = torch.sin(math.pi * tau) / (b * torch.tan(math.pi * tau / b))
    return torch.where(p == 0, 1.0, torch.where(p % m == 0, 0.0, u))


def _decimate(b, m):
    """D^T [B x M]: a block is back at B samples as out[t] = sum_j c[j] D^T[t, j]."""
    if b == m:
        return torch.eye(b, dtype=torch.float64, device=DEV)
    num = torch.arange(m, device=DEV)[None, :] * b - torch.arange(b, device=DEV)[:, None] * m
    whole = num // m
    tau = num.double() / m
    d = torch.sin(math.pi * tau) / torch.tan(math.pi * tau / b) + torch.cos(math.pi * tau)
    at = (whole % b == 0).double() * b + 1.0 - 2.0 * (whole % 2).double()
    return torch.where(num % m == 0, at, d) / m


def _codes(w, osr, levels, b=256):
    """Codes (int8 [n, k_up]) and row scales (fp32 [n]) of weights w."""
    n, k = w.shape
    nb, m = k // b, int(round(osr * b))
    v = (w.view(n * nb, b) @ _sylvester(b).float()).t()
    x = _upsample(b, m).float().t().contiguous() @ v                      # [M, n * nb]
    s = x.abs().amax(0).view(n, nb).amax(1)
    step = s[:, None].expand(n, nb).reshape(-1)
    theta = step * 0.5
    out = torch.empty(m, n * nb, dtype=torch.int8, device=DEV)
    u = torch.zeros(n * nb, device=DEV)
    for j in range(m):
        u += x[j]
        if levels == 3:
            c = (u > theta).to(torch.int8) - (u < -theta).to(torch.int8)
        else:
            c = (u >= 0).to(torch.int8) * 2 - 1
        out[j] = c
        u -= c * step
    return out.view(m, n, nb).permute(1, 2, 0).reshape(n, nb * m), s


def _pack(c, levels, base3):
    """Codes in the storage format: 16-byte chunks, the 64 rows of a panel side by side."""
    n, k_up = c.shape
    per = 80 if base3 else (64 if levels == 3 else 128)
    chunks, n_pad = -(-k_up // per), -(-n // 64) * 64
    if base3:
        d = torch.zeros(n, chunks * per, dtype=torch.int8, device=DEV)
        d[:, :k_up] = c
        d = d.view(n, chunks * 16, 5)
        v = torch.zeros(n, chunks * 16, dtype=torch.int16, device=DEV)
        for i in range(5):
            v = v * 3 + (d[..., i] + 1)
        q = ((v.int() * 256 + 242) // 243).to(torch.uint8)
    else:
        f = (c & 3) if levels == 3 else (c > 0).to(torch.int8)
        bits = 2 if levels == 3 else 1
        p = torch.zeros(n, chunks * per, dtype=torch.uint8, device=DEV)
        p[:, :k_up] = f.to(torch.uint8)
        p = p.view(n, chunks * 16, 8 // bits)
        q = torch.zeros(n, chunks * 16, dtype=torch.uint8, device=DEV)
        for i in range(8 // bits):
            q |= p[..., i] << (bits * i)
    rows = torch.zeros(n_pad, chunks * 16, dtype=torch.uint8, device=DEV)
    rows[:n] = q
    return rows.view(n_pad // 64, 64, chunks, 16).permute(0, 2, 1, 3).contiguous().view(-1)


def _linear_inputs(case, seed):
    """Per group: x, and (codes, scales) of each of its linears."""
    out = []
    for gi, (k, ns, osr) in enumerate(_groups(case["groups"])):
        x = torch.randn(case["m"], k, generator=_gen(seed, 100 * gi), device=DEV).to(_TYPES[case["dtype"]])
        coded = [_codes(_weights(_gen(seed, 100 * gi + 1 + j), n, k), osr, case["levels"])
                 for j, n in enumerate(ns)]
        out.append((k, ns, osr, x, coded))
    return out


def _calibration_rows(seed, rows, k):
    """Token rows: a low-rank part plus noise, as the inputs of a layer are correlated."""
    g = _gen(seed, 5)
    r = max(8, k // 16)
    low = torch.randn(rows, r, generator=g, device=DEV) @ torch.randn(r, k, generator=g, device=DEV)
    return (low / math.sqrt(r) + 0.3 * torch.randn(rows, k, generator=g, device=DEV)).contiguous()


def _damping(x, k):
    return 0.01 * float((x.double() ** 2).sum()) * 2 / k      # 1 % of the mean diagonal


def _factor(h, lam):
    """U upper with U^T U = (H + lam I)^-1: with the index order reversed, the inverse of a
    Cholesky factor."""
    k = h.shape[0]
    low = torch.linalg.cholesky((h + lam * torch.eye(k, dtype=h.dtype, device=DEV)).flip(0, 1))
    inv = torch.linalg.solve_triangular(low, torch.eye(k, dtype=h.dtype, device=DEV), upper=False)
    return inv.flip(0, 1).contiguous()


def _layout(n, k, osr, levels, block, base3):
    layout = sdq.sdq_layout_init(n, k, osr, levels, block)
    if base3:
        sdq.sdq_layout_set_packing(layout, sdq.SDQ_PACK_BASE3)
    sdq.sdq_prepare_layout(layout)
    return layout


def _bytes(n):
    return torch.empty(max(1, n), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "linear":
        calls = []
        for k, ns, osr, x, coded in _linear_inputs(case, seed):
            encs = [sdq.Encoded(_layout(n, k, osr, case["levels"], 256, case["base3"]),
                                _pack(c, case["levels"], case["base3"]), s)
                    for n, (c, s) in zip(ns, coded)]
            ys = [torch.empty(case["m"], n, device=DEV) for n in ns]
            layouts = [e.layout for e in encs]
            calls.append({"x": x, "encs": encs, "ys": ys,
                          "group": sdq.LinearGroup(encs, ys) if len(ns) > 1 else None,
                          "ws": _bytes(sdq.sdq_linear_group_workspace_bytes(layouts, case["m"]))})
        return {"kind": kind, "calls": calls}
    if kind == "encode":
        layout = _layout(case["n"], case["k"], case["osr"], case["levels"], case["block"], case["base3"])
        return {"kind": kind, "w": _weights(_gen(seed, 1), case["n"], case["k"]), "layout": layout,
                "codes": _bytes(sdq.sdq_codes_bytes(layout)), "scales": torch.empty(case["n"], device=DEV),
                "ws": _bytes(sdq.sdq_quantize_workspace_bytes(layout))}
    if kind == "calibrate":
        k = case["k"]
        x = _calibration_rows(seed, case["rows"], k)
        return {"kind": kind, "x": x, "lam": _damping(x, k),
                "h": torch.empty(k, k, dtype=torch.float64, device=DEV),
                "u": torch.empty(k, k, dtype=torch.float64, device=DEV),
                "ws": _bytes(sdq.sdq_hessian_factor_workspace_bytes(k))}
    k = case["k"]
    x = _calibration_rows(seed, min(2048, 2 * k), k)
    xd = x.double()
    layout = _layout(case["n"], k, case["osr"], case["levels"], case["block"], False)
    return {"kind": kind, "w": _weights(_gen(seed, 1), case["n"], k), "layout": layout,
            "u": _factor(2 * (xd.t() @ xd), _damping(x, k)),
            "codes": _bytes(sdq.sdq_codes_bytes(layout)), "scales": torch.empty(case["n"], device=DEV),
            "ws": _bytes(sdq.sdq_quantize_compensated_workspace_bytes(layout))}


def run(state):
    kind = state["kind"]
    if kind == "linear":
        out = []
        for c in state["calls"]:
            if c["group"] is not None:
                sdq.sdq_linear_group(c["x"], c["group"], c["ws"])
            else:
                sdq.linear(c["x"], c["encs"][0], workspace=c["ws"], out=c["ys"][0])
            out += c["ys"]
        return out
    if kind == "encode":
        sdq.sdq_quantize(state["w"], state["layout"], state["codes"], state["scales"], state["ws"])
        return [state["codes"], state["scales"]]
    if kind == "calibrate":
        state["h"].zero_()
        sdq.sdq_hessian_accumulate(state["x"], state["h"])
        sdq.sdq_hessian_factor(state["h"], state["lam"], state["u"], state["ws"])
        return [state["h"], state["u"]]
    sdq.sdq_quantize_compensated(state["w"], state["layout"], state["u"], state["codes"], state["scales"],
                                 state["ws"])
    return [state["codes"], state["scales"]]


def _bits(case):
    return 1 if case["levels"] == 2 else (1.6 if case.get("base3") else 2)


def work(case):
    """The inputs once, the outputs once; the contraction over the codes and the expansion of the
    activations to the oversampled length (linears), the interpolation of every block (encoder)."""
    kind = case["kind"]
    if kind == "linear":
        by = fl = 0
        size = 4 if case["dtype"] == "f32" else 2
        for k, ns, osr in _groups(case["groups"]):
            k_up = (k // 256) * int(round(osr * 256))
            by += case["m"] * k * size + sum(n * k_up * _bits(case) / 8 + 4 * n + 4 * case["m"] * n for n in ns)
            fl += 2 * case["m"] * k_up * (256 + sum(ns))
        return {"bytes": by, "flops": fl}
    if kind == "calibrate":
        k, rows = case["k"], case["rows"]
        return {"bytes": 4 * rows * k + 3 * 8 * k * k, "flops": rows * k * (k + 1) + 2 * k ** 3 / 3}
    n, k, b = case["n"], case["k"], case["block"]
    m = int(round(case["osr"] * b))
    k_up = (k // b) * m
    by = 4 * n * k + n * k_up * _bits(case) / 8 + 4 * n
    interpolation = 2 * n * (k // b) * (m - math.gcd(b, m)) * b
    if kind == "encode":
        return {"bytes": by, "flops": interpolation}
    # the loop's correction of the later columns, and each block's reconstruction
    return {"bytes": by + 8 * k * (k + b) // 2, "flops": 2 * interpolation + n * k * (k - b) + 2 * n * k_up * b}


def tolerance(case):
    kind = case["kind"]
    if kind == "linear":
        # up to 16 rows: 32-bit sums; more: the activations at the oversampled length in 16 bits
        return {"rel": 1e-5, "max": 1e-4} if case["m"] <= 16 else {"rel": 1e-3, "max": 8e-3}
    if kind == "calibrate":
        return {"rel": 1e-10, "max": 1e-8}
    if kind == "compensate":
        # sums in another order round some 64-bit values the other way to 32 bits, and the rest of such
        # a row's codes follows another, equally good path
        return {"rel": 0.0, "max": 0.0, "differ": 0.01}
    return "exact"                                        # codes and scales are defined bit for bit


def exact(case, seed):
    kind = case["kind"]
    if kind == "linear":
        out = []
        for k, ns, osr, x, coded in _linear_inputs(case, seed):
            m_up, nb = int(round(osr * 256)), k // 256
            e = _sylvester(256) @ _decimate(256, m_up)
            xt = (x.double().view(-1, 256) @ e).view(case["m"], nb * m_up)
            for n, (c, s) in zip(ns, coded):
                y = torch.empty(case["m"], n, dtype=torch.float64, device=DEV)
                for r in range(0, n, 2048):
                    y[:, r:r + 2048] = xt @ c[r:r + 2048].double().t().contiguous()
                out.append(y * s.double()[None, :])
        return out
    if kind == "calibrate":
        x = _calibration_rows(seed, case["rows"], case["k"])
        xd = x.double()
        h = 2 * (xd.t().contiguous() @ xd)
        return [h, _factor(h, _damping(x, case["k"]))]
    w = _weights(_gen(seed, 1), case["n"], case["k"])
    b = case["block"]
    u = _sylvester(b) @ _upsample(b, int(round(case["osr"] * b)))
    scales = torch.cat([(r.double().view(-1, b) @ u).view(r.shape[0], -1).abs().amax(1) for r in w.split(256)])
    return [None, scales]                                 # codes are decisions, not computed numbers
