"""The work that a user of this framework has it do, as cases to be timed.

A case is one call of a public entry point on compressed layers that are
resident on the GPU: the fused decode-GEMV of token generation (one layer, or
the layers of a block that share an input), decompression to BF16 weights or
to one-byte codes (one layer, or a block of layers), and the prefill linear
layer on the matrix cores.  Weights are synthetic (heavy-tailed rows with a
log-normal scale, or Gaussian rows with outliers), quantised at a scale that
gives the case's entropy; the layer views, workspaces and outputs are kept
between calls, as a serving program keeps them.
"""
import math

import torch

import paper_2601_22787_amd as eq

Q_MAX = {1: 448.0, 2: 127.0}  # base formats: 1 = E4M3, 2 = Int8
SAMPLE_ROWS = 512             # rows that the scale search quantises


def _case(name, op, shapes, version, bits, **more):
    """shapes: the layers of the call as rows x columns, joined by '+'.
    fmt: base format; tokens: rows of the input; tile or chunk layout by the
    rules below; order: version 2 cut over sorted rows; dist: 't4', 't5'
    (Student t) or 'outliers'; bias: with a bias vector."""
    c = {"name": name, "op": op, "shapes": shapes, "version": version, "bits": bits, "fmt": 1,
         "tokens": 0, "order": False, "dist": "t5", "bias": False}
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: one token through a small projection, where the
        # launches and the host's part count
        _case("gemv small", "gemv", "1024x1024", 2, 2.0, tokens=1),
        # one token through a 4096-wide attention projection, 3 bits, in the
        # default one-symbol container
        _case("gemv attention v1", "gemv", "4096x4096", 1, 3.0, tokens=1),
        # eight sequences through an MLP down projection in the same container
        _case("gemv down b8 v1", "gemv", "4096x11008", 1, 2.0, tokens=8, dist="outliers"),
        # one token through the largest matrix of a 70B model's MLP at 2 bits
        _case("gemv large", "gemv", "8192x28672", 2, 2.0, tokens=1, dist="t4"),
        # the query, key and value projections of a 70B block, one token
        _case("qkv", "gemv_multi", "8192x8192+1024x8192+1024x8192", 2, 3.0, tokens=1),
        # the gate and up projections of a 7B block for eight sequences, rows
        # with and without outliers sorted apart
        _case("gate up b8", "gemv_multi", "11008x4096+11008x4096", 2, 2.0, tokens=8, order=True,
              dist="outliers"),
        # a speculative batch on a layer of odd sizes in the Int8 format
        _case("gemv ragged int8", "gemv", "3001x4840", 1, 4.0, tokens=3, fmt=2, bias=True),
        # block-wise decompression of a 70B block's attention to BF16
        _case("attention to bf16", "bf16_multi", "8192x8192+1024x8192+1024x8192+8192x8192", 1,
              3.0),
        # a large layer kept for generation, decompressed for other use
        _case("large to bf16 v2", "bf16", "28672x8192", 2, 3.0),
        # the one-byte block buffer of a 7B block's MLP, ahead of its prefill
        _case("mlp to codes v2", "codes_multi", "11008x4096+11008x4096+4096x11008", 2, 2.0,
              dist="outliers"),
        # a short prompt: 100 tokens through a layer kept for generation
        _case("prefill short", "gemm", "11008x4096", 2, 2.5, tokens=100, fmt=2, bias=True),
        # a long prompt through the largest matrix
        _case("prefill long", "gemm", "8192x28672", 1, 2.0, tokens=2048, dist="t4"),
    ]


MOST_PARAMS = 8192 * 28672
MOST_GEMM = MOST_PARAMS * 2048


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng, params, step):
    """About `params` weights, neither side under 256 nor over 28672; most
    widths are whole multiples of 128, some only of `step`."""
    side = math.sqrt(params)
    cols = min(28672, max(256, int(side * math.exp(rng.uniform(-1.0, 1.0)))))
    grain = 128 if rng.random() < 0.7 else step
    cols = max(256, cols // grain * grain)
    rows = min(28672, max(256, params // cols))
    if rng.random() < 0.5:
        rows = max(256, rows // 128 * 128)
    return rows, cols


def draw(rng):
    op = rng.choice(["gemv", "gemv", "gemv_multi", "bf16", "codes", "bf16_multi", "codes_multi",
                     "gemm", "gemm"])
    version = rng.choice([1, 2])
    n = rng.choice([2, 3]) if op.endswith("_multi") else 1
    total = _log(rng, 1 << 18, MOST_PARAMS)
    step = 16 if op == "gemm" else 4
    rows, cols = _shape(rng, max(1 << 17, total // n), step)
    while rows * cols * n > MOST_PARAMS:
        rows = rows // 2
    shapes = [(rows, cols)]
    for _ in range(n - 1):
        r = max(256, rows // rng.choice([1, 1, 4, 8]))
        shapes.append((r, cols))
    tokens = 0
    if op.startswith("gemv"):
        tokens = rng.randint(1, 8)
    elif op == "gemm":
        tokens = min(_log(rng, 9, 2048), max(9, MOST_GEMM // (rows * cols)))
    return {"op": op, "shapes": "+".join("%dx%d" % s for s in shapes), "version": version,
            "bits": round(rng.uniform(2.0, 4.0), 2), "fmt": rng.choice([1, 1, 2]),
            "tokens": tokens, "order": version == 2 and rng.random() < 0.25,
            "dist": rng.choice(["t4", "t5", "outliers"]),
            "bias": tokens > 0 and rng.random() < 0.5}


def _shapes(case):
    return [tuple(int(v) for v in s.split("x")) for s in case["shapes"].split("+")]


def _chunk(case):
    """Symbols per chunk, one for the layers of a call: 4096 when its largest
    matrix has up to 2M weights, 16384 up to 64M, 65536 beyond."""
    n = max(r * c for r, c in _shapes(case))
    return 4096 if n <= 1 << 21 else 16384 if n < 1 << 26 else 65536


def _layout(case, rows, cols):
    """Version 1: chunk symbols and lanes; version 2: tile rows and columns
    (the taller tile when the matrix has 2048 of them)."""
    c = _chunk(case)
    if case["version"] == 1:
        return c, 256 if c >= 65536 else 64
    tall, tc = (256, 256) if c >= 65536 else (128, c // 128)
    tiles = -(-rows // tall) * -(-cols // tc)
    return (tall if tiles >= 2048 else tall // 2), tc


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) % (1 << 62))
    return g


def _weights(case, g, rows, cols):
    """BF16 weights on the GPU."""
    if case["dist"] == "outliers":
        w = torch.randn(rows, cols, device="cuda", generator=g)
        u = torch.rand(rows, cols, device="cuda", generator=g)
        w = torch.where(u < 0.0005, 20.0, torch.where(u > 0.9995, -20.0, w))
        del u
        sigma = 0.7
    else:
        nu = int(case["dist"][1:])
        chi = torch.zeros(rows, cols, device="cuda")
        for _ in range(nu):
            chi += torch.randn(rows, cols, device="cuda", generator=g).square_()
        w = torch.randn(rows, cols, device="cuda", generator=g) / (chi / nu).sqrt_()
        del chi
        sigma = 0.5
    w *= torch.exp(sigma * torch.randn(rows, 1, device="cuda", generator=g))
    return w.to(torch.bfloat16)


def _quantise(w, s, fmt):
    """Values of the codes of weights w (float) at row scales s (float)."""
    u = (w / s).clamp_(-Q_MAX[fmt], Q_MAX[fmt])
    if fmt == 2:
        return u.round_()
    return u.to(torch.float8_e4m3fn).float()


def _entropy(v):
    """Bits per value of the empirical distribution of the integers v (< 1024)."""
    n = torch.bincount(v.reshape(-1), minlength=1024).double()
    p = n[n > 0] / n.sum()
    return float(-(p * p.log2()).sum())


def _scales(case, w):
    """BF16 row scales: AbsMax times the multiplier whose codes have the
    case's entropy on sampled rows."""
    fmt = case["fmt"]
    top = w.abs().amax(dim=1).float()
    pick = torch.linspace(0, w.shape[0] - 1, min(SAMPLE_ROWS, w.shape[0]), device="cuda").long()
    sw, st = w[pick].float(), top[pick]
    lo, hi = -4.0, 24.0
    for _ in range(18):
        mid = (lo + hi) / 2
        s = (st * (2.0 ** mid / Q_MAX[fmt])).to(torch.bfloat16).float()[:, None]
        v = _quantise(sw, s, fmt)
        ids = (v + 512).int() if fmt == 2 else \
            (v + 0.0).to(torch.float8_e4m3fn).view(torch.uint8).int()
        if _entropy(ids) > case["bits"]:
            lo = mid
        else:
            hi = mid
    return (top * (2.0 ** ((lo + hi) / 2) / Q_MAX[fmt])).to(torch.bfloat16)


def _inputs(case, g, rows_list, cols):
    x = b = None
    if case["tokens"]:
        x = torch.randn(case["tokens"], cols, device="cuda", generator=g).to(torch.bfloat16)
        if case["bias"]:
            b = [torch.randn(r, device="cuda", generator=g).to(torch.bfloat16) for r in rows_list]
    return x, b


def prepare(case, seed):
    g = _generator(seed)
    shapes = _shapes(case)
    layers = []
    for rows, cols in shapes:
        w = _weights(case, g, rows, cols)
        s = _scales(case, w)
        bits = w.view(torch.int16).cpu().numpy().view("uint16")
        s16 = s.view(torch.int16).cpu().numpy().view("uint16")
        del w
        if case["version"] == 1:
            c, lanes = _layout(case, rows, cols)
            blob = eq.eqe_encode(bits, 1.0, chunk_syms=c, lanes=lanes, base_format=case["fmt"],
                                 scale_bf16=s16)
        else:
            tr, tc = _layout(case, rows, cols)
            blob = eq.eqe_encode2(bits, 1.0, tile_rows=tr, tile_cols=tc,
                                  base_format=case["fmt"], scale_bf16=s16,
                                  row_order=case["order"])
        layers.append(eq.Layer(blob))
    x, bias = _inputs(case, g, [r for r, _ in shapes], shapes[0][1])
    state = {"case": dict(case), "layers": layers, "x": x, "bias": bias, "ws": None}
    op, t = case["op"], case["tokens"]
    kind = {"bf16": torch.bfloat16, "codes": torch.uint8}.get(op.split("_")[0])
    if kind is not None:
        state["out"] = [torch.empty(r, c, dtype=kind, device="cuda") for r, c in shapes]
    else:
        state["out"] = [torch.empty(t, r, dtype=torch.float32, device="cuda") for r, _ in shapes]
        state["ws"] = (eq.multi_workspace(layers, t) if op == "gemv_multi" else
                       layers[0].workspace(t) if op == "gemv" else layers[0].gemm_workspace(t))
    return state


def run(state):
    op, layers, out = state["case"]["op"], state["layers"], state["out"]
    x, b, ws, t = state["x"], state["bias"], state["ws"], state["case"]["tokens"]
    if op == "gemv":
        eq.eq_decode_gemv(layers[0], x, t, b[0] if b else None, out[0], ws)
    elif op == "gemv_multi":
        eq.eq_decode_gemv_multi(layers, x, t, b, out, ws)
    elif op == "gemm":
        eq.eq_decode_gemm(layers[0], x, t, b[0] if b else None, out[0], ws)
    elif op == "bf16":
        eq.eq_decode_bf16(layers[0], out[0])
    elif op == "codes":
        eq.eq_decode_codes(layers[0], out[0])
    elif op == "bf16_multi":
        eq.eq_decode_bf16_multi(layers, out)
    else:
        eq.eq_decode_codes_multi(layers, out)
    return out


def work(case):
    """Bytes: the payload at the case's entropy, the coder states (4 bytes a
    lane and chunk, or a tile row and tile), the scales, inputs and outputs.
    FLOPs: the products of the linear layer."""
    t, op, total, flops = case["tokens"], case["op"], 0.0, 0.0
    for rows, cols in _shapes(case):
        a, b = _layout(case, rows, cols)
        states = rows * cols / a * b if case["version"] == 1 else rows * -(-cols // b)
        total += rows * cols * case["bits"] / 8 + 4 * states + 2 * rows
        if t:
            total += 4 * t * rows + (2 * rows if case["bias"] else 0)
            flops += 2.0 * rows * cols * t
        else:
            total += rows * cols * (2 if op.startswith("bf16") else 1)
    if t:
        total += 2 * t * _shapes(case)[0][1]
    return {"bytes": total, "flops": flops}


def tolerance(case):
    """Decoding is lossless and the dequantised product is rounded once, so
    codes and BF16 weights are exact.  The linear layers form exact products
    and add them in fp32: they are 2e-8 to 1.3e-7 of the result's norm off
    the sums in 64 bits, and longer serial sums would be a few times that."""
    if not case["tokens"]:
        return "exact"
    return {"rel": 2e-6, "max": 1e-4}


def exact(case, seed):
    g = _generator(seed)
    shapes = _shapes(case)
    fmt, values = case["fmt"], []
    for rows, cols in shapes:
        w = _weights(case, g, rows, cols)
        s = _scales(case, w).float()[:, None]
        v = torch.cat([_quantise(w[i:i + 1024].float(), s[i:i + 1024], fmt)
                       for i in range(0, rows, 1024)])
        del w
        if case["op"].startswith("codes"):
            v += 0.0  # one zero
            values.append((v.to(torch.int8) if fmt == 2 else
                           v.to(torch.float8_e4m3fn)).view(torch.uint8))
        else:
            values.append((v, s.double()))
    if case["op"].startswith("codes"):
        return values
    if not case["tokens"]:
        return [v.double() * s for v, s in values]
    x, bias = _inputs(case, g, [r for r, _ in shapes], shapes[0][1])
    out = []
    for i, (v, s) in enumerate(values):
        y = torch.cat([x.double() @ v[k:k + 4096].double().t().contiguous()
                       for k in range(0, v.shape[0], 4096)], dim=1) * s.t()
        out.append(y + bias[i].double() if bias else y)
    return out
