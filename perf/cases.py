"""Timed cases of libentro: the calls that a user of the library makes, over the sizes they are made at.

A case is a dict of plain values.  Its "call" says which entry points one pass goes through:

  single    entro_decode / entro_decode_dequant on one tensor
  plan      a launch over many tensors, prepared once (entro_plan_init) and run again and again (entro_plan_run)
  batch     entro_decode_batch / entro_decode_dequant_batch: validated, prepared and launched on every call
  gemv      entro_decode_gemv on one tensor
  step      a token step: per layer one prepared GEMV launch for each group of products that may run together
  compress  range, quantisation, codebook and encoding of one fp32 tensor that lies in device memory

"model" names one of the weight sets of synth/configs.py, of which a case takes the first "layers" layers; an empty
"model" means "tensors" matrices of rows x cols.  Weights come from the seed by the same laws as in synth/ (drawn on
the device, which is quick) and go through the library's own device-side compression; the entry points inside the
segments are what entro_sub_index defines, added up on the device.  Outputs are zeroed once and written by every pass.
"""
import numpy as np
import torch

import paper_2505_02380_amd as E
import synth

DEV = "cuda:0"
OUTS = {"u8": E.ENTRO_U8, "u4": E.ENTRO_U4_PACKED, "f32": E.ENTRO_F32, "bf16": E.ENTRO_BF16}
DTYPES = {"u8": torch.uint8, "u4": torch.uint8, "f32": torch.float32, "bf16": torch.bfloat16}
CFG = {"smol": 2, "phi3": 3, "mistral": 4}
# products of a layer that depend on each other's results go into launches of their own
GROUPS = {"phi3": ((0, 1), (1, 2), (2, 3), (3, 4)), "mistral": ((0, 3), (3, 4), (4, 6), (6, 7))}
# mean code length in bits, as these laws give it at the sizes used here (a quarter of a bit more for small tensors)
MEAN_BITS = {("t4", 8): 3.2, ("t5", 8): 3.5, ("laplace", 8): 5.0, ("uniform", 8): 7.95,
             ("t4", 4): 1.3, ("t5", 4): 1.3, ("laplace", 4): 1.55, ("uniform", 4): 4.0}


def _case(name, call, **kw):
    c = {"name": name, "call": call, "model": "", "layers": 0, "tensors": 1, "rows": 0, "cols": 0, "bits": 8, "dist": "t5",
         "out": "bf16", "chunk": 4096, "sub": 256, "max_len": 0}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call there is: one norm-gain vector of the 1.7B model, a few microseconds of work behind a launch
        _case("norm_gain_f32", "single", rows=1, cols=2048, dist="uniform", out="f32"),
        # one square attention matrix decoded to bytes with its entry points: the smallest weight tensor of the sets
        _case("one_2048x2048_u8", "single", rows=2048, cols=2048, dist="t4", out="u8"),
        # the same kind of call as the README shows it: a tensor encoded without entry points, straight to bf16
        _case("one_4096x4096_bf16_plain", "single", rows=4096, cols=4096, sub=0),
        # a layer brought in just before it is used: seven tensors, validated and launched by one call
        _case("mistral_layer_bf16_batch", "batch", model="mistral", layers=1),
        # a few matrices of no round size, exact fp32 weights (a fine-tuning job that loads its base weights)
        _case("ragged_f32", "plan", tensors=5, rows=3001, cols=1283, out="f32", sub=512),
        # whole models at load time: bytes, packed nibbles, and the largest: every weight of the 7B model as bf16
        _case("smol_all_u8", "plan", model="smol", layers=24, dist="t4", out="u8"),
        _case("phi3_all_u4", "plan", model="phi3", layers=32, bits=4, dist="laplace", out="u4", chunk=8192, sub=512),
        _case("mistral_all_bf16", "plan", model="mistral", layers=32),
        # one product at batch 1 as the README shows it, without entry points
        _case("one_gemv_4096x4096_plain", "gemv", rows=4096, cols=4096, out="f32", sub=0),
        # token generation: a step over all layers, four dependent launches each
        _case("mistral_token_step", "step", model="mistral", layers=32, out="f32"),
        _case("phi3_token_step_bf16", "step", model="phi3", layers=32, bits=4, dist="laplace", out="bf16", chunk=8192, sub=512),
        # the way in: one large fp32 matrix compressed on the device
        _case("compress_14336x4096", "compress", rows=14336, cols=4096, sub=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    call = rng.choice(["single", "plan", "plan", "batch", "gemv", "step", "compress"])
    bits = rng.choice([8, 8, 4])
    chunk = rng.choice([1024, 2048, 4096, 4096, 8192])
    c = _case("", call, bits=bits, chunk=chunk, dist=rng.choice(["t4", "t5", "t5", "laplace"]))
    del c["name"]
    c["max_len"] = rng.choice([0, 0, 14])
    # entry points as a user sets them: none, or every 128 to 512 symbols (at most 16 a segment)
    c["sub"] = rng.choice([0, max(chunk // 16, 128), max(chunk // 16, 256), max(chunk // 8, 256)])
    c["rows"] = _log_int(rng, 1, 16384)
    c["cols"] = _log_int(rng, 64, 16384)
    if rng.random() < 0.7:                       # layers of models are multiples of 64 or so; the rest is of any size
        c["rows"] = max(64, c["rows"] // 64 * 64)
        c["cols"] = max(64, c["cols"] // 64 * 64)
    most = 1 << 28
    if call in ("plan", "batch", "step"):
        c["tensors"] = rng.randint(1, 28)
    if call == "single" and c["sub"] == 0:
        most = 1 << 26
    if call in ("gemv", "step"):
        c["out"] = rng.choice(["f32", "bf16"])
        c["cols"] = max(64, c["cols"] // 8 * 8)  # activation vectors are whole 16-byte pieces
        if call == "gemv":
            most = 1 << 26
    elif call == "compress":
        c["sub"], most = 0, 1 << 26
    else:
        c["out"] = rng.choice(["u8", "f32", "bf16", "bf16"] + (["u4", "u4"] if bits == 4 else []))
    while c["rows"] * c["cols"] * c["tensors"] > most:
        if c["tensors"] > 1:
            c["tensors"] -= 1
        else:
            c["rows"] //= 2
    return c


def _shapes(case):
    """[(rows, cols, law)] of the case's tensors."""
    if case["model"]:
        return [(s.rows, s.cols, {"uniform": "uniform", "laplace": "laplace"}.get(s.dist, case["dist"]))
                for s in synth.config_tensors(CFG[case["model"]], case["layers"])]
    return [(case["rows"], case["cols"], case["dist"])] * case["tensors"]


def _weights(n, dist, outliers, gen):
    """n fp32 weights on the device by one of the laws of synth/ (chi-square variables as sums of exponentials and a square)."""
    def exp(k=1.0):
        return torch.empty(n, device=DEV).exponential_(1.0, generator=gen).mul_(k)
    if dist == "uniform":
        return torch.rand(n, device=DEV, generator=gen).mul_(0.4).add_(0.8)
    if dist == "laplace":
        return exp().sub_(exp()).mul_(0.015)
    df = 4 if dist == "t4" else 5
    chi = exp(2.0).add_(exp(2.0))
    if df == 5:
        chi.add_(torch.randn(n, device=DEV, generator=gen).square_())
    w = torch.randn(n, device=DEV, generator=gen).div_(chi.div_(df).sqrt_()).mul_(0.02)
    if outliers:
        at = torch.randint(n, (max(1, n // 1000),), device=DEV, generator=gen).unique()
        sign = torch.randint(2, (at.numel(),), device=DEV, generator=gen).mul_(2).sub_(1)
        w[at] = sign.float() * (10.0 * float(w.std()))
    return w


def _entry_points(q, cb, sub):
    """entro_sub_index on the device: stream bits of every `sub` symbols."""
    n = q.numel()
    ln = torch.from_numpy(np.ctypeslib.as_array(cb.len).copy()).to(DEV).to(torch.int32)
    full = n // sub * sub
    parts = [ln[q[lo:min(lo + (1 << 26), full)].int()].view(-1, sub).sum(1) for lo in range(0, full, 1 << 26)]
    if full < n:
        parts.append(ln[q[full:].int()].sum().view(1))
    return torch.cat(parts).to(torch.int16)


def _tensor(case, rows, cols, dist, gen):
    """One compressed tensor in device memory."""
    w = _weights(rows * cols, dist, case["model"] == "smol" and dist != "uniform", gen)
    scheme = E.ENTRO_UNSIGNED if dist == "uniform" else E.ENTRO_ASYMMETRIC
    d, q = E.compress_on_device(w, case["bits"], scheme, case["chunk"], rows=rows, cols=cols, max_len=case["max_len"], return_q=True)
    if case["sub"]:
        d.enc.sub_symbols = case["sub"]
        d.sub_bits = _entry_points(q, d.enc.cb, case["sub"])
    return d


def _views(sizes, dtype, align=16):
    """One zeroed buffer and a 16-byte aligned view of it for every size (in elements)."""
    step = align // torch.empty(0, dtype=dtype).element_size()
    flat = torch.zeros(sum(-(-s // step) * step for s in sizes), dtype=dtype, device=DEV)
    views, pos = [], 0
    for s in sizes:
        views.append(flat[pos:pos + s])
        pos += -(-s // step) * step
    return flat, views


def _workspace(ts, op):
    return torch.zeros(max(256, E.entro_workspace_bytes(ts, op)), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    call, out = case["call"], case["out"]
    if call == "compress":
        n = case["rows"] * case["cols"]
        arena = torch.zeros((n * case["bits"] // 8 + 79) // 16 * 16, dtype=torch.uint8, device=DEV)   # no Huffman code of 2^bits symbols needs more
        return {"case": case, "w": _weights(n, case["dist"], False, gen), "out": arena}
    shapes = _shapes(case)
    dts = [_tensor(case, r, c, d, gen) for r, c, d in shapes]
    st = {"case": case, "dts": dts, "type": OUTS[out]}
    if call in ("gemv", "step"):
        flat, ys = _views([r for r, _, _ in shapes], DTYPES[out])
        if case["model"]:
            per = len(shapes) // case["layers"]
            groups = [(per * l + a, per * l + b) for l in range(case["layers"]) for a, b in GROUPS[case["model"]]]
        else:
            groups = [(i, i + 1) for i in range(len(shapes))]
        st.update(out=flat, xs=[], ws=[], plans=[])
        for a, b in groups:                      # the products of a group multiply the same activations
            x = torch.randn(shapes[a][1], device=DEV, generator=gen).to(torch.bfloat16)
            st["xs"].append(x)
            ts = [dts[i].ctensor(ys[i], x) for i in range(a, b)]
            if call == "gemv":
                need = E.entro_gemv_workspace_bytes(ts[0])
                st["t"] = ts[0]
                st["ws"] = torch.zeros(need, dtype=torch.uint8, device=DEV) if need else None
            else:
                st["ws"].append(_workspace(ts, E.ENTRO_OP_GEMV))
                st["plans"].append(E.entro_plan_init(ts, E.ENTRO_OP_GEMV, st["type"], st["ws"][-1]))
        return st
    sizes = [r * c for r, c, _ in shapes]
    st["out"], views = _views([(n + 1) // 2 for n in sizes] if out == "u4" else sizes, DTYPES[out])
    ts = [d.ctensor(v) for d, v in zip(dts, views)]
    op = E.ENTRO_OP_DECODE if out in ("u8", "u4") else E.ENTRO_OP_DEQUANT
    if call == "single":
        st["t"] = ts[0]
        st["fn"] = E.entro_decode if op == E.ENTRO_OP_DECODE else E.entro_decode_dequant
        return st
    st["ws"] = _workspace(ts, op)
    if call == "batch":
        st["ts"] = ts
        st["fn"] = E.entro_decode_batch if op == E.ENTRO_OP_DECODE else E.entro_decode_dequant_batch
    else:
        st["plan"] = E.entro_plan_init(ts, op, st["type"], st["ws"])
    return st


def run(st):
    case = st["case"]
    call = case["call"]
    if call == "compress":
        d, q = E.compress_on_device(st["w"], case["bits"], E.ENTRO_ASYMMETRIC, case["chunk"], rows=case["rows"], cols=case["cols"],
                                    max_len=case["max_len"], return_q=True)
        st["out"][:d.stream.numel()].copy_(d.stream)          # where the program gathers the model's streams
        return [st["out"], d.offsets, q, d.enc.qp.scale, d.enc.qp.zero_point]
    if call == "single":
        st["fn"](st["t"], st["type"])
    elif call == "batch":
        st["fn"](st["ts"], st["type"], st["ws"])
    elif call == "plan":
        E.entro_plan_run(st["plan"])
    elif call == "gemv":
        E.entro_decode_gemv(st["t"], st["type"], st["ws"])
    else:
        for p in st["plans"]:
            E.entro_plan_run(p)
    return st["out"]


def work(case):
    """Compressed bytes and offset tables in and results out (and, for the product, the activations); for compression the
    fp32 weights in and symbols, stream and offsets out."""
    nbytes, flops = 0.0, 0.0
    for rows, cols, dist in _shapes(case):
        n = rows * cols
        packed = n * MEAN_BITS[(dist, case["bits"])] / 8 + 8 * (n / case["chunk"] + 1)
        if case["call"] == "compress":
            nbytes += 4 * n + n + packed
        elif case["call"] in ("gemv", "step"):
            nbytes += packed + 2 * cols + rows * (4 if case["out"] == "f32" else 2)
            flops += 2.0 * n
        else:
            nbytes += packed + n * {"u8": 1, "u4": 0.5, "f32": 4, "bf16": 2}[case["out"]]
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Decoded integers, (q - z) * s and compressed streams are what they are to the last bit.  A GEMV sums exact products in
    fp32 in an order that is the implementation's own; with bf16 results half an ulp of the result comes on top."""
    if case["call"] not in ("gemv", "step"):
        return "exact"
    return {"rel": 1e-6, "max": 1e-5} if case["out"] == "f32" else {"rel": 4e-3, "max": 8e-3}


def _quantised(w, bits, dist):
    """(q - z, s) of fp32 weights, by the definition of the grid (fp32, true division, half to even), the difference as fp32."""
    top = (1 << bits) - 1
    lo, hi = w.min(), w.max()
    unsigned = dist == "uniform"
    s = (hi / torch.full_like(hi, top)) if unsigned else (hi - lo) / torch.full_like(hi, top)
    z = torch.zeros_like(s) if unsigned else torch.round(-lo / s)
    return torch.round(w / s).add_(z).clamp_(0, top).sub_(z), s


def exact(case, seed):
    """What run() returns, in 64 bits from the same weights: q and z are integers, s is the fp32 number that the grid has."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    call, out = case["call"], case["out"]
    if call == "compress":
        w = _weights(case["rows"] * case["cols"], case["dist"], False, gen)
        return [None, None, None, float((w.max() - w.min()).item() / ((1 << case["bits"]) - 1)), None]
    shapes = _shapes(case)
    if out in ("u8", "u4") or call not in ("gemv", "step") and sum(r * c for r, c, _ in shapes) > 1 << 28:
        return None                              # whole numbers, or too much to hold in 64 bits
    held = []
    for rows, cols, dist in shapes:
        d, s = _quantised(_weights(rows * cols, dist, case["model"] == "smol" and dist != "uniform", gen), case["bits"], dist)
        held.append((d.to(torch.bfloat16), s.double()))          # (integers of at most 256 in magnitude)
    if call in ("gemv", "step"):
        flat, ys = _views([r for r, _, _ in shapes], torch.float64, 16 * 8 // torch.empty(0, dtype=DTYPES[out]).element_size())
        per = len(shapes) // case["layers"] if case["model"] else 1
        groups = [(per * l + a, per * l + b) for l in range(case["layers"]) for a, b in GROUPS[case["model"]]] if case["model"] \
            else [(i, i + 1) for i in range(len(shapes))]
        for a, b in groups:
            x = torch.randn(shapes[a][1], device=DEV, generator=gen).to(torch.bfloat16).double()
            for i in range(a, b):
                ys[i].copy_((held[i][0].view(shapes[i][0], shapes[i][1]).double() * x).sum(1) * held[i][1])
        return flat
    sizes = [r * c for r, c, _ in shapes]
    flat, views = _views(sizes, torch.float64, 16 * 8 // torch.empty(0, dtype=DTYPES[out]).element_size())
    for v, (d, s) in zip(views, held):
        v.copy_(d.double() * s)
    return flat
