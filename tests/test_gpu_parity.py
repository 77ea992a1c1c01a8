"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle.

Bars: decoded integers bit-exact; fp32 dequant bit-exact; bf16 within 1 ulp
(the kernels round to nearest even, so equality is expected and asserted as
<= 1 ulp); GEMV relative error <= 1e-3 against the fp64 oracle, both as
||y - y*||_2 / ||y*||_2 and as max_r |y_r - y*_r| <= 1e-3 * max(|y*_r|, rms(y*)).
Inputs never come from the HIP path: symbols, codebooks and streams are built
by the oracle (or by the host library and re-decoded by the oracle)."""
import os

import numpy as np
import pytest
import torch

import oracle
import synth
import paper_2505_02380_amd as E
from paper_2505_02380_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _oracle_encoded(sym, bits, chunk, rows=0, cols=0, s=1.0, z=0, sub=0):
    """EncodedTensor whose codebook, stream (and entry points inside the segments, if sub is given) all come from
    the oracle."""
    ln, code, _ = oracle.codebook_from_symbols(sym, bits)
    stream, off = oracle.encode(sym, ln, code, chunk)
    full = np.zeros(1 << bits, np.uint8)
    full[: ln.size] = ln
    cb = E.entro_codebook_from_lengths(full, bits)
    assert np.array_equal(cb.codes(), code)
    qp = B.QParams(np.float32(s), int(z), bits, E.ENTRO_ASYMMETRIC)
    enc = B.EncodedTensor(stream, off, sym.size, chunk, cb, qp, rows, cols)
    if sub:
        enc.sub_symbols, enc.sub_bits = sub, oracle.sub_index(sym, ln, chunk, sub)
    return enc


def _bf16_ulp_diff(a_bits, b_bits):
    def key(u):
        u = u.astype(np.int32)
        return np.where(u & 0x8000, 0x8000 - u, u)       # monotone integer order of bf16 patterns
    return np.abs(key(a_bits) - key(b_bits))


def _gpu_decode(enc, out_type, batch=False):
    dt = E.to_device(enc, DEV)
    nbytes = enc.n if out_type == E.ENTRO_U8 else (enc.n + 1) // 2
    out = torch.full((nbytes + 64,), 0xAB, dtype=torch.uint8, device=DEV)      # guard bytes behind the output
    t = dt.ctensor(out)
    if batch:
        ws = torch.zeros(E.entro_workspace_bytes([t], E.ENTRO_OP_DECODE), dtype=torch.uint8, device=DEV)
        E.entro_decode_batch([t], out_type, ws)
    else:
        E.entro_decode(t, out_type)
    torch.cuda.synchronize()
    res = out.cpu().numpy()
    assert np.all(res[nbytes:] == 0xAB), "wrote past the end of the output"
    return res[:nbytes]


def _gpu_dequant(enc, out_type, batch=False):
    dt = E.to_device(enc, DEV)
    dtype = torch.float32 if out_type == E.ENTRO_F32 else torch.bfloat16
    out = torch.zeros(enc.n + 16, dtype=dtype, device=DEV)
    t = dt.ctensor(out)
    if batch:
        ws = torch.zeros(E.entro_workspace_bytes([t], E.ENTRO_OP_DEQUANT), dtype=torch.uint8, device=DEV)
        E.entro_decode_dequant_batch([t], out_type, ws)
    else:
        E.entro_decode_dequant(t, out_type)
    torch.cuda.synchronize()
    assert torch.all(out[enc.n:] == 0), "wrote past the end of the output"
    if out_type == E.ENTRO_F32:
        return out[: enc.n].cpu().numpy()
    return out[: enc.n].view(torch.int16).cpu().numpy().view(np.uint16)


def _gpu_gemv(enc, xb, y_type, batch=False):
    dt = E.to_device(enc, DEV)
    x = torch.from_numpy(xb.view(np.int16)).to(DEV).view(torch.bfloat16)
    y = torch.zeros(enc.rows + 8, dtype=torch.float32 if y_type == E.ENTRO_F32 else torch.bfloat16, device=DEV)
    t = dt.ctensor(y, x)
    if batch:
        ws = torch.zeros(max(E.entro_workspace_bytes([t], E.ENTRO_OP_GEMV), 16), dtype=torch.uint8, device=DEV)
        E.entro_decode_gemv_batch([t], y_type, ws)
    else:
        need = E.entro_gemv_workspace_bytes(t)
        ws = torch.zeros(need, dtype=torch.uint8, device=DEV) if need else None
        E.entro_decode_gemv(t, y_type, ws)
    torch.cuda.synchronize()
    assert torch.all(y[enc.rows:] == 0)
    return y[: enc.rows].float().cpu().numpy().astype(np.float64)


def _assert_gemv_close(y, y_ref, tol=1e-3):
    rel = np.linalg.norm(y - y_ref) / np.linalg.norm(y_ref)
    rms = np.sqrt(np.mean(y_ref ** 2))
    worst = np.max(np.abs(y - y_ref) / np.maximum(np.abs(y_ref), rms))
    assert rel <= tol and worst <= tol, (rel, worst)


# ---------------------------------------------------------------- integer decode
@pytest.mark.parametrize("batch", [False, True])
def test_config1_round_trip_bit_exact(batch):
    spec = synth.config_tensors(1)[0]
    w = synth.make_tensor(spec)
    q, s, z = oracle.quantize(w, 8, oracle.ASYMMETRIC)
    enc = _oracle_encoded(q, 8, 4096, s=s, z=z)
    assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8, batch), q)
    # the host library's own chain, re-decoded by the oracle
    enc2 = E.encode_tensor(w, 8, E.ENTRO_ASYMMETRIC, 4096)
    ref = oracle.decode(enc2.stream, enc2.offsets, enc2.n, 4096, enc2.cb.lengths(), enc2.cb.codes())
    assert np.array_equal(_gpu_decode(enc2, E.ENTRO_U8, batch), ref)


@pytest.mark.parametrize("bits", [8, 4])
def test_adversarial_streams_bit_exact(bits):
    for name, sym, chunk in synth.adversarial_symbol_cases(bits):
        enc = _oracle_encoded(sym, bits, chunk)
        assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8), sym), name
        assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8, batch=True), sym), name
        if bits == 4:
            assert np.array_equal(_gpu_decode(enc, E.ENTRO_U4_PACKED), oracle.pack_u4(sym)), name


def test_odd_chunk_sizes_take_the_scalar_store_path():
    rng = np.random.default_rng(31)
    sym = np.minimum(rng.geometric(0.4, 40001) - 1, 255).astype(np.uint8)
    for chunk in (1, 7, 1000, 4100):
        enc = _oracle_encoded(sym, 8, chunk)
        assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8), sym), chunk
    sym4 = (sym & 15).astype(np.uint8)
    for chunk in (2, 30, 1002):
        enc = _oracle_encoded(sym4, 4, chunk)
        assert np.array_equal(_gpu_decode(enc, E.ENTRO_U4_PACKED), oracle.pack_u4(sym4)), chunk


def test_shorter_last_segment_of_every_shape():
    # the last segment's whole blocks go through the row path and the rest through the scalar path:
    # sweep its length over none / less than a block / whole blocks / blocks and a rest, alone in the
    # tensor, alone in its wave (65 segments) and beside full ones
    rng = np.random.default_rng(77)
    chunk = 512
    base = np.minimum(rng.geometric(0.3, 66 * chunk) - 1, 255).astype(np.uint8)
    base[rng.random(base.size) < 0.002] = 255                       # a few long codes
    for full in (0, 1, 64, 65):
        for last in (1, 63, 64, 65, 127, 128, 129, 256, 383, 511):
            sym = base[: full * chunk + last]
            enc = _oracle_encoded(sym, 8, chunk, s=0.0123, z=3)
            tag = (full, last)
            assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8), sym), tag
            assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8, batch=True), sym), tag
            ref32 = oracle.dequant_f32(sym, enc.qp.scale, 3)
            assert np.array_equal(_gpu_dequant(enc, E.ENTRO_F32).view(np.uint32), ref32.view(np.uint32)), tag
            refb = oracle.dequant_bf16(sym, enc.qp.scale, 3)
            assert _bf16_ulp_diff(_gpu_dequant(enc, E.ENTRO_BF16, batch=True), refb).max() <= 1, tag
            sym4 = (sym & 15).astype(np.uint8)
            enc4 = _oracle_encoded(sym4, 4, chunk)
            assert np.array_equal(_gpu_decode(enc4, E.ENTRO_U4_PACKED), oracle.pack_u4(sym4)), tag
            assert np.array_equal(_gpu_decode(enc4, E.ENTRO_U8), sym4), tag
            assert _bf16_ulp_diff(_gpu_dequant(enc4, E.ENTRO_BF16), oracle.dequant_bf16(sym4, enc4.qp.scale, 0)).max() <= 1, tag


def test_codes_of_every_length_up_to_32():
    # lengths 1..31, 32, 32: the deepest code the format allows; symbols drawn so long codes are common
    ln = np.zeros(256, np.uint8)
    ln[:33] = list(range(1, 32)) + [32, 32]
    rng = np.random.default_rng(32)
    sym = rng.integers(0, 33, 30000).astype(np.uint8)
    code = oracle.canonical_codes(ln)
    stream, off = oracle.encode(sym, ln, code, 512)
    cb = E.entro_codebook_from_lengths(ln, 8)
    enc = B.EncodedTensor(stream, off, sym.size, 512, cb, B.QParams(1.0, 0, 8, 1))
    assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8), sym)


def test_more_long_prefixes_than_the_second_level_holds():
    # lengths 1..7, eight codes of 14 bits and 240 of 15: Kraft sum exactly 1; the 15-bit codes own 120
    # prefixes of the first-level table, so every one of them goes through the canonical search
    ln = np.zeros(256, np.uint8)
    ln[:7] = range(1, 8)
    ln[7:15] = 14
    ln[15:255] = 15
    assert sum(2.0 ** -int(l) for l in ln if l) == 1.0
    rng = np.random.default_rng(15)
    sym = rng.integers(0, 255, 64 * 1024 + 77).astype(np.uint8)          # long codes everywhere
    code = oracle.canonical_codes(ln)
    for chunk in (1024, 4096):
        stream, off = oracle.encode(sym, ln, code, chunk)
        cb = E.entro_codebook_from_lengths(ln, 8)
        enc = B.EncodedTensor(stream, off, sym.size, chunk, cb, B.QParams(1.0, 0, 8, 1))
        assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8), sym)
        assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8, batch=True), sym)


@pytest.mark.parametrize("bits,deepest", [(8, 9), (8, 10), (8, 11), (8, 14), (8, 15), (8, 20), (8, 21), (4, 9), (4, 10), (4, 14), (4, 15)])
def test_staircase_codes_around_the_widths_of_the_tables(bits, deepest):
    # lengths 1, 2, ..., d, d with d at the widths of the table pieces (10 bits searched and copied, 14 indexed, 20 in
    # the second level; 9 for the single codes of pair tables), decoded through every kind of table
    ln = np.zeros(1 << bits, np.uint8)
    ln[: deepest + 1] = list(range(1, deepest + 1)) + [deepest]
    rng = np.random.default_rng(100 * bits + deepest)
    cols, chunk = 512, 2048
    sym = rng.integers(0, deepest + 1, 70 * cols).astype(np.uint8)
    code = oracle.canonical_codes(ln)
    stream, off = oracle.encode(sym, ln, code, chunk)
    qp = B.QParams(np.float32(0.25), 7, bits, E.ENTRO_ASYMMETRIC)
    enc = B.EncodedTensor(stream, off, sym.size, chunk, E.entro_codebook_from_lengths(ln, bits), qp, sym.size // cols, cols)
    x = synth.make_x_bf16(9, deepest, cols)
    y_ref, _ = oracle.gemv(sym, enc.rows, cols, 0.25, 7, x)
    for batch in (False, True):
        assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8, batch), sym)
        assert np.array_equal(_gpu_dequant(enc, E.ENTRO_F32, batch), oracle.dequant_f32(sym, 0.25, 7))
        _assert_gemv_close(_gpu_gemv(enc, x, E.ENTRO_F32, batch), y_ref)


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("bits,deepest", [(8, 9), (8, 14), (8, 15), (8, 21), (8, 32), (4, 9), (4, 14), (4, 15)])
def test_lane_per_segment_codes_of_every_length_every_output(bits, deepest, batch):
    # segments of 384 symbols are too short to be shared by lanes: the kernels that give each a lane, with blocks in full and in
    # part, two wavefronts of segments and a shorter last one, whose symbols go one by one
    ln = np.zeros(1 << bits, np.uint8)
    ln[: deepest + 1] = list(range(1, deepest + 1)) + [deepest]
    rng = np.random.default_rng(deepest)
    cols, chunk = 192, 384
    sym = rng.integers(0, deepest + 1, 211 * cols).astype(np.uint8)
    stream, off = oracle.encode(sym, ln, oracle.canonical_codes(ln), chunk)
    qp = B.QParams(np.float32(0.25), 7, bits, E.ENTRO_ASYMMETRIC)
    enc = B.EncodedTensor(stream, off, sym.size, chunk, E.entro_codebook_from_lengths(ln, bits), qp, sym.size // cols, cols)
    x = synth.make_x_bf16(9, deepest, cols)
    y_ref, _ = oracle.gemv(sym, enc.rows, cols, 0.25, 7, x)
    assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8, batch), sym)
    assert np.array_equal(_gpu_dequant(enc, E.ENTRO_F32, batch), oracle.dequant_f32(sym, 0.25, 7))
    assert np.array_equal(_gpu_dequant(enc, E.ENTRO_BF16, batch), oracle.dequant_bf16(sym, 0.25, 7))
    if bits == 4:
        assert np.array_equal(_gpu_decode(enc, E.ENTRO_U4_PACKED, batch), oracle.pack_u4(sym))
    _assert_gemv_close(_gpu_gemv(enc, x, E.ENTRO_F32, batch), y_ref)
    _assert_gemv_close(_gpu_gemv(enc, x, E.ENTRO_BF16, batch), y_ref, tol=5e-3)   # y itself rounded to bf16


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("chunk,segments,last", [
    (512, 3, 0), (1024, 9, 0), (4096, 5, 0), (8192, 2, 0), (4096, 3, 1), (4096, 2, 63), (4096, 2, 65), (4096, 1, 4095), (3072, 4, 257),
    (448, 3, 0)])
@pytest.mark.parametrize("run", [False, True])
def test_segments_without_entry_points_cut_into_pieces(bits, chunk, segments, last, run):
    # 8 to 64 lanes per segment that find their starts themselves, short last segments, and (448) segments that are too
    # short for that;
    # `run`: a first segment of one symbol only, where every guess is a true start
    rng = np.random.default_rng(chunk + last + bits)
    top, n = (1 << bits) - 1, segments * chunk + last
    mid = (top + 1) // 2
    sym = np.clip(np.rint(rng.standard_t(5, n) * (12.0 if bits == 8 else 1.0) + mid), 0, top).astype(np.uint8)
    if run:
        sym[:chunk] = mid + (2 if bits == 8 else 1)
    sym[n // 2] = 0                                            # codes of the far tails
    sym[n - 1] = top
    enc = _oracle_encoded(sym, bits, chunk, 1, n, 0.25, 7 if bits == 8 else 3)
    z = enc.qp.zero_point
    assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8), sym)
    assert np.array_equal(_gpu_dequant(enc, E.ENTRO_F32), oracle.dequant_f32(sym, 0.25, z))
    if bits == 4:
        assert np.array_equal(_gpu_decode(enc, E.ENTRO_U4_PACKED), oracle.pack_u4(sym))


def _with_runs(bits, chunk, segments, last, fraction, every, seed):
    """Bell-shaped symbols; every `every`-th segment holds a run of one symbol, at an odd place behind codes of other
    lengths, whose code does not fall into step when it is read from a wrong bit."""
    rng = np.random.default_rng(seed)
    top, n = (1 << bits) - 1, segments * chunk + last
    mid = (top + 1) // 2
    sym = np.clip(np.rint(rng.standard_t(5, n) * (9.0 if bits == 8 else 1.0) + mid), 0, top).astype(np.uint8)
    run = int(chunk * fraction)
    for k in range(seed % every, segments, every):
        at = k * chunk + 5 + int(rng.integers(0, chunk - run - 5))
        sym[at: at + run] = mid + (k % 7 if bits == 8 else k % 3)
    return sym


@pytest.mark.parametrize("bits,chunk", [(8, 4096), (8, 2048), (8, 1024), (8, 512), (4, 4096), (4, 2048), (4, 8192)])
@pytest.mark.parametrize("fraction,every", [(0.5, 3), (0.9, 1), (0.97, 64)])
def test_runs_inside_segments_without_entry_points(bits, chunk, fraction, every):
    # lanes in a run agree on their starts one after the other, those beside it at once
    for segments, last in ((70, 0), (9, chunk // 3 + 1), (1, 0)):
        sym = _with_runs(bits, chunk, segments, last, fraction, every, segments)
        enc = _oracle_encoded(sym, bits, chunk, 1, sym.size, 0.25, 7)
        assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8), sym)
        assert np.array_equal(_gpu_dequant(enc, E.ENTRO_F32), oracle.dequant_f32(sym, 0.25, 7))
        assert np.array_equal(_gpu_dequant(enc, E.ENTRO_BF16), oracle.dequant_bf16(sym, 0.25, 7))
        if bits == 4:
            assert np.array_equal(_gpu_decode(enc, E.ENTRO_U4_PACKED), oracle.pack_u4(sym))


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("bits,chunk,cols,sub", [
    (8, 512, 64, 0), (8, 640, 72, 0), (8, 1152, 4104, 0), (8, 3968, 14336, 0), (8, 8192, 3072, 0), (4, 512, 200, 0), (4, 4096, 8, 0),
    (4, 8192, 5000, 0), (8, 4096, 4096, 256), (8, 1536, 72, 384), (8, 8192, 14336, 512), (8, 1024, 2048, 1024), (4, 4096, 3072, 256),
    (4, 8192, 200, 1024)])
def test_segments_shared_by_lanes_every_output_and_product(bits, chunk, cols, sub, batch):
    """Rows shorter and longer than a wavefront's unit, segments of odd lengths, a run that keeps guesses out of step, codes
    longer than the tables, and a stretch of rare symbols whose stream is longer than the unit's copy holds."""
    rows = -(-(11 * chunk + 300) // cols)
    n, top = rows * cols, (1 << bits) - 1
    rng = np.random.default_rng(chunk + cols)
    sym = np.clip(np.rint(rng.standard_t(3, n) * (9.0 if bits == 8 else 0.8) + (top + 1) // 2), 0, top).astype(np.uint8)
    sym[chunk + 7: chunk + 7 + chunk // 2] = (top + 1) // 2
    sym[5 * chunk + 3: 6 * chunk + 9] = rng.integers(0, top + 1, chunk + 6)
    z = 100 if bits == 8 else 6
    enc = _oracle_encoded(sym, bits, chunk, rows, cols, 0.25, z, sub)
    assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8, batch), sym)
    assert np.array_equal(_gpu_dequant(enc, E.ENTRO_F32, batch), oracle.dequant_f32(sym, 0.25, z))
    assert np.array_equal(_gpu_dequant(enc, E.ENTRO_BF16, batch), oracle.dequant_bf16(sym, 0.25, z))
    if bits == 4:
        assert np.array_equal(_gpu_decode(enc, E.ENTRO_U4_PACKED, batch), oracle.pack_u4(sym))
    xb = synth.make_x_bf16(0, 3, cols)
    y_ref, _ = oracle.gemv(sym, rows, cols, 0.25, z, xb)
    # fp32 sums of exact products: at most cols roundings of half an ulp, relative to the terms' magnitudes
    terms = np.abs((sym.astype(np.float64).reshape(rows, cols) - z) * 0.25) @ np.abs((xb.astype(np.uint32) << 16).view(np.float32).astype(np.float64))
    assert np.all(np.abs(_gpu_gemv(enc, xb, E.ENTRO_F32, batch) - y_ref) <= (cols + 2) * 2.0 ** -24 * terms)
    assert np.all(np.abs(_gpu_gemv(enc, xb, E.ENTRO_BF16, batch) - y_ref) <= 2.0 ** -8 * np.abs(y_ref) + (cols + 2) * 2.0 ** -24 * terms)


@pytest.mark.parametrize("y_type", [E.ENTRO_F32, E.ENTRO_BF16])
def test_tensors_of_different_segments_shared_in_one_launch(y_type):
    # alphabets, pieces, rows per unit and bits per symbol differ from tensor to tensor; the first is long enough for shares of
    # workgroups that start and end inside it
    rng = np.random.default_rng(5)
    encs, refs, xs = [], [], []
    for i, (bits, chunk, sub, rows, cols) in enumerate([(8, 4096, 512, 700, 3072), (4, 8192, 1024, 37, 8192), (8, 4096, 512, 20, 14336),
                                                        (4, 4096, 256, 9, 1000), (8, 1024, 512, 60, 64), (8, 8192, 8192, 33, 4096)]):
        top = (1 << bits) - 1
        sym = np.clip(np.rint(rng.standard_t(4, rows * cols) * ((3.0 + i) if bits == 8 else 1.0) + (top + 1) // 2), 0, top).astype(np.uint8)
        encs.append(_oracle_encoded(sym, bits, chunk, rows, cols, 0.02 * (i + 1), 5 + i, sub))
        refs.append(sym)
        xs.append(synth.make_x_bf16(2, i, cols))
    dts = [E.to_device(e, DEV) for e in encs]
    outs = [torch.zeros(e.n, dtype=torch.uint8, device=DEV) for e in encs]
    ts = [d.ctensor(o) for d, o in zip(dts, outs)]
    ws = torch.zeros(E.entro_workspace_bytes(ts, E.ENTRO_OP_DECODE), dtype=torch.uint8, device=DEV)
    plan = E.entro_plan_init(ts, E.ENTRO_OP_DECODE, E.ENTRO_U8, ws)
    assert plan.shared_wave_bytes > 0
    E.entro_plan_run(plan)
    for o, r in zip(outs, refs):
        assert np.array_equal(o.cpu().numpy(), r)
    ys = [torch.zeros(e.rows, dtype=torch.float32 if y_type == E.ENTRO_F32 else torch.bfloat16, device=DEV) for e in encs]
    xd = [torch.from_numpy(x.view(np.int16)).to(DEV).view(torch.bfloat16) for x in xs]
    ts = [d.ctensor(y, x) for d, y, x in zip(dts, ys, xd)]
    ws = torch.zeros(E.entro_workspace_bytes(ts, E.ENTRO_OP_GEMV), dtype=torch.uint8, device=DEV)
    plan = E.entro_plan_init(ts, E.ENTRO_OP_GEMV, y_type, ws)
    assert plan.shared_wave_bytes > 0
    for _ in range(2):
        for y in ys:
            y.zero_()
        E.entro_plan_run(plan)
        for e, y, r, x in zip(encs, ys, refs, xs):
            y_ref, _ = oracle.gemv(r, e.rows, e.cols, e.qp.scale, e.qp.zero_point, x)
            terms = np.abs((r.astype(np.float64).reshape(e.rows, e.cols) - e.qp.zero_point) * e.qp.scale) @ \
                np.abs((x.astype(np.uint32) << 16).view(np.float32).astype(np.float64))
            half_ulp = 0.0 if y_type == E.ENTRO_F32 else 2.0 ** -8
            assert np.all(np.abs(y.float().cpu().numpy() - y_ref) <= half_ulp * np.abs(y_ref) + (e.cols + 2) * 2.0 ** -24 * terms)


@pytest.mark.parametrize("bits,chunk,segments", [(8, 8192, 2700), (8, 1024, 17000), (4, 512, 41000), (8, 512, 49152), (8, 512, 49153)])
def test_more_segments_than_wavefronts_single_calls(bits, chunk, segments):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(segments)
    w = torch.randn(segments * chunk, device=DEV, generator=gen)
    d, q = E.compress_on_device(w, bits, E.ENTRO_ASYMMETRIC, chunk, return_q=True)
    out = torch.zeros(q.numel(), dtype=torch.uint8, device=DEV)
    E.entro_decode(d.ctensor(out), E.ENTRO_U8)
    assert torch.equal(out, q)


@pytest.mark.parametrize("chunk,sub", [(4096, 0), (640, 0), (4096, 512), (8192, 0)])
@pytest.mark.parametrize("run_len", [2, 11, 12, 13, 20, 32])
def test_runs_of_codes_around_the_starts_that_a_lane_keeps(chunk, sub, run_len):
    # twelve starts behind a lane's guess are kept: runs of shorter and of longer codes, in whole segments and beside other codes
    lengths = np.array(list(range(1, 32)) + [32, 32])
    rng = np.random.default_rng(chunk + run_len)
    n = 9 * chunk + chunk // 3 + 5
    sym = rng.choice(lengths.size, n, p=0.5 ** lengths / (0.5 ** lengths).sum()).astype(np.uint8)
    for k in (0, 2, 5, 9):
        sym[k * chunk + (3 if k else 0): min(n, (k + 1) * chunk - (k % 3) * 7)] = run_len - 1      # symbol s has a code of s + 1 bits
    sym[6 * chunk + 50: 6 * chunk + 50 + chunk // 2] = np.tile([run_len - 1, 1], chunk)[: chunk // 2]
    cb = E.entro_codebook_from_lengths(np.pad(lengths, (0, 256 - lengths.size)).astype(np.uint8), 8)
    stream, off = E.entro_encode(sym, cb, chunk)
    enc = B.EncodedTensor(stream, off, n, chunk, cb, B.QParams(np.float32(0.25), 7, 8, E.ENTRO_ASYMMETRIC), 1, n)
    if sub:
        enc.sub_symbols, enc.sub_bits = sub, E.entro_sub_index(sym, cb, chunk, sub)
    assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8), sym)
    assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8, batch=True), sym)
    assert np.array_equal(_gpu_dequant(enc, E.ENTRO_BF16), oracle.dequant_bf16(sym, 0.25, 7))


@pytest.mark.parametrize("out_type,dtype,waves", [(E.ENTRO_U8, torch.uint8, 14), (E.ENTRO_F32, torch.float32, 16), (E.ENTRO_BF16, torch.bfloat16, 16)])
def test_the_line_between_shared_segments_and_a_lane_each(out_type, dtype, waves):
    # three sixteenths of the lanes that the device holds for this output, and one segment more; peaked data, whose lookups answer
    # many codes, so that the launch's estimated time does not draw the line before
    line = torch.cuda.get_device_properties(0).multi_processor_count * 64 * waves * 3 // 16
    gen = torch.Generator(device=DEV)
    gen.manual_seed(waves)
    op = E.ENTRO_OP_DECODE if out_type == E.ENTRO_U8 else E.ENTRO_OP_DEQUANT
    for segments in (line, line + 1):
        w = torch.randn(segments * 512, device=DEV, generator=gen).pow_(3)
        d, q = E.compress_on_device(w, 8, E.ENTRO_ASYMMETRIC, 512, return_q=True)
        ref = q if out_type == E.ENTRO_U8 else ((q.to(torch.float32) - d.enc.qp.zero_point) * float(d.enc.qp.scale)).to(dtype)
        y = torch.zeros(q.numel(), dtype=dtype, device=DEV)
        t = d.ctensor(y)
        ws = torch.zeros(E.entro_workspace_bytes([t], op), dtype=torch.uint8, device=DEV)
        plan = E.entro_plan_init([t], op, out_type, ws)
        assert (plan.shared_wave_bytes > 0) == (segments == line)
        E.entro_plan_run(plan)
        assert torch.equal(y, ref)
        y.zero_()
        (E.entro_decode if op == E.ENTRO_OP_DECODE else E.entro_decode_dequant)(t, out_type)
        assert torch.equal(y, ref)


# segments longer than lanes share in LDS: 8 to 64 lanes look for their starts in each (find_start)
SEARCHED = [(8, 16384, 70), (8, 12288, 300), (8, 65536, 5), (8, 8704, 9), (8, 1 << 20, 1), (4, 16384, 70), (4, 12288, 9), (4, 65536, 5), (4, 1 << 20, 1)]


@pytest.mark.parametrize("bits,chunk,segments", SEARCHED)
@pytest.mark.parametrize("fraction,every", [(0.0, 1), (0.5, 3), (0.97, 2)])
def test_long_segments_without_entry_points_every_output(bits, chunk, segments, fraction, every):
    # bell-shaped symbols, and runs on which the wavefronts that hold them give the search up
    for last in (0, 1, 63, chunk // 3 + 1, chunk - 1):
        if chunk == 1 << 20 and last not in (0, chunk // 3 + 1):
            continue
        sym = _with_runs(bits, chunk, segments, last, fraction, every, last % 7)
        sym[sym.size // 2], sym[-1] = 0, (1 << bits) - 1
        enc = _oracle_encoded(sym, bits, chunk, 1, sym.size, 0.25, 7)
        assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8), sym)
        assert np.array_equal(_gpu_dequant(enc, E.ENTRO_F32), oracle.dequant_f32(sym, 0.25, 7))
        assert np.array_equal(_gpu_dequant(enc, E.ENTRO_BF16), oracle.dequant_bf16(sym, 0.25, 7))
        if bits == 4:
            assert np.array_equal(_gpu_decode(enc, E.ENTRO_U4_PACKED), oracle.pack_u4(sym))


@pytest.mark.parametrize("bits,chunk,segments", SEARCHED)
def test_long_segments_whose_offsets_do_not_fit(bits, chunk, segments):
    sym = _with_runs(bits, chunk, segments, chunk // 2 + 3, 0.0, 1, 1)
    enc = _oracle_encoded(sym, bits, chunk, 1, sym.size, 0.25, 7)
    true = enc.offsets.copy()
    for end in (true[-1] - 300, true[-2], true[-2] - 5, np.uint64(0), true[-1] + 900, np.uint64(1) << np.uint64(63)):
        enc.offsets = true.copy()
        enc.offsets[-1] = end
        assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8), sym)
        assert np.array_equal(_gpu_dequant(enc, E.ENTRO_BF16), oracle.dequant_bf16(sym, 0.25, 7))
    k = segments // 2
    for shift in (-37, 41) if k else ():                       # a segment begins inside a neighbour: as the oracle decodes it
        enc.offsets = true.copy()
        enc.offsets[k] = np.uint64(int(true[k]) + shift)
        ref = oracle.decode_chunks(enc.stream, enc.offsets, sym.size, chunk, enc.cb.lengths(), enc.cb.codes(), k, 1, sym.copy())
        assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8), ref)


def test_dense_segments_of_8192_are_searched():
    # where the search for starts is the faster of the two, though the segments fit LDS: 4096 of them at 7.5 bits a symbol
    gen = torch.Generator(device=DEV)
    gen.manual_seed(5)
    w = torch.randn(4096 * 8192 - 1000, device=DEV, generator=gen).clamp_(-3.0, 3.0)
    d, q = E.compress_on_device(w, 8, E.ENTRO_ASYMMETRIC, 8192, return_q=True)
    out = torch.zeros(q.numel(), dtype=torch.uint8, device=DEV)
    E.entro_decode(d.ctensor(out), E.ENTRO_U8)
    assert torch.equal(out, q)
    for out_type, dtype in ((E.ENTRO_F32, torch.float32), (E.ENTRO_BF16, torch.bfloat16)):
        y = torch.zeros(q.numel(), dtype=dtype, device=DEV)
        E.entro_decode_dequant(d.ctensor(y), out_type)
        assert torch.equal(y, ((q.to(torch.float32) - d.enc.qp.zero_point) * float(d.enc.qp.scale)).to(dtype))


@pytest.mark.parametrize("bits,chunk", [(8, 4096), (8, 512), (4, 4096)])
def test_segments_without_entry_points_whose_offsets_do_not_fit(bits, chunk):
    # a segment starts where the table says and holds the symbols that it holds, wherever the table puts its end: as the oracle
    # decodes it
    sym = _with_runs(bits, chunk, 5, chunk // 2 + 3, 0.5, 64, 1)
    enc = _oracle_encoded(sym, bits, chunk, 1, sym.size, 0.25, 7)
    true = enc.offsets.copy()
    for end in (true[-1] - 300, true[-2], true[-2] - 5, np.uint64(0), true[-1] + 900, np.uint64(1) << np.uint64(63)):
        enc.offsets = true.copy()
        enc.offsets[-1] = end
        for batch in (False, True):
            assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8, batch), sym)
            assert np.array_equal(_gpu_dequant(enc, E.ENTRO_BF16, batch), oracle.dequant_bf16(sym, 0.25, 7))
    for shift in (-37, 41):                                    # segment 2 begins inside a neighbour: as one lane decodes it
        enc.offsets = true.copy()
        enc.offsets[2] = np.uint64(int(true[2]) + shift)
        ref = oracle.decode_chunks(enc.stream, enc.offsets, sym.size, chunk, enc.cb.lengths(), enc.cb.codes(), 2, 1, sym.copy())
        for batch in (False, True):
            assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8, batch), ref)


def _times_us(calls, inner=5):
    """Times of the calls, taken in turn."""
    times = [[] for _ in calls]
    for f in calls:
        f()
    for _ in range(12):
        for f, t in zip(calls, times):
            a, b = torch.cuda.Event(True), torch.cuda.Event(True)
            a.record()
            for _ in range(inner):
                f()
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b) * 1000 / inner)
    return [float(np.median(t)) for t in times]


# Codes whose lengths have a common divisor: reading from a wrong bit does not fall into step, so lanes never share a segment.
EVEN_LENGTHS = {8: [2, 2, 2, 4, 4, 4, 6, 6, 6, 6], 4: [2, 2, 2, 4, 4, 4, 4]}


def _out_of_step(bits, chunk, n, rows=1, cols=0, sub=0):
    """n symbols under such a code."""
    lengths = np.array(EVEN_LENGTHS[bits])
    sym = np.random.default_rng(n).choice(lengths.size, n, p=0.5 ** lengths).astype(np.uint8)
    cb = E.entro_codebook_from_lengths(np.pad(lengths, (0, (1 << bits) - lengths.size)).astype(np.uint8), bits)
    stream, off = E.entro_encode(sym, cb, chunk)
    enc = B.EncodedTensor(stream, off, n, chunk, cb, B.QParams(np.float32(0.25), 7, bits, E.ENTRO_ASYMMETRIC), rows, cols or n)
    if sub:
        enc.sub_symbols, enc.sub_bits = sub, E.entro_sub_index(sym, cb, chunk, sub)
    return enc, sym


def _single_and_lane_per_segment_us(sym, bits, chunk, out):
    """Times of the call on one tensor without entry points, and of a prepared launch over as many segments of as many symbols
    under a code that does not fall into step: it decodes a segment with a lane, and finds its tables built."""
    cb = E.entro_build_codebook(sym, bits)
    stream, off = E.entro_encode(sym, cb, chunk)
    enc = B.EncodedTensor(stream, off, sym.size, chunk, cb, B.QParams(np.float32(0.25), 7, bits, E.ENTRO_ASYMMETRIC), 1, sym.size)
    op = E.ENTRO_OP_DEQUANT if out == E.ENTRO_BF16 else E.ENTRO_OP_DECODE
    y = torch.zeros(sym.size, dtype=torch.bfloat16 if out == E.ENTRO_BF16 else torch.uint8, device=DEV)
    dt, lane = E.to_device(enc, DEV), E.to_device(_out_of_step(bits, chunk, sym.size)[0], DEV)
    t, tl = dt.ctensor(y), lane.ctensor(y)
    ws = torch.zeros(E.entro_workspace_bytes([tl], op), dtype=torch.uint8, device=DEV)
    plan = E.entro_plan_init([tl], op, out, ws)
    assert plan.shared_wave_bytes == 0
    call = E.entro_decode_dequant if out == E.ENTRO_BF16 else E.entro_decode
    return _times_us([lambda: call(t, out), lambda: E.entro_plan_run(plan)])


@pytest.mark.parametrize("bits,chunk,out", [(8, 4096, E.ENTRO_BF16), (8, 2048, E.ENTRO_U8), (4, 4096, E.ENTRO_U4_PACKED)])
def test_segments_without_entry_points_are_cut(bits, chunk, out):
    # bell-shaped data in few segments
    sym = _with_runs(bits, chunk, (1 << 23) // chunk, 0, 0.0, 1, 3)
    single, lane = _single_and_lane_per_segment_us(sym, bits, chunk, out)
    assert single <= 0.85 * lane, (single, lane)


@pytest.mark.parametrize("bits,chunk,out,most", [(8, 1024, E.ENTRO_BF16, 1.5), (4, 4096, E.ENTRO_U4_PACKED, 1.9)])
def test_runs_cost_little_more_than_a_lane_per_segment(bits, chunk, out, most):
    """Data that does not fall into step takes rounds until the lanes agree: so many times a launch that decodes a segment with
    a lane, at the most."""
    segments = (1 << 24) // chunk if chunk > 1024 else 1 << 15
    single, lane = _single_and_lane_per_segment_us(_with_runs(bits, chunk, segments, 0, 0.9, 20, 3), bits, chunk, out)
    assert single <= most * lane, (single, lane)


@pytest.mark.parametrize("bits,out,most", [(8, E.ENTRO_BF16, 0.75), (4, E.ENTRO_U4_PACKED, 1.15)])
def test_runs_in_every_segment_are_counted_once_a_start(bits, out, most):
    """A run in each of 4096 segments of 8192 symbols: 0.55 and 0.91 of a lane per segment's time; 0.97 and 1.39 where every
    round counts a lane's stretch again."""
    sym = _with_runs(bits, 8192, 4096, 0, 0.9, 1, 3)
    single, lane = _single_and_lane_per_segment_us(sym, bits, 8192, out)
    assert single <= most * lane, (single, lane)


@pytest.mark.parametrize("bits,out", [(8, E.ENTRO_BF16), (8, E.ENTRO_U8), (4, E.ENTRO_U4_PACKED)])
def test_prepared_decoding_without_entry_points_shares_segments(bits, out):
    # 4096 segments of 4096 symbols: 0.31, 0.29 and 0.41 of a lane per segment's time
    sym = _with_runs(bits, 4096, 4096, 0, 0.0, 1, 3)
    encs = [_oracle_encoded(sym, bits, 4096, 1, sym.size, 0.25, 7), _out_of_step(bits, 4096, sym.size)[0]]
    op = E.ENTRO_OP_DEQUANT if out == E.ENTRO_BF16 else E.ENTRO_OP_DECODE
    y = torch.zeros(sym.size, dtype=torch.bfloat16 if out == E.ENTRO_BF16 else torch.uint8, device=DEV)
    dts, plans = [E.to_device(e, DEV) for e in encs], []
    ws = [torch.zeros(E.entro_workspace_bytes([d.ctensor(y)], op), dtype=torch.uint8, device=DEV) for d in dts]
    for d, w in zip(dts, ws):
        plans.append(E.entro_plan_init([d.ctensor(y)], op, out, w))
    assert [p.shared_wave_bytes > 0 for p in plans] == [True, False]
    us = _times_us([lambda p=p: E.entro_plan_run(p) for p in plans])
    assert us[0] <= 0.6 * us[1], us
    E.entro_plan_run(plans[0])
    if out == E.ENTRO_BF16:
        assert np.array_equal(y.view(torch.int16).cpu().numpy().view(np.uint16), oracle.dequant_bf16(sym, 0.25, 7))
    else:
        assert np.array_equal(y.cpu().numpy()[: sym.size * bits // 8], sym if bits == 8 else oracle.pack_u4(sym))


@pytest.mark.parametrize("sub,shared", [(512, True), (256, False)])
def test_products_of_4bit_rows_in_pieces(sub, shared):
    # without places (_plan_of).  16384 pieces, rows of eight of them: shared in pieces of 512 (15.7 us, 25.3 with a lane each), not of 256 (17.3, and 14.9)
    rows, cols = 2048, 8 * sub
    enc, sym = _out_of_step(4, 16 * sub, rows * cols, rows, cols, sub)
    rng = np.random.default_rng(sub)
    bell = np.clip(np.rint(rng.laplace(size=rows * cols) * 0.7 + 7), 0, 15).astype(np.uint8)
    x = synth.make_x_bf16(9, sub, cols)
    xd = torch.from_numpy(x.view(np.int16)).to(DEV).view(torch.bfloat16)
    us, plans = [], []
    for e, s in ((_oracle_encoded(bell, 4, 16 * sub, rows, cols, 0.25, 7, sub), bell), (enc, sym)):
        dt, y = E.to_device(e, DEV), torch.zeros(rows, dtype=torch.float32, device=DEV)
        plan, ws = _plan_of([dt.ctensor(y, xd)], E.ENTRO_F32, places=False)
        plans.append(plan)
        us.append(_times_us([lambda: E.entro_plan_run(plan)], 20)[0])
        y_ref, _ = oracle.gemv(s, rows, cols, 0.25, 7, x)
        _assert_gemv_close(y.cpu().numpy().astype(np.float64), y_ref)
    assert [p.shared_wave_bytes > 0 for p in plans] == [shared, False]
    assert not shared or us[0] <= 0.85 * us[1], us


def test_twice_the_segments_take_twice_the_time():
    # 28672 segments of 8192 symbols fit a wavefront's LDS nine or ten to a workgroup and are still shared, or searched: 2.0 times
    # the time of half of them (4.5 where they got a lane each)
    us, calls = [], []
    for segments in (14336, 28672):
        gen = torch.Generator(device=DEV)
        gen.manual_seed(segments)
        d, q = E.compress_on_device(torch.randn(segments * 8192, device=DEV, generator=gen), 8, E.ENTRO_ASYMMETRIC, 8192, return_q=True)
        out = torch.zeros(q.numel(), dtype=torch.uint8, device=DEV)
        t = d.ctensor(out)
        E.entro_decode(t, E.ENTRO_U8)
        assert torch.equal(out, q)
        us.append(_times_us([lambda: E.entro_decode(t, E.ENTRO_U8)])[0])
    assert us[1] <= 2.6 * us[0], us


@pytest.mark.parametrize("bits,most,chunk,segments,shared", [(8, 3.0, 512, 40960, False), (8, 3.0, 512, 14336, True), (4, 9.0, 1024, 40960, False),
                                                             (4, 9.0, 1024, 24576, True)])
def test_products_share_pieces_only_where_that_is_not_slower(bits, most, chunk, segments, shared):
    """Products without places (_plan_of).  The more bits a symbol takes, the more a shared segment costs and the fewer segments are shared.  Of the time of a lane
    per segment: up to 1.26 (a lane each as well, but the yardstick's stream is a third as long as 7.5 bits a symbol make it),
    2.1 where the number of segments alone decides."""
    cols, gen = 1024, torch.Generator(device=DEV)
    gen.manual_seed(segments)
    rows = segments * chunk // cols
    w = torch.randn(rows * cols, device=DEV, generator=gen).clamp_(-most, most)
    d, q = E.compress_on_device(w, bits, E.ENTRO_ASYMMETRIC, chunk, rows=rows, cols=cols, return_q=True)
    x = torch.randn(cols, device=DEV, generator=gen).to(torch.bfloat16)
    lane, plans, ws = E.to_device(_out_of_step(bits, chunk, rows * cols, rows, cols)[0], DEV), [], []
    ys = [torch.zeros(rows, dtype=torch.float32, device=DEV) for _ in range(2)]
    for dt, y in zip((d, lane), ys):
        plan, room = _plan_of([dt.ctensor(y, x)], E.ENTRO_F32, places=False)
        plans.append(plan)
        ws.append(room)
    assert [p.shared_wave_bytes > 0 for p in plans] == [shared, False]
    us = _times_us([lambda p=p: E.entro_plan_run(p) for p in plans])
    terms = (q.view(rows, cols).to(torch.float32) - d.enc.qp.zero_point).double() * float(d.enc.qp.scale) * x.double()
    # fp32 sums of exact products: at most cols roundings of half an ulp, relative to the terms' magnitudes
    assert bool(((ys[0].double() - terms.sum(1)).abs() <= (cols + 2) * 2.0 ** -24 * terms.abs().sum(1)).all())
    assert us[0] <= 1.45 * us[1], us


@pytest.mark.parametrize("lengths", [
    list(range(1, 15)) + [15, 15],                 # the deepest complete code over 16 symbols
    [1, 3, 3, 4, 4, 5, 5, 6, 6, 7, 7, 8, 8, 8, 8, 0],   # complete over 15 symbols; codes up to 8 bits
    [7, 7, 7, 7, 7, 7, 7, 7, 8, 8, 8, 8, 8, 8, 8, 8],   # incomplete: pairs of 14..16 bits straddle the table width
])
def test_4bit_packed_pairs_that_the_table_does_not_hold(lengths):
    # packed 4-bit output decodes two symbols per lookup where both codes fit into the table index;
    # here many pairs do not (symbols drawn uniformly, so long codes are as common as short ones)
    ln = np.zeros(16, np.uint8)
    ln[:] = lengths
    rng = np.random.default_rng(sum(lengths))
    used = int(np.count_nonzero(ln))
    sym = rng.integers(0, used, 96 * 1024 + 301).astype(np.uint8)
    sym[: 40 * 1024] = np.minimum(rng.geometric(0.5, 40 * 1024) - 1, used - 1)   # and a stretch of mostly short ones
    code = oracle.canonical_codes(ln)
    for chunk in (256, 4096, 1002):
        stream, off = oracle.encode(sym, ln, code, chunk)
        cb = E.entro_codebook_from_lengths(ln, 4)
        enc = B.EncodedTensor(stream, off, sym.size, chunk, cb, B.QParams(1.0, 0, 4, 1))
        assert np.array_equal(_gpu_decode(enc, E.ENTRO_U4_PACKED), oracle.pack_u4(sym)), chunk
        assert np.array_equal(_gpu_decode(enc, E.ENTRO_U4_PACKED, batch=True), oracle.pack_u4(sym)), chunk
        assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8), sym), chunk


@pytest.mark.parametrize("max_len", [11, 14, 16])
def test_length_limited_codebooks_decode_like_any_other(max_len):
    # codes capped below, at and above the first-level table's width; lengths from the oracle's
    # minimisation, stream from the oracle's encoder, decoded on the GPU and by the oracle's tree walk
    spec = synth.config_tensors(4)[1]                          # k: 1024 x 4096, the longest codes of the set
    w = synth.make_tensor(spec)
    q, s, z = oracle.quantize(w, 8, oracle.ASYMMETRIC)
    cnt = oracle.histogram(q, 8)
    ln, cost = oracle.limited_lengths(cnt, max_len)
    assert ln.max() <= max_len and oracle.huffman_lengths(cnt).max() > 16
    code = oracle.canonical_codes(ln)
    stream, off = oracle.encode(q, ln, code, 4096)
    assert int(off[-1]) == cost
    cb = E.entro_codebook_from_lengths(ln, 8)
    enc = B.EncodedTensor(stream, off, q.size, 4096, cb, B.QParams(np.float32(s), int(z), 8, E.ENTRO_ASYMMETRIC))
    assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8, batch=True), q)
    assert np.array_equal(oracle.decode(stream, off, q.size, 4096, ln, code), q)
    assert _bf16_ulp_diff(_gpu_dequant(enc, E.ENTRO_BF16), oracle.dequant_bf16(q, s, z)).max() <= 1
    # the library's own limited codebook costs the same and decodes the same
    enc2 = E.encode_tensor(w, 8, E.ENTRO_ASYMMETRIC, 4096, max_len=max_len)
    assert enc2.cb.max_len <= max_len and enc2.total_bits == cost
    assert np.array_equal(_gpu_decode(enc2, E.ENTRO_U8), q)


def test_phi3_shaped_4bit_packed():
    spec = synth.config_tensors(3)[1]                          # o: 3072 x 3072, Laplace, 4-bit
    w = synth.make_tensor(spec)
    q, s, z = oracle.quantize(w, 4, oracle.ASYMMETRIC)
    enc = _oracle_encoded(q, 4, 8192, s=s, z=z)
    assert np.array_equal(_gpu_decode(enc, E.ENTRO_U4_PACKED, batch=True), oracle.pack_u4(q))
    assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8), q)
    # the byte, fp32 and bf16 outputs of an all-4-bit launch also decode two symbols per lookup
    assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8, batch=True), q)
    f = _gpu_dequant(enc, E.ENTRO_F32, batch=True)
    assert np.array_equal(f.view(np.uint32), oracle.dequant_f32(q, s, z).view(np.uint32))
    b = _gpu_dequant(enc, E.ENTRO_BF16)
    assert _bf16_ulp_diff(b, oracle.dequant_bf16(q, s, z)).max() <= 1


def test_4bit_and_8bit_tensors_in_one_launch():
    # a launch with both alphabets cannot use the two-codes-per-entry tables: every tensor, the 4-bit
    # ones included, goes through the single-code tables
    rng = np.random.default_rng(48)
    encs, refs = [], []
    for bits, n in ((4, 300 * 1024 + 5), (8, 200 * 1024), (4, 64 * 1024)):
        sym = np.minimum(rng.geometric(0.35, n) - 1, (1 << bits) - 1).astype(np.uint8)
        encs.append(_oracle_encoded(sym, bits, 1024, s=np.float32(0.05), z=2))
        refs.append(sym)
    dts = [E.to_device(e, DEV) for e in encs]
    outs = [torch.zeros(e.n, dtype=torch.bfloat16, device=DEV) for e in encs]
    ts = [d.ctensor(o) for d, o in zip(dts, outs)]
    ws = torch.zeros(E.entro_workspace_bytes(ts, E.ENTRO_OP_DEQUANT), dtype=torch.uint8, device=DEV)
    plan = E.entro_plan_init(ts, E.ENTRO_OP_DEQUANT, E.ENTRO_BF16, ws)
    assert plan.pair_tables == 0
    E.entro_plan_run(plan)
    torch.cuda.synchronize()
    for e, o, r in zip(encs, outs, refs):
        got = o.view(torch.int16).cpu().numpy().view(np.uint16)
        assert _bf16_ulp_diff(got, oracle.dequant_bf16(r, e.qp.scale, e.qp.zero_point)).max() <= 1
    only4 = [ts[0], ts[2]]
    plan4 = E.entro_plan_init(only4, E.ENTRO_OP_DEQUANT, E.ENTRO_BF16, ws)
    assert plan4.pair_tables == 1


# ----------------------------------------------------------------------- dequant
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("batch", [False, True])
def test_dequant_fp32_bit_exact_and_bf16_within_one_ulp(bits, batch):
    spec = synth.TensorSpec(4, 0, 1, "k", 1024, 4096, "student_t", 5.0, 0.02, 0.0, bits, 1, 4242 + bits)
    w = synth.make_tensor(spec)
    q, s, z = oracle.quantize(w, bits, oracle.ASYMMETRIC)
    enc = _oracle_encoded(q, bits, 4096, s=s, z=z)
    f = _gpu_dequant(enc, E.ENTRO_F32, batch)
    assert np.array_equal(f.view(np.uint32), oracle.dequant_f32(q, s, z).view(np.uint32))
    b = _gpu_dequant(enc, E.ENTRO_BF16, batch)
    assert _bf16_ulp_diff(b, oracle.dequant_bf16(q, s, z)).max() <= 1


def test_dequant_ragged_and_unsigned_and_offgrid_zero_point():
    rng = np.random.default_rng(5)
    sym = rng.integers(170, 256, 2048).astype(np.uint8)        # norm-gain-like, one half-full segment
    enc = _oracle_encoded(sym, 8, 4096, s=np.float32(1.2 / 255), z=0)
    assert np.array_equal(_gpu_dequant(enc, E.ENTRO_F32).view(np.uint32),
                          oracle.dequant_f32(sym, enc.qp.scale, 0).view(np.uint32))
    sym = np.minimum(rng.geometric(0.2, 3 * 4096 + 5) - 1, 255).astype(np.uint8)
    for z in (-255, 300, 17):
        enc = _oracle_encoded(sym, 8, 4096, s=np.float32(0.37), z=z)
        assert np.array_equal(_gpu_dequant(enc, E.ENTRO_F32).view(np.uint32),
                              oracle.dequant_f32(sym, enc.qp.scale, z).view(np.uint32))
        assert _bf16_ulp_diff(_gpu_dequant(enc, E.ENTRO_BF16), oracle.dequant_bf16(sym, enc.qp.scale, z)).max() <= 1


# -------------------------------------------------------------------------- gemv
@pytest.mark.parametrize("rows,cols,chunk", [
    (96, 4096, 4096),        # one row per segment
    (40, 14336, 4096),       # a row is 3.5 segments (the `down` projection)
    (300, 2048, 4096),       # two rows per segment
    (77, 300, 4096),         # rows do not divide segments
    (5, 9000, 1024),         # long rows, ragged last segment
    (1, 100, 4096),          # a single short row
    (512, 128, 1024),        # eight whole rows per segment
    (300, 192, 1024),        # five and a third rows per segment
    (160, 3072, 8192),       # the phi3 shapes: two and two thirds rows per segment
    (4096 + 11, 64, 4096),   # the shortest rows the kernel takes: one per block; ragged last segment
    (100, 72, 512),          # a block may hold the end of one row and the start of the next
    (64, 4096, 64),          # the shortest segments: sixty-four per row
    (7, 1000, 4096),         # rows of 125 pieces of eight, segments of four rows and a bit
    (31, 60, 128),           # rows shorter than a block: element by element
])
@pytest.mark.parametrize("batch", [False, True])
def test_gemv_against_fp64_oracle(rows, cols, chunk, batch):
    spec = synth.TensorSpec(4, 0, 0, "g", rows, cols, "student_t", 5.0, 0.02, 0.0, 8, 1, 9000 + rows)
    w = synth.make_tensor(spec)
    q, s, z = oracle.quantize(w, 8, oracle.ASYMMETRIC)
    enc = _oracle_encoded(q, 8, chunk, rows, cols, s, z)
    xb = synth.make_x_bf16(0, rows % 7, cols)
    y_ref, _ = oracle.gemv(q, rows, cols, s, z, xb)
    _assert_gemv_close(_gpu_gemv(enc, xb, E.ENTRO_F32, batch), y_ref)
    y_bf = _gpu_gemv(enc, xb, E.ENTRO_BF16, batch)
    assert np.all(np.abs(y_bf - y_ref) <= 2.0 ** -7 * np.abs(y_ref) + 1e-3 * np.sqrt(np.mean(y_ref ** 2)))


@pytest.mark.parametrize("rows,cols,chunk", [
    (160, 3072, 8192),       # phi3 shapes: two and two thirds rows per segment
    (64, 8192, 8192),        # one row per segment
    (96, 4096, 1024),        # four segments per row
    (520, 128, 4096),        # thirty-two rows per segment
    (33, 144, 256),          # rows and blocks out of step
    (50, 200, 512),          # cols a multiple of 8 but not of 16
    (300, 64, 256),          # the shortest rows the kernel takes: one per half block
    (90, 72, 128),           # a half block may hold the end of one row and the start of the next
    (40, 100, 256),          # cols not a multiple of 8: element by element, with the pair tables
    (3, 8192, 256),          # a few long rows of many segments
])
@pytest.mark.parametrize("batch", [False, True])
def test_gemv_4bit_two_symbols_per_lookup(rows, cols, chunk, batch):
    rng = np.random.default_rng(rows + cols)
    sym = np.minimum(rng.geometric(0.45, rows * cols) - 1, 15).astype(np.uint8)
    sym[rng.random(sym.size) < 0.01] = 15                      # some long codes
    enc = _oracle_encoded(sym, 4, chunk, rows=rows, cols=cols, s=np.float32(0.07), z=6)
    xb = synth.make_x_bf16(1, rows % 4, cols)
    y_ref, _ = oracle.gemv(sym, rows, cols, enc.qp.scale, 6, xb)
    _assert_gemv_close(_gpu_gemv(enc, xb, E.ENTRO_F32, batch), y_ref)
    _assert_gemv_close(_gpu_gemv(enc, xb, E.ENTRO_BF16, batch), y_ref, tol=5e-3)   # y itself rounded to bf16: half an ulp, up to 2^-8 of the value, on top of the 1e-3


def test_gemv_unit_vector_picks_a_column_exactly():
    rows, cols = 64, 4096
    rng = np.random.default_rng(1)
    q = rng.integers(0, 256, rows * cols).astype(np.uint8)
    s, z = np.float32(0.0123), 131
    enc = _oracle_encoded(q, 8, 4096, rows, cols, s, z)
    e = np.zeros(cols, np.float32)
    e[1234] = 1.0
    y = _gpu_gemv(enc, synth.f32_to_bf16_bits(e), E.ENTRO_F32)
    col = oracle.dequant_f32(q, s, z).reshape(rows, cols)[:, 1234]
    assert np.array_equal(y.astype(np.float32), col)


# ------------------------------------------------------------- batched launches
# ------------------------------------------------- entry points inside the segments
@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("bits,chunk,sub,n", [(8, 4096, 256, 300 * 4096), (8, 4096, 256, 70 * 4096 + 1000), (8, 4096, 1024, 9 * 4096 + 5),
                                              (8, 2048, 128, 64 * 2048 + 130), (8, 1024, 64, 33 * 1024 + 63), (4, 8192, 512, 20 * 8192 + 700),
                                              (8, 4096, 4096, 3 * 4096 + 17), (8, 1000, 250, 17 * 1000 + 3)])
def test_entry_points_inside_segments_every_output(bits, chunk, sub, n, batch):
    """A lane decodes a piece of a segment from its entry point: the outputs are those of the oracle's plain decode."""
    rng = np.random.default_rng(n + sub)
    sym = np.clip(np.rint(rng.standard_t(4, n) * (6 if bits == 8 else 0.8) + (1 << (bits - 1))), 0, (1 << bits) - 1).astype(np.uint8)
    enc = _oracle_encoded(sym, bits, chunk, s=0.0173, z=(1 << (bits - 1)) + 3, sub=sub)
    q = oracle.decode(enc.stream, enc.offsets, n, chunk, enc.cb.lengths(), enc.cb.codes())
    assert np.array_equal(q, sym)
    assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8, batch), q)
    if bits == 4:
        assert np.array_equal(_gpu_decode(enc, E.ENTRO_U4_PACKED, batch), oracle.pack_u4(q))
    w32 = _gpu_dequant(enc, E.ENTRO_F32, batch)
    assert np.array_equal(w32.view(np.uint32), oracle.dequant_f32(q, enc.qp.scale, enc.qp.zero_point).view(np.uint32))
    assert _bf16_ulp_diff(_gpu_dequant(enc, E.ENTRO_BF16, batch), oracle.dequant_bf16(q, enc.qp.scale, enc.qp.zero_point)).max() <= 1


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("rows,cols,chunk,sub", [(128, 4096, 4096, 256), (96, 14336, 4096, 256), (300, 1024, 4096, 512), (65, 1536, 2048, 128),
                                                 (40, 200, 1024, 64), (520, 128, 4096, 1024), (67, 8192, 2048, 128),
                                                 (200, 2048, 2048, 128)])
def test_gemv_with_entry_points_inside_segments(rows, cols, chunk, sub, batch):
    rng = np.random.default_rng(rows * cols + sub)
    sym = np.clip(np.rint(rng.standard_t(5, rows * cols) * 6 + 128), 0, 255).astype(np.uint8)
    enc = _oracle_encoded(sym, 8, chunk, rows, cols, s=0.011, z=125, sub=sub)
    xb = synth.f32_to_bf16_bits(rng.standard_normal(cols).astype(np.float32))
    y_ref, _ = oracle.gemv(sym, rows, cols, enc.qp.scale, enc.qp.zero_point, xb)
    _assert_gemv_close(_gpu_gemv(enc, xb, E.ENTRO_F32, batch), y_ref)
    plain = _oracle_encoded(sym, 8, chunk, rows, cols, s=0.011, z=125)
    # against the same product with one lane per segment: the same sums in another order
    assert np.allclose(_gpu_gemv(enc, xb, E.ENTRO_F32, batch), _gpu_gemv(plain, xb, E.ENTRO_F32, batch), rtol=1e-4, atol=1e-4)


def test_large_launch_merges_pieces_into_coarser_lanes():
    """A launch with more pieces than the chip has lanes lets a lane take 2^k pieces (the coarsest cut that still
    gives every lane slot a lane): 40 M symbols with entry points every 64 symbols in segments of 1024."""
    n, chunk, sub = 40 * 1024 * 1024, 1024, 64
    rng = np.random.default_rng(5)
    sym = np.clip(np.rint(rng.standard_t(4, n) * 5 + 128), 0, 255).astype(np.uint8)
    enc = _oracle_encoded(sym, 8, chunk, s=0.02, z=131, sub=sub)
    assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8, True), sym)
    assert _bf16_ulp_diff(_gpu_dequant(enc, E.ENTRO_BF16, False), oracle.dequant_bf16(sym, enc.qp.scale, enc.qp.zero_point)).max() <= 1


def test_last_round_of_every_stretch_is_drawn_with_finer_lanes_every_output():
    """A launch of several rounds per workgroup over tensors with entry points inside their segments: the last
    round of every stretch is decoded by lanes that take pieces instead of segments (and as before for the
    tensor that has no entry points); every output element, guard bytes between the outputs."""
    rng = np.random.default_rng(61)
    chunk = 256
    shapes = [(2500, 64), (1125, 64), (2125, 128), (37, 0), (750, 32)]     # (units of 64 segments, entry-point spacing)
    encs, refs = [], []
    for i, (units, sub) in enumerate(shapes):
        n = units * 64 * chunk - (0 if i != 2 else 21 * chunk + 5)          # tensor 2 ends inside a segment
        sym = np.minimum(rng.geometric(0.12 + 0.05 * i, n) - 1, 255).astype(np.uint8)
        encs.append(_oracle_encoded(sym, 8, chunk, s=np.float32(0.01), z=2 + i, sub=sub))
        refs.append(sym)
    dts = [E.to_device(e, DEV) for e in encs]
    for op, out_type, dtype, width in ((E.ENTRO_OP_DECODE, E.ENTRO_U8, torch.uint8, 1),
                                       (E.ENTRO_OP_DEQUANT, E.ENTRO_BF16, torch.bfloat16, 2),
                                       (E.ENTRO_OP_DEQUANT, E.ENTRO_F32, torch.float32, 4)):
        guard = 64 // width
        sizes = [(e.n + guard - 1) // guard * guard + guard for e in encs]   # every output 64-byte aligned, a guard behind it
        buf = torch.full((sum(sizes),), 7, dtype=dtype, device=DEV)
        outs, pos = [], 0
        for e, sz in zip(encs, sizes):
            outs.append(buf[pos:pos + e.n])
            pos += sz
        ts = [d.ctensor(o) for d, o in zip(dts, outs)]
        ws = torch.zeros(E.entro_workspace_bytes(ts, op), dtype=torch.uint8, device=DEV)
        plan = E.entro_plan_init(ts, op, out_type, ws)
        E.entro_plan_run(plan)
        torch.cuda.synchronize()
        pos = 0
        for e, r, o, sz in zip(encs, refs, outs, sizes):
            if dtype == torch.uint8:
                assert np.array_equal(o.cpu().numpy(), r)
            elif dtype == torch.bfloat16:
                assert np.array_equal(o.view(torch.int16).cpu().numpy().view(np.uint16),
                                      oracle.dequant_bf16(r, e.qp.scale, e.qp.zero_point))
            else:
                assert np.array_equal(o.view(torch.int32).cpu().numpy().view(np.uint32),
                                      oracle.dequant_f32(r, e.qp.scale, e.qp.zero_point).view(np.uint32))
            assert bool((buf[pos + e.n:pos + sz] == 7).all()), "a guard element was written"
            pos += sz


def test_staged_plan_init_does_not_block_and_batch_calls_return_before_their_kernel_ends():
    from paper_2505_02380_amd.workload import prepare_config
    encs = prepare_config(4, layers=8)
    dts = [E.to_device(e, DEV) for e in encs]
    outs = [torch.zeros(e.n, dtype=torch.bfloat16, device=DEV) for e in encs]
    ts = [d.ctensor(o) for d, o in zip(dts, outs)]
    ws = torch.zeros(E.entro_workspace_bytes(ts, E.ENTRO_OP_DEQUANT), dtype=torch.uint8, device=DEV)
    staging = torch.zeros(E.entro_plan_staging_bytes(ts, E.ENTRO_OP_DEQUANT), dtype=torch.uint8).pin_memory()
    assert staging.numel() > 0
    torch.cuda.synchronize()
    # something long in front of it on the stream: the staged form must not wait for it
    filler = torch.empty(1 << 30, dtype=torch.uint8, device=DEV)
    for _ in range(8):
        filler.fill_(1)
    busy = torch.cuda.Event()
    busy.record()
    plan = E.entro_plan_init_staged(ts, E.ENTRO_OP_DEQUANT, E.ENTRO_BF16, ws, staging)
    E.entro_plan_run(plan)
    assert not busy.query(), "entro_plan_init_staged or entro_plan_run waited for the stream"
    torch.cuda.synchronize()
    first = [o.clone() for o in outs]
    for o in outs:
        o.zero_()
    # the batch form waits once for the stream (so large a table is copied), then enqueues: it is back before its kernel ends
    done = torch.cuda.Event()
    E.entro_decode_dequant_batch(ts, E.ENTRO_BF16, ws)
    done.record()
    assert not done.query(), "entro_decode_dequant_batch returned only after its kernel had ended"
    torch.cuda.synchronize()
    for a, b in zip(first, outs):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    e = encs[3]
    q = oracle.decode(e.stream, e.offsets, e.n, e.chunk_symbols, e.cb.lengths(), e.cb.codes())
    assert _bf16_ulp_diff(outs[3].view(torch.int16).cpu().numpy().view(np.uint16),
                          oracle.dequant_bf16(q, e.qp.scale, e.qp.zero_point)).max() <= 1


@pytest.mark.parametrize("chunk,sub", [(4096, 256), (4096, 0), (1024, 512)])
@pytest.mark.parametrize("count", [2, 5, 11, 12, 13, 14, 24, 25, 26, 27, 40])
def test_batch_calls_whose_table_travels_as_arguments_and_is_copied(count, chunk, sub):
    """Tensors of unequal sizes, a lane per piece or segment each (codes that do not fall into step), so many that their table takes
    one to three kernels' arguments or more, where it is copied: to the last bit what a prepared launch gives, whose table is copied
    always.  A call whose table travels does not wait for what is in front of it."""
    rng, dts, syms = np.random.default_rng(count), [], []
    shapes = [(301, 4096), (97, 1000), (9, 14336), (1, 64), (40, 1001), (700, 72)]
    for i in range(count):
        rows, cols = shapes[i % 6]
        rows += int(rng.integers(0, 5))
        enc, sym = _out_of_step(8 if i % 5 else 4, chunk, rows * cols, rows, cols, sub)
        dts.append(E.to_device(enc, DEV))
        syms.append(sym)
    small = [i for i, d in enumerate(dts) if d.enc.cols % 8 == 0]          # (activations of whole pieces of eight)
    xs = [torch.from_numpy(synth.make_x_bf16(1, i, d.enc.cols).view(np.int16)).to(DEV).view(torch.bfloat16) for i, d in enumerate(dts)]
    filler = torch.empty(1 << 30, dtype=torch.uint8, device=DEV)
    for op, out, dtype in ((E.ENTRO_OP_DECODE, E.ENTRO_U8, torch.uint8), (E.ENTRO_OP_DEQUANT, E.ENTRO_BF16, torch.bfloat16),
                           (E.ENTRO_OP_DEQUANT, E.ENTRO_F32, torch.float32), (E.ENTRO_OP_GEMV, E.ENTRO_F32, torch.float32)):
        gemv, runs = op == E.ENTRO_OP_GEMV, []
        which = small if gemv else range(count)
        call = {E.ENTRO_OP_DECODE: E.entro_decode_batch, E.ENTRO_OP_DEQUANT: E.entro_decode_dequant_batch, E.ENTRO_OP_GEMV: E.entro_decode_gemv_batch}[op]
        for prepared in (False, True):
            outs = [torch.full((dts[i].enc.rows if gemv else syms[i].size,), 77, dtype=dtype, device=DEV) for i in which]
            ts = [dts[i].ctensor(o, xs[i] if gemv else None) for i, o in zip(which, outs)]
            ws = torch.zeros(E.entro_workspace_bytes(_without_places(ts) if gemv else ts, op), dtype=torch.uint8, device=DEV)
            if prepared:
                plan = E.entro_plan_init(ts, op, out, ws)
                assert plan.shared_wave_bytes == 0 and plan.wide_tables != 2
                E.entro_plan_run(plan)
            else:
                call(ts, out, ws)
                torch.cuda.synchronize()
                for o in outs:
                    o.fill_(78)
                for _ in range(8):
                    filler.fill_(1)
                busy = torch.cuda.Event()
                busy.record()
                call(ts, out, ws)
                assert count > 5 or not busy.query(), "waited for the stream"
            runs.append(outs)
        for a, b, i in zip(*runs, which):
            assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
            if not gemv:
                ref = syms[i] if op == E.ENTRO_OP_DECODE else (oracle.dequant_f32 if out == E.ENTRO_F32 else oracle.dequant_bf16)(syms[i], 0.25, 7)
                got = a.cpu().numpy() if out != E.ENTRO_BF16 else a.view(torch.int16).cpu().numpy().view(np.uint16)
                assert np.array_equal(got, ref)
            else:
                y_ref, _ = oracle.gemv(syms[i], dts[i].enc.rows, dts[i].enc.cols, 0.25, 7, synth.make_x_bf16(1, i, dts[i].enc.cols))
                _assert_gemv_close(a.cpu().numpy().astype(np.float64), y_ref)


def test_many_tensors_in_one_launch():
    rng = np.random.default_rng(12)
    encs, refs = [], []
    for i, (n, chunk) in enumerate([(300000, 4096), (2048, 4096), (4096 * 300 + 1, 4096), (70000, 1000), (5, 4096)]):
        sym = np.minimum(rng.geometric(0.1 + 0.15 * i, n) - 1, 255).astype(np.uint8)
        encs.append(_oracle_encoded(sym, 8, chunk, s=np.float32(0.01 * (i + 1)), z=10 * i))
        refs.append(sym)
    dts = [E.to_device(e, DEV) for e in encs]
    outs = [torch.zeros(e.n, dtype=torch.uint8, device=DEV) for e in encs]
    ts = [d.ctensor(o) for d, o in zip(dts, outs)]
    ws = torch.zeros(E.entro_workspace_bytes(ts, E.ENTRO_OP_DECODE), dtype=torch.uint8, device=DEV)
    plan = E.entro_plan_init(ts, E.ENTRO_OP_DECODE, E.ENTRO_U8, ws)
    for _ in range(2):                                         # a prepared plan can be replayed
        for o in outs:
            o.zero_()
        E.entro_plan_run(plan)
        torch.cuda.synchronize()
        for o, r in zip(outs, refs):
            assert np.array_equal(o.cpu().numpy(), r)
    fouts = [torch.zeros(e.n, dtype=torch.bfloat16, device=DEV) for e in encs]
    ts = [d.ctensor(o) for d, o in zip(dts, fouts)]
    E.entro_decode_dequant_batch(ts, E.ENTRO_BF16, ws)
    torch.cuda.synchronize()
    for e, o, r in zip(encs, fouts, refs):
        got = o.view(torch.int16).cpu().numpy().view(np.uint16)
        assert _bf16_ulp_diff(got, oracle.dequant_bf16(r, e.qp.scale, e.qp.zero_point)).max() <= 1


def test_launch_with_a_few_units_per_work_item():
    # 64-symbol segments make many units (64 segments each) out of little data: ~880 units over the
    # chip's workgroups give work items of a few units, workgroup shares that start and end inside
    # tensors, stretches shorter than a workgroup has wavefronts, and a last unit that is not full
    rng = np.random.default_rng(88)
    chunk, cols = 64, 128
    encs, refs, xs = [], [], []
    for i, units in enumerate((300, 77, 500, 1)):
        n = units * 64 * chunk - (0 if i != 2 else 38 * chunk)          # tensor 2 ends inside a unit
        sym = np.minimum(rng.geometric(0.2 + 0.1 * i, n) - 1, 255).astype(np.uint8)
        encs.append(_oracle_encoded(sym, 8, chunk, rows=n // cols, cols=cols, s=np.float32(0.02), z=3 + i))
        refs.append(sym)
        xs.append(synth.make_x_bf16(9, i, cols))
    dts = [E.to_device(e, DEV) for e in encs]
    outs = [torch.zeros(e.n, dtype=torch.uint8, device=DEV) for e in encs]
    ts = [d.ctensor(o) for d, o in zip(dts, outs)]
    ws = torch.zeros(E.entro_workspace_bytes(ts, E.ENTRO_OP_DECODE), dtype=torch.uint8, device=DEV)
    plan = E.entro_plan_init(ts, E.ENTRO_OP_DECODE, E.ENTRO_U8, ws)
    assert 1 < plan.item_units < 10
    E.entro_plan_run(plan)
    torch.cuda.synchronize()
    for o, r in zip(outs, refs):
        assert np.array_equal(o.cpu().numpy(), r)
    ys = [torch.zeros(e.rows, dtype=torch.float32, device=DEV) for e in encs]
    xd = [torch.from_numpy(x.view(np.int16)).to(DEV).view(torch.bfloat16) for x in xs]
    ts = [d.ctensor(y, x) for d, y, x in zip(dts, ys, xd)]
    wsg = torch.zeros(max(256, E.entro_workspace_bytes(ts, E.ENTRO_OP_GEMV)), dtype=torch.uint8, device=DEV)
    E.entro_decode_gemv_batch(ts, E.ENTRO_F32, wsg)
    torch.cuda.synchronize()
    for e, y, r, x in zip(encs, ys, refs, xs):
        y_ref, _ = oracle.gemv(r, e.rows, cols, e.qp.scale, e.qp.zero_point, x)
        _assert_gemv_close(y.cpu().numpy().astype(np.float64), y_ref)


def test_random_shapes_all_outputs():
    """Seeded sweep over sizes, segment lengths, alphabets and code-length profiles, every output type,
    single and batched: bit-exact integers and fp32, bf16 within 1 ulp, GEMV within 1e-3."""
    # ENTRO_SWEEP_SEED / ENTRO_SWEEP_CASES widen the sweep for a soak run
    rng = np.random.default_rng(int(os.environ.get("ENTRO_SWEEP_SEED", "2025")))
    chunks8 = [1, 64, 128, 192, 256, 1000, 1024, 4096, 8192]
    for case in range(int(os.environ.get("ENTRO_SWEEP_CASES", "150"))):
        bits = 4 if case % 3 == 0 else 8
        A = 1 << bits
        chunk = int(rng.choice(chunks8))
        if bits == 4 and chunk % 2:
            chunk += 1
        n = int(rng.integers(1, 40 * chunk + 2)) if chunk > 64 else int(rng.integers(1, 5000))
        if case % 2:                                             # a matrix shape, for the GEMV below
            cols = int(rng.choice([8192, 4096, 3072, 1024, 192, 72, 64, 40, 7]))
            n = cols * max(1, n // cols)
        kind = case % 4
        if kind == 0:
            sym = np.minimum(rng.geometric(rng.uniform(0.05, 0.7), n) - 1, A - 1)
        elif kind == 1:
            sym = rng.integers(0, A, n)
        elif kind == 2:
            sym = np.where(rng.random(n) < 0.97, rng.integers(0, 3, n), rng.integers(0, A, n))   # rare long codes
        else:
            sym = np.full(n, int(rng.integers(0, A)))
            sym[rng.integers(0, n, max(1, n // 50))] = int(rng.integers(0, A))
        sym = sym.astype(np.uint8)
        z = int(rng.integers(-3, A + 3))
        enc = _oracle_encoded(sym, bits, chunk, s=np.float32(rng.uniform(1e-3, 1.0)), z=z)
        tag = (case, bits, chunk, n, kind)
        batch = bool(case & 1)
        assert np.array_equal(_gpu_decode(enc, E.ENTRO_U8, batch), sym), tag
        if bits == 4:
            assert np.array_equal(_gpu_decode(enc, E.ENTRO_U4_PACKED, not batch), oracle.pack_u4(sym)), tag
        f = _gpu_dequant(enc, E.ENTRO_F32, not batch)
        assert np.array_equal(f.view(np.uint32), oracle.dequant_f32(sym, enc.qp.scale, z).view(np.uint32)), tag
        b = _gpu_dequant(enc, E.ENTRO_BF16, batch)
        assert _bf16_ulp_diff(b, oracle.dequant_bf16(sym, enc.qp.scale, z)).max() <= 1, tag
        # a matrix shape for the same symbols, if n factors conveniently
        for cols in (8192, 4096, 3072, 1024, 192, 72, 64, 40, 7):
            if n % cols == 0:
                rows = n // cols
                encg = _oracle_encoded(sym, bits, chunk, rows=rows, cols=cols, s=enc.qp.scale, z=z)
                xb = synth.make_x_bf16(case, 0, cols)
                y_ref, _ = oracle.gemv(sym, rows, cols, enc.qp.scale, z, xb)
                if np.linalg.norm(y_ref) > 0:
                    _assert_gemv_close(_gpu_gemv(encg, xb, E.ENTRO_F32, batch), y_ref)
                break


def test_mistral_layer_launch_shape_sampled_against_oracle():
    """Four mistral-7B-shaped layers in the batched launch bench.py uses (more work items than the chip
    holds workgroups, so workgroups walk several items and tensors); sampled segments vs the oracle."""
    from paper_2505_02380_amd.workload import prepare_config
    encs = prepare_config(4, layers=4)
    dts = [E.to_device(e, DEV) for e in encs]
    outs = [torch.zeros(e.n, dtype=torch.bfloat16, device=DEV) for e in encs]
    ts = [d.ctensor(o) for d, o in zip(dts, outs)]
    ws = torch.zeros(E.entro_workspace_bytes(ts, E.ENTRO_OP_DEQUANT), dtype=torch.uint8, device=DEV)
    E.entro_decode_dequant_batch(ts, E.ENTRO_BF16, ws)
    torch.cuda.synchronize()
    rng = np.random.default_rng(0)
    for e, o in zip(encs, outs):
        n_chunks = e.offsets.size - 1
        picks = sorted(set([0, n_chunks - 1] + rng.integers(0, n_chunks, 6).tolist()))
        host = o.view(torch.int16).cpu().numpy().view(np.uint16)
        for k in picks:
            q = oracle.decode_chunks(e.stream, e.offsets, e.n, e.chunk_symbols, e.cb.lengths(), e.cb.codes(), k, 1)
            lo, hi = k * e.chunk_symbols, min((k + 1) * e.chunk_symbols, e.n)
            ref = oracle.dequant_bf16(q[lo:hi], e.qp.scale, e.qp.zero_point)
            assert _bf16_ulp_diff(host[lo:hi], ref).max() <= 1, (e.name, k)
    # the same layer through the fused GEMV (7 linears in one launch)
    xs = [torch.from_numpy(synth.make_x_bf16(i // 7, i % 7, e.cols).view(np.int16)).to(DEV).view(torch.bfloat16)
          for i, e in enumerate(encs)]
    ys = [torch.zeros(e.rows, dtype=torch.float32, device=DEV) for e in encs]
    ts = [d.ctensor(y, x) for d, y, x in zip(dts, ys, xs)]
    ws = torch.zeros(E.entro_workspace_bytes(ts, E.ENTRO_OP_GEMV), dtype=torch.uint8, device=DEV)
    E.entro_decode_gemv_batch(ts, E.ENTRO_F32, ws)
    torch.cuda.synchronize()
    for i, (e, y) in enumerate(zip(encs, ys)):
        rows = sorted(set([0, e.rows - 1] + rng.integers(0, e.rows, 4).tolist()))
        yh = y.cpu().numpy().astype(np.float64)
        xb = synth.make_x_bf16(i // 7, i % 7, e.cols)
        sub = np.empty((len(rows), e.cols), np.uint8)
        for j, r in enumerate(rows):
            k0, k1 = (r * e.cols) // e.chunk_symbols, ((r + 1) * e.cols - 1) // e.chunk_symbols
            q = oracle.decode_chunks(e.stream, e.offsets, e.n, e.chunk_symbols, e.cb.lengths(), e.cb.codes(),
                                     k0, k1 - k0 + 1)
            sub[j] = q[r * e.cols:(r + 1) * e.cols]
        y_ref, _ = oracle.gemv(sub, len(rows), e.cols, e.qp.scale, e.qp.zero_point, xb)
        rms = np.sqrt(np.mean(yh ** 2))
        assert np.max(np.abs(yh[rows] - y_ref) / np.maximum(np.abs(y_ref), rms)) <= 1e-3, e.name


def test_prepared_launches_replay_in_a_hip_graph():
    """entro_plan_run only enqueues kernels (no allocation, no copies, no memset), so it can be captured:
    every replay of the graph must give the eager result, with eager work and synchronisation between
    the replays."""
    rng = np.random.default_rng(4242)
    encs, refs_q = [], []
    for rows, cols, chunk in [(96, 4096, 4096), (40, 1024, 4096), (33, 3072, 1024)]:
        sym = np.minimum(rng.geometric(0.3, rows * cols) - 1, 255).astype(np.uint8)
        encs.append(_oracle_encoded(sym, 8, chunk, rows=rows, cols=cols, s=np.float32(0.01), z=3))
        refs_q.append(sym)
    dts = [E.to_device(e, DEV) for e in encs]
    # dequant -> bf16
    outs = [torch.zeros(e.n, dtype=torch.bfloat16, device=DEV) for e in encs]
    ts = [d.ctensor(o) for d, o in zip(dts, outs)]
    ws = torch.zeros(E.entro_workspace_bytes(ts, E.ENTRO_OP_DEQUANT), dtype=torch.uint8, device=DEV)
    plan = E.entro_plan_init(ts, E.ENTRO_OP_DEQUANT, E.ENTRO_BF16, ws)
    # GEMV -> fp32 (the third tensor's rows straddle segments: two kernels per launch)
    xs = [torch.from_numpy(synth.make_x_bf16(7, i, e.cols).view(np.int16)).to(DEV).view(torch.bfloat16) for i, e in enumerate(encs)]
    ys = [torch.zeros(e.rows, dtype=torch.float32, device=DEV) for e in encs]
    dts_g = [E.to_device(e, DEV) for e in encs]
    tg = [d.ctensor(y, x) for d, y, x in zip(dts_g, ys, xs)]
    wsg = torch.zeros(max(256, E.entro_workspace_bytes(tg, E.ENTRO_OP_GEMV)), dtype=torch.uint8, device=DEV)
    plan_g = E.entro_plan_init(tg, E.ENTRO_OP_GEMV, E.ENTRO_F32, wsg)
    torch.cuda.synchronize()
    E.entro_plan_run(plan)
    E.entro_plan_run(plan_g)
    torch.cuda.synchronize()
    eager_o = [o.clone() for o in outs]
    eager_y = [y.clone() for y in ys]
    for e, q, o in zip(encs, refs_q, eager_o):
        assert _bf16_ulp_diff(o.view(torch.int16).cpu().numpy().view(np.uint16),
                              oracle.dequant_bf16(q, e.qp.scale, e.qp.zero_point)).max() <= 1
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            E.entro_plan_run(plan)
            E.entro_plan_run(plan_g)
    torch.cuda.synchronize()
    for rep in range(3):
        for o in outs:
            o.fill_(1.0)                                   # eager work between the replays
        for y in ys:
            y.fill_(-7.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for o, ref in zip(outs, eager_o):
            assert torch.equal(o.view(torch.int16), ref.view(torch.int16)), rep
        for y, ref in zip(ys, eager_y):
            assert torch.equal(y, ref), rep                # the row sums are taken in a fixed order: bit-identical


def test_plain_uint8_gemv_comparison_kernel_matches_the_oracle():
    """bench.py's comparison kernel (its own shared object, not the library): all products in one launch."""
    import bench_kernels
    shapes = [(300, 4096), (7, 14336), (1000, 64), (33, 1040), (1, 16)]
    products, refs = [], []
    for rows, cols in shapes:
        rng = np.random.default_rng(rows)
        q = np.minimum(rng.geometric(0.05, rows * cols) - 1, 255).astype(np.uint8)
        xb = synth.make_x_bf16(2, rows % 5, cols)
        y_ref, _ = oracle.gemv(q, rows, cols, np.float32(0.013), 21, xb)
        y = torch.full((rows + 4,), 9.0, dtype=torch.float32, device=DEV)
        products.append((torch.from_numpy(q).to(DEV), rows, cols, np.float32(0.013), 21,
                         torch.from_numpy(xb.view(np.int16)).to(DEV).view(torch.bfloat16), y))
        refs.append(y_ref)
    bench_kernels.PlainGemv(products, DEV).run()
    torch.cuda.synchronize()
    for (q, rows, cols, s, z, x, y), y_ref in zip(products, refs):
        got = y.cpu().numpy()
        assert np.all(got[rows:] == 9.0)
        _assert_gemv_close(got[:rows].astype(np.float64), y_ref)


@pytest.mark.parametrize("y_type", [E.ENTRO_F32, E.ENTRO_BF16])
def test_few_units_per_workgroup_run_side_by_side(y_type):
    """A prepared launch with a unit for each SIMD of every compute unit takes as long as one with a single unit per
    compute unit, whatever the order in which the wavefronts of a workgroup get there: 1.05 times as long (1.21 where
    two wavefronts of a SIMD may take units while another SIMD has none)."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    cols, sub, us = 8192, 512, []
    for units in (1, 4):
        rows = units * cus * 64 * sub // cols
        enc, sym = _out_of_step(4, 16 * sub, rows * cols, rows, cols, sub)   # (a code that lanes do not share pieces of)
        dt = E.to_device(enc, DEV)
        x = torch.from_numpy(synth.make_x_bf16(9, units, cols).view(np.int16)).to(DEV).view(torch.bfloat16)
        y = torch.zeros(rows, dtype=torch.float32 if y_type == E.ENTRO_F32 else torch.bfloat16, device=DEV)
        plan, ws = _plan_of([dt.ctensor(y, x)], y_type, places=False)
        assert plan.shared_wave_bytes == 0
        us.append(_times_us([lambda: E.entro_plan_run(plan)], 20)[0])
        y_ref, _ = oracle.gemv(sym, rows, cols, 0.25, 7, synth.make_x_bf16(9, units, cols))
        _assert_gemv_close(y.float().cpu().numpy().astype(np.float64), y_ref, 1e-3 if y_type == E.ENTRO_F32 else 5e-3)
    assert us[1] <= 1.13 * us[0], us


def _refill(dt, enc):
    """Another tensor of the same codebook and sizes into dt's buffers."""
    other = E.to_device(enc, DEV)
    for name in ("stream", "offsets", "sub_bits"):
        if getattr(dt, name, None) is not None:
            getattr(dt, name).copy_(getattr(other, name))


def _without_places(ts):
    """The same products with a zero-point for which no places are noted: their room is that of a launch without any."""
    other = [B.CTensor.from_buffer_copy(t) for t in ts]
    for t in other:
        t.qp.zero_point = 1000
    return other


# forms that k_fine takes
NOTED_FORMS = [
    (8, 4096, 256, 67, 4096, 128),       # a row to a unit of 64 lanes
    (8, 1024, 128, 333, 64, -1),         # a row to a lane, a last unit of 13 lanes, the lowest zero-point
    (4, 2048, 128, 45, 1024, 16),        # four rows to a unit, the highest zero-point
    (8, 4096, 256, 21, 14336, 256),      # four units of lanes of 56 symbols (chains of 32 and 24) to a row
    (4, 8192, 512, 19, 3072, 7),         # lanes of 48 symbols across the ends of pieces
    (8, 4096, 512, 9, 16384, 100),       # more activations than LDS holds
    (8, 4096, 0, 13, 4160, 3),           # rows over units: partial sums; no entry points
    (4, 1024, 64, 37, 192, 5),           # rows that begin inside units and end in them, too
    (8, 1024, 256, 40, 1056, 90),        # lanes of 48 symbols, partial sums
    (4, 2048, 512, 11, 2080, -1),        # lanes of 32 symbols, partial sums, a last piece that is shorter
    (8, 1024, 0, 19, 3072, 90),          # three pieces to a unit, whose lanes share a piece's search by 21
    (4, 2048, 0, 37, 1024, 6),           # two pieces to a unit
    (4, 4096, 0, 5, 1600, 2),            # one piece to a unit, the last one of 3904 symbols
]


@pytest.mark.parametrize("y_type", [E.ENTRO_F32, E.ENTRO_BF16])
@pytest.mark.parametrize("bits,chunk,sub,rows,cols,z", NOTED_FORMS)
def test_products_of_lanes_at_noted_places(bits, chunk, sub, rows, cols, z, y_type):
    """Prepared products whose lanes begin where the preparation noted it: against the oracle, when the tensor's buffers have been
    given other contents of the same codebook and sizes since, and when the places have been noted anew for those."""
    top, n = (1 << bits) - 1, rows * cols
    rng = np.random.default_rng(rows * cols + bits)
    # (a heavy tail: codes longer than the first level's 14 bits, where the alphabet is large enough)
    spread = rng.standard_t(2.2, n) * (2.5 if bits == 8 else 0.8)
    first = np.clip(np.rint(spread) + (top + 1) // 2, 0, top).astype(np.uint8)
    x = synth.make_x_bf16(3, cols, cols)
    xd = torch.from_numpy(x.view(np.int16)).to(DEV).view(torch.bfloat16)
    dt, plan = None, None
    y = torch.zeros(rows, dtype=torch.float32 if y_type == E.ENTRO_F32 else torch.bfloat16, device=DEV)
    for sym in (first, np.roll(first, 1), rng.permutation(first)):
        enc = _oracle_encoded(sym, bits, chunk, rows, cols, 0.25, z, sub)
        if plan is None:
            dt = E.to_device(enc, DEV)
            ts = [dt.ctensor(y, xd)]
            ws = torch.zeros(E.entro_workspace_bytes(ts, E.ENTRO_OP_GEMV), dtype=torch.uint8, device=DEV)
            plan = E.entro_plan_init(ts, E.ENTRO_OP_GEMV, y_type, ws)
            assert plan.wide_tables == 2
        else:
            _refill(dt, enc)
        terms = (sym.reshape(rows, cols).astype(np.float64) - z) * 0.25 * (x.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
        # fp32 sums of exact products: at most cols roundings of half an ulp, relative to the terms' magnitudes; bf16: half an ulp on top
        bound = (cols + 2) * 2.0 ** -24 * np.abs(terms).sum(1) + (2.0 ** -8 * np.abs(terms.sum(1)) if y_type == E.ENTRO_BF16 else 0.0)
        for _ in range(2):
            y.fill_(7.0)
            E.entro_plan_run(plan)
            assert (np.abs(y.double().cpu().numpy() - terms.sum(1)) <= bound).all()


@pytest.mark.parametrize("bits,chunk,sub,rows,cols,z", NOTED_FORMS)
def test_products_do_not_depend_on_how_their_places_were_found(bits, chunk, sub, rows, cols, z):
    """The sums of a prepared product are taken in an order that depends on the launch, never on the run: when its buffers have been
    given other contents, the first run, which finds the places, the next one, which finds them noted, and a plan prepared for
    these contents agree to the last bit."""
    top, n = (1 << bits) - 1, rows * cols
    rng = np.random.default_rng(rows * cols + bits + 1)
    first = np.clip(np.rint(rng.standard_t(2.2, n) * (2.5 if bits == 8 else 0.8)) + (top + 1) // 2, 0, top).astype(np.uint8)
    x = torch.from_numpy(rng.standard_normal(cols).astype(np.float32)).to(DEV).to(torch.bfloat16)
    y = torch.zeros(rows, dtype=torch.float32, device=DEV)

    def plan_of(dt):
        ts = [dt.ctensor(y, x)]
        ws = torch.zeros(E.entro_workspace_bytes(ts, E.ENTRO_OP_GEMV), dtype=torch.uint8, device=DEV)
        plan = E.entro_plan_init(ts, E.ENTRO_OP_GEMV, E.ENTRO_F32, ws)
        assert plan.wide_tables == 2
        return plan, ws, dt

    def bits_of(plan):
        y.fill_(7.0)
        E.entro_plan_run(plan[0])
        return y.view(torch.int32).clone()
    dt = E.to_device(_oracle_encoded(first, bits, chunk, rows, cols, 0.25, z, sub), DEV)
    plan = plan_of(dt)
    for sym in (np.roll(first, 1), rng.permutation(first)):
        enc = _oracle_encoded(sym, bits, chunk, rows, cols, 0.25, z, sub)
        _refill(dt, enc)
        found, noted, fresh = bits_of(plan), bits_of(plan), bits_of(plan_of(E.to_device(enc, DEV)))
        assert torch.equal(found, noted) and torch.equal(noted, fresh)


def _plan_of(ts, out, places=True):
    """A prepared product, and its workspace: with places where the form allows it, or in a workspace that has no room for any."""
    ws = torch.zeros(E.entro_workspace_bytes(ts if places else _without_places(ts), E.ENTRO_OP_GEMV), dtype=torch.uint8, device=DEV)
    plan = E.entro_plan_init(ts, E.ENTRO_OP_GEMV, out, ws)
    assert (plan.wide_tables == 2) == places and (plan.shared_wave_bytes == 0 or not places)
    return plan, ws


@pytest.mark.parametrize("bits,chunk,sub,rows,cols,z", NOTED_FORMS)
def test_products_of_lanes_with_more_bits_than_their_columns_hold(bits, chunk, sub, rows, cols, z):
    """Stretches of long codes among short ones, up to 2^16 bits of a unit and more: against the oracle and, to the last bit, in every
    run the same, with the places noted beforehand, found anew and noted then."""
    top, n = (1 << bits) - 1, rows * cols
    lengths = np.array(list(range(1, 32)) + [32, 32] if bits == 8 else list(range(1, 15)) + [15, 15])
    rng = np.random.default_rng(n + bits)
    first = rng.choice(lengths.size, n, p=0.5 ** lengths / (0.5 ** lengths).sum()).astype(np.uint8)
    for at in rng.integers(0, n, n // 4096 + 2):             # stretches of 200 symbols with codes of 10 bits and more
        first[at:at + 200] = rng.integers(9, 15, first[at:at + 200].size)
    unit = n // 2 // 4096 * 4096                             # and a whole unit, or what there is, of the longest codes
    first[unit:unit + min(4096, n // 12)] = lengths.size - 1
    x = synth.make_x_bf16(3, cols, cols)
    xd = torch.from_numpy(x.view(np.int16)).to(DEV).view(torch.bfloat16)
    cb = E.entro_codebook_from_lengths(np.pad(lengths, (0, top + 1 - lengths.size)).astype(np.uint8), bits)
    y = torch.zeros(rows, dtype=torch.float32, device=DEV)

    def held(sym):
        stream, off = E.entro_encode(sym, cb, chunk)
        enc = B.EncodedTensor(stream, off, n, chunk, cb, B.QParams(np.float32(0.25), z, bits, E.ENTRO_ASYMMETRIC), rows, cols)
        if sub:
            enc.sub_symbols, enc.sub_bits = sub, E.entro_sub_index(sym, cb, chunk, sub)
        return enc
    other, dt, plan = rng.permutation(first), None, None
    for sym in (first, np.roll(first, 1), other):
        if dt is None:
            dt = E.to_device(held(sym), DEV)
            plan = _plan_of([dt.ctensor(y, xd)], E.ENTRO_F32)
        else:
            _refill(dt, held(sym))
        terms = (sym.reshape(rows, cols).astype(np.float64) - z) * 0.25 * (x.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
        bound = (cols + 2) * 2.0 ** -24 * np.abs(terms).sum(1)   # fp32 sums of exact products
        fresh, runs = _plan_of([dt.ctensor(y, xd)], E.ENTRO_F32), []
        for p in (plan, plan, fresh):
            y.fill_(7.0)
            E.entro_plan_run(p[0])
            assert (np.abs(y.double().cpu().numpy() - terms.sum(1)) <= bound).all()
            runs.append(y.view(torch.int32).clone())
        assert torch.equal(runs[0], runs[1]) and torch.equal(runs[1], runs[2])


def test_rows_of_wide_spread_take_no_longer_than_a_lane_per_piece():
    """Rows of different spread under one scale: some lanes have more bits than their columns hold.  0.3 of the time that a lane per
    piece takes (1.25 where such a unit was walked in every launch)."""
    rows, cols, gen = 4096, 4096, torch.Generator(device=DEV)
    gen.manual_seed(1)
    w = torch.randn(rows, cols, device=DEV, generator=gen) * torch.exp(torch.randn(rows, 1, device=DEV, generator=gen) * 0.8) * 0.02
    d, q = E.compress_on_device(w.clamp_(-0.4, 0.4).view(-1), 8, E.ENTRO_ASYMMETRIC, 4096, rows=rows, cols=cols, return_q=True)
    d.enc.sub_symbols = 256
    ln = torch.from_numpy(d.enc.cb.lengths().astype(np.int32)).to(DEV)
    d.sub_bits = ln[q.int()].view(-1, 256).sum(1).to(torch.int16)
    x = torch.randn(cols, device=DEV, generator=gen).to(torch.bfloat16)
    assert int(ln[q.int()].view(-1, 64).sum(1).max()) > 512 and float(ln[q.int()].float().mean()) < 6.0
    ys = [torch.zeros(rows, dtype=torch.float32, device=DEV) for _ in range(2)]
    plans = [_plan_of([d.ctensor(y, x)], E.ENTRO_F32, places) for y, places in zip(ys, (True, False))]
    us = _times_us([lambda p=p: E.entro_plan_run(p[0]) for p in plans], 10)
    assert float((ys[0] - ys[1]).norm() / ys[1].norm()) <= 1e-6
    assert us[0] <= 0.7 * us[1], us


@pytest.mark.parametrize("bits,chunk,sub,rows,cols", [(8, 4096, 256, 3000, 4096), (8, 4096, 0, 101, 2880), (4, 4096, 512, 3072, 3072)])
def test_products_under_codes_that_do_not_fall_into_step(bits, chunk, sub, rows, cols):
    # places are walked, not guessed: such codes have them like any other (9.3, 9.8 and 7.5 us; without 22.5, 245 and 26.0)
    enc, sym = _out_of_step(bits, chunk, rows * cols, rows, cols, sub)
    x = synth.make_x_bf16(5, 0, cols)
    dt, xd = E.to_device(enc, DEV), torch.from_numpy(x.view(np.int16)).to(DEV).view(torch.bfloat16)
    y = torch.zeros(rows, dtype=torch.float32, device=DEV)
    plans = [_plan_of([dt.ctensor(y, xd)], E.ENTRO_F32, places) for places in (True, False)]
    us = _times_us([lambda p=p: E.entro_plan_run(p[0]) for p in plans], 10)
    sym, runs = np.roll(sym, 3), []                          # and other contents, where no search of starts would end soon
    stream, off = E.entro_encode(sym, enc.cb, chunk)
    other = B.EncodedTensor(stream, off, enc.n, chunk, enc.cb, enc.qp, rows, cols)
    if sub:
        other.sub_symbols, other.sub_bits = sub, E.entro_sub_index(sym, enc.cb, chunk, sub)
    _refill(dt, other)
    for _ in range(2):
        E.entro_plan_run(plans[0][0])
        runs.append(y.clone())
    assert torch.equal(runs[0], runs[1])
    y_ref, _ = oracle.gemv(sym, rows, cols, 0.25, 7, x)
    terms = np.abs((sym.reshape(rows, cols).astype(np.float64) - 7) * 0.25) @ np.abs((x.astype(np.uint32) << 16).view(np.float32).astype(np.float64))
    assert np.all(np.abs(y.double().cpu().numpy() - y_ref) <= (cols + 2) * 2.0 ** -24 * terms)
    assert us[0] <= us[1], us


@pytest.mark.parametrize("bits,rows,cols,z", [(8, 67, 4096, 128), (4, 37, 192, 5)])
def test_products_with_room_for_no_places_run_without_them(bits, rows, cols, z):
    rng = np.random.default_rng(cols)
    sym = np.clip(np.rint(rng.standard_normal(rows * cols) * (3 if bits == 8 else 1)) + (1 << (bits - 1)), 0, (1 << bits) - 1).astype(np.uint8)
    enc = _oracle_encoded(sym, bits, 1024, rows, cols, 0.25, z, 64 if bits == 4 else 128)
    x = synth.make_x_bf16(3, cols, cols)
    y_ref, _ = oracle.gemv(sym, rows, cols, 0.25, z, x)
    dt, xd = E.to_device(enc, DEV), torch.from_numpy(x.view(np.int16)).to(DEV).view(torch.bfloat16)
    y = torch.zeros(rows, dtype=torch.float32, device=DEV)
    ts = [dt.ctensor(y, xd)]
    most, least = (E.entro_workspace_bytes(t, E.ENTRO_OP_GEMV) for t in (ts, _without_places(ts)))
    staged, staged_least = (E.entro_plan_staging_bytes(t, E.ENTRO_OP_GEMV) for t in (ts, _without_places(ts)))
    assert most > least and staged >= staged_least

    def room(n):
        return torch.zeros(n, dtype=torch.uint8, device=DEV)

    def pinned(n):
        return torch.zeros(n, dtype=torch.uint8).pin_memory()
    # (workspace, staging memory or none, are places noted?)
    for ws, staging, noted in [(room(most), None, True), (room(most - 16), None, False), (room(least), None, False),
                               (room(most), pinned(staged), True), (room(least), pinned(staged_least), False)]:
        if staging is None:
            plan = E.entro_plan_init(ts, E.ENTRO_OP_GEMV, E.ENTRO_F32, ws)
        else:
            plan = E.entro_plan_init_staged(ts, E.ENTRO_OP_GEMV, E.ENTRO_F32, ws, staging)
        assert (plan.wide_tables == 2) == noted
        y.zero_()
        E.entro_plan_run(plan)
        _assert_gemv_close(y.cpu().numpy().astype(np.float64), y_ref)
    # a batch product never notes places, and takes the room of a launch without any
    ws = room(least)
    y.zero_()
    E.entro_decode_gemv_batch(ts, E.ENTRO_F32, ws)
    _assert_gemv_close(y.cpu().numpy().astype(np.float64), y_ref)
    with pytest.raises(E.EntroError) as e:
        E.entro_decode_gemv_batch(ts, E.ENTRO_F32, room(least - 16))
    assert e.value.status == B.ENTRO_ERR_CAPACITY
    with pytest.raises(E.EntroError) as e:
        E.entro_plan_init_staged(ts, E.ENTRO_OP_GEMV, E.ENTRO_F32, ws, pinned(staged_least - 16))
    assert e.value.status == B.ENTRO_ERR_CAPACITY


@pytest.mark.parametrize("bits", [8, 4])
def test_more_products_in_one_launch_than_a_grid_has_rows(bits):
    # 65537 products of one and two rows (about 70 KB of workspace each)
    count, cols = 65537, 64
    rng = np.random.default_rng(bits)
    encs = [_oracle_encoded(np.clip(np.rint(rng.standard_normal(r * cols) * 2) + 7, 0, 15).astype(np.uint8), bits, 64, r, cols, 0.25, 7) for r in (1, 2)]
    x = torch.from_numpy(synth.make_x_bf16(6, 0, cols).view(np.int16)).to(DEV).view(torch.bfloat16)
    y = torch.zeros(count, 4, dtype=torch.float32, device=DEV)
    dts, step = [E.to_device(e, DEV) for e in encs], y.element_size() * 4
    kinds = [d.ctensor(y, x) for d in dts]
    ts = [B.CTensor.from_buffer_copy(kinds[i & 1]) for i in range(count)]
    for i, t in enumerate(ts):
        t.out = y.data_ptr() + step * i
    plan, ws = _plan_of(ts, E.ENTRO_F32)
    E.entro_plan_run(plan)
    y = y.cpu().numpy()
    for k, e in enumerate(encs):
        q = oracle.decode(e.stream, e.offsets, e.n, e.chunk_symbols, e.cb.lengths(), e.cb.codes())
        y_ref, _ = oracle.gemv(q, e.rows, cols, 0.25, 7, synth.make_x_bf16(6, 0, cols))
        assert np.abs(y[k::2, :e.rows] - y_ref).max() <= 1e-5 * max(1.0, np.abs(y_ref).max()) and not y[k::2, e.rows:].any()


def test_products_that_lanes_of_noted_places_do_not_take():
    """Zero-points that the tables' values cannot hold, codes too long for a lane's stream, shapes that do not cut into lanes, mixed
    alphabets and single runs go the ways they went."""
    def wide(forms, batch=False):
        encs, xs, syms = [], [], []
        for bits, chunk, sub, rows, cols, z, spread in forms:
            top = (1 << bits) - 1
            sym = np.clip(np.rint(np.random.default_rng(cols).standard_normal(rows * cols) * spread) + (top + 1) // 2, 0, top).astype(np.uint8)
            encs.append(_oracle_encoded(sym, bits, chunk, rows, cols, 0.5, z, sub))
            xs.append(synth.make_x_bf16(4, cols, cols))
            syms.append(sym)
        xd = [torch.from_numpy(x.view(np.int16)).to(DEV).view(torch.bfloat16) for x in xs]
        ys = [torch.zeros(e.rows, dtype=torch.float32, device=DEV) for e in encs]
        dts = [E.to_device(e, DEV) for e in encs]
        ts = [d.ctensor(y, x) for d, y, x in zip(dts, ys, xd)]
        ws = torch.zeros(E.entro_workspace_bytes(ts, E.ENTRO_OP_GEMV), dtype=torch.uint8, device=DEV)
        plan = E.entro_plan_init(ts, E.ENTRO_OP_GEMV, E.ENTRO_F32, ws)
        E.entro_plan_run(plan)
        for y, e, s, x, f in zip(ys, encs, syms, xs, forms):
            _assert_gemv_close(y.cpu().numpy().astype(np.float64), oracle.gemv(s, e.rows, e.cols, 0.5, f[5], x)[0])
        return plan.wide_tables == 2
    base = (8, 4096, 256, 33, 4096, 128, 3.0)
    four = (4, 4096, 256, 33, 4096, 7, 1.0)
    assert wide([base, base]) and wide([four])
    assert not wide([base, four])
    assert not wide([base[:5] + (257, 3.0)]) and not wide([four[:5] + (17, 1.0)])
    assert not wide([base[:6] + (60.0,)])                        # 7.9 bits a symbol
    assert not wide([(8, 4096, 256, 33, 4100, 128, 3.0)])        # rows that are not whole pieces of eight activations
    assert not wide([(8, 8192, 0, 33, 4096, 128, 3.0)])          # a unit's first bit is not in the tables
    assert not wide([(8, 4000, 0, 33, 4096, 128, 3.0)])


@pytest.mark.parametrize("out", [E.ENTRO_F32, E.ENTRO_BF16])
@pytest.mark.parametrize("lengths", [[8] * 256, [7] * 60 + [8] * 76 + [9] * 120, [5, 2, 3, 3, 4, 5, 4, 5, 2, 5], [1, 1], [3] * 7 + [6] * 8,
                                     [1, 2, 3, 4, 5, 5], [1]])
def test_small_calls_under_codes_of_nearly_one_length(lengths, out):
    # four neighbouring lengths at most, and two codes that have more or leave space unused; pieces and segments of whole blocks and
    # not, a last one that is shorter, lanes of one wavefront and of two
    cb = E.entro_codebook_from_lengths(np.pad(np.array(lengths, np.uint8), (0, 256 - min(256, len(lengths))))[:256], 8)
    rng = np.random.default_rng(len(lengths))
    for n, chunk, sub in ((1, 4096, 0), (2048, 4096, 256), (2049, 2048, 128), (33000, 4096, 256), (5000, 1000, 0)):
        sym = rng.integers(0, min(256, len(lengths)), n).astype(np.uint8)
        stream, off = E.entro_encode(sym, cb, chunk)
        enc = B.EncodedTensor(stream, off, n, chunk, cb, B.QParams(np.float32(0.37), 11, 8, E.ENTRO_ASYMMETRIC), 1, n)
        if sub:
            enc.sub_symbols, enc.sub_bits = sub, E.entro_sub_index(sym, cb, chunk, sub)
        y = torch.zeros(n + 8, dtype=torch.float32 if out == E.ENTRO_F32 else torch.bfloat16, device=DEV)
        E.entro_decode_dequant(E.to_device(enc, DEV).ctensor(y), out)
        if out == E.ENTRO_F32:
            assert np.array_equal(y.cpu().numpy()[:n], oracle.dequant_f32(sym, 0.37, 11))
        else:
            assert np.array_equal(y.view(torch.int16).cpu().numpy().view(np.uint16)[:n], oracle.dequant_bf16(sym, 0.37, 11))
        assert float(y[n:].abs().sum()) == 0.0
