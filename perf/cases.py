"""Performance cases of the FP8 <-> MXFP4 conversions: what a training or dispatch program calls, and at which sizes.

The listed cases are the named workloads of this repository (hidden 7168, expert width 2048, 32 experts of
Zipf-distributed lengths, top-8 dispatch into per-token records, [65536, 7168] activations) and its tiny and ordinary
sizes; `draw` spreads the same calls over the whole range of row counts, widths, splits and fan-outs.  Every result is
a set of bytes or of power-of-two scales, so two correct implementations agree bit for bit.
"""
import math

import torch

import paper_2603_02731_amd as mx

DEV = "cuda:0"
CHUNK = 1 << 25  # elements worked on at a time where inputs or reference results are made

OPS = ("quant", "quant_bf16", "quant_gather", "quant_scatter", "dequant", "dequant_records", "step",
       "row_to_col", "row_to_col_experts", "fp8_col", "fp8_col_experts")


def listed():
    return [
        # a handful of rows, as in a unit of work of a small model or a debugging run: launch and call overhead
        {"name": "quant_tiny", "op": "quant", "M": 256, "K": 512},
        # one micro-batch of 4096 tokens through the three flat conversions of a training step, in their order
        {"name": "step_4096", "op": "step", "M": 4096, "K": 7168},
        # the activations of a large global batch, quantized for storage
        {"name": "quant_65536", "op": "quant", "M": 65536, "K": 7168},
        # the paper's own quantizer input, BF16 activations
        {"name": "quant_bf16_16384", "op": "quant_bf16", "M": 16384, "K": 7168},
        # dispatch with the map from copies to tokens: every copy's record is quantized from its token's row
        {"name": "gather_8192_top8", "op": "quant_gather", "M": 8192, "K": 7168, "fanout": 8, "experts": 32,
         "records": True},
        # dispatch with the map from tokens to copies: every token is quantized once, written to eight records
        {"name": "scatter_65536_top8", "op": "quant_scatter", "M": 65536, "K": 7168, "fanout": 8, "experts": 32,
         "records": True},
        # the receiving side of the dispatch: records back to blockwise FP8
        {"name": "dequant_records_65536", "op": "dequant_records", "M": 65536, "K": 7168},
        # the weight-gradient operand of a dense layer
        {"name": "row_to_col_65536", "op": "row_to_col", "M": 65536, "K": 7168},
        # expert activations as routing leaves them, no padding: k-rows start at any byte
        {"name": "row_to_col_ragged_2048", "op": "row_to_col_experts", "M": 65536, "K": 2048, "experts": 32,
         "skew": 1.2, "pad": 1},
        # the FP8 form of the weight-gradient operand, one expert-FFN micro-batch
        {"name": "fp8_col_16384x2048", "op": "fp8_col", "M": 16384, "K": 2048, "requant": False},
        # 32 experts padded to whole scale groups, full hidden width
        {"name": "fp8_col_padded_7168", "op": "fp8_col_experts", "M": 65536, "K": 7168, "experts": 32, "skew": 1.2,
         "pad": 128, "requant": False},
        # the same without padding, under the re-quantizing reading
        {"name": "requant_col_ragged_7168", "op": "fp8_col_experts", "M": 65536, "K": 7168, "experts": 32,
         "skew": 1.2, "pad": 1, "requant": True},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(OPS)
    K = 128 * _log_uniform(rng, 4, 64)  # 512 .. 8192, odd multiples of 128 among them
    M = _log_uniform(rng, 64, 65536)
    c = {"op": op, "K": K}
    if op in ("quant_gather", "quant_scatter"):
        c["fanout"] = rng.randint(1, 8)
        c["experts"] = rng.choice((8, 32, 64, 128, 256))
        c["records"] = rng.random() < 0.5
        # no larger than the listed dispatches
        most = (8192 if op == "quant_gather" else 65536) * 7168 * 8 // (K * c["fanout"])
        M = min(M, most, 65536)
    elif op in ("step", "row_to_col"):
        M = 32 * max(1, M // 32)
    elif op == "fp8_col":
        M = 128 * max(1, M // 128)
        c["requant"] = rng.random() < 0.5
    elif op in ("row_to_col_experts", "fp8_col_experts"):
        M = _log_uniform(rng, 2048, 57344)
        c["experts"] = rng.choice((1, 4, 8, 16, 32, 64, 128))
        c["skew"] = rng.choice((0.0, 0.5, 1.2))
        c["pad"] = rng.choice((1, 1, 16, 128))
        if op == "fp8_col_experts":
            c["requant"] = rng.random() < 0.5
    if op == "step":
        M = min(M, 32768)
    c["M"] = M
    return c


# ---- shapes and inputs


def _splits(case):
    """Rows of every expert, largest first: Zipf shares of M tokens (skew 0: equal shares, the remainder to the
    first), padded up to a multiple of `pad`."""
    E, M = case["experts"], case["M"]
    w = [(r + 1.0) ** -case["skew"] for r in range(E)]
    t = [int(M * v / sum(w)) for v in w]
    t[0] += M - sum(t)
    p = case["pad"]
    return [-(-n // p) * p for n in t]


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _chunks(rows, K, group=1):
    step = max(group, CHUNK // max(K, 1) // group * group)
    return [(r, min(rows, r + step)) for r in range(0, rows, step)]


def _activations(rows, K, seed):
    """float32 row chunks of Student-t(3) activations with 1 % outlier channels, 100 times the others."""
    g = _gen(seed)
    gain = torch.ones(K, device=DEV)
    gain[torch.randperm(K, generator=g, device=DEV)[: max(1, K // 100)]] = 100.0
    for r0, r1 in _chunks(rows, K):
        z = torch.randn(r1 - r0, K, generator=g, device=DEV)
        chi = torch.zeros_like(z)
        for _ in range(3):
            chi += torch.randn(r1 - r0, K, generator=g, device=DEV) ** 2
        yield r0, r1, z / torch.sqrt(chi / 3.0) * gain


def _fp8_input(rows, K, seed):
    """Blockwise FP8: E4M3 bytes and one FP32 scale amax/448 per 1x128 tile."""
    x = torch.empty(rows, K, dtype=torch.uint8, device=DEV)
    s = torch.empty(rows, K // 128, device=DEV)
    for r0, r1, v in _activations(rows, K, seed):
        t = v.view(r1 - r0, K // 128, 128)
        a = t.abs().amax(-1, keepdim=True) / 448.0
        y = (t / torch.where(a > 0, a, torch.ones_like(a))).clamp(-448.0, 448.0)
        x[r0:r1] = y.to(torch.float8_e4m3fn).view(torch.uint8).view(r1 - r0, K)
        s[r0:r1] = a.view(r1 - r0, K // 128)
    return x, s


def _power(e):
    """2^e as float64, from the bits of its exponent field."""
    return ((e.long() + 1023) << 52).view(torch.float64)


def _mxfp4(v):
    """Rows of v (a multiple of 32 long) as packed E2M1 codes and UE8M0 bytes: per 32 elements the smallest power of
    two 2^k with max|v| <= 6 * 2^k, then round-to-nearest-even onto 0 .5 1 1.5 2 3 4 6."""
    rows, n = v.shape
    u = v.abs().view(rows, n // 32, 32)
    mant, e = torch.frexp(u.amax(-1))
    b = torch.where(mant > 0, e - 3 + (mant > 0.75).to(e.dtype) + 127, torch.zeros_like(e)).clamp(0, 254)
    u = u * _power(127 - b).to(u.dtype).unsqueeze(-1)
    code = (u > 0.25).to(torch.uint8)
    for at, tie_up in ((0.75, True), (1.25, False), (1.75, True), (2.5, False), (3.5, True), (5.0, False)):
        code += (u >= at) if tie_up else (u > at)
    code = code.view(rows, n) | (torch.signbit(v).to(torch.uint8) << 3)
    return code[:, 0::2] | (code[:, 1::2] << 4), b.to(torch.uint8)


def _mxfp4_input(rows, K, seed):
    q = torch.empty(rows, K // 2, dtype=torch.uint8, device=DEV)
    sf = torch.empty(rows, K // 32, dtype=torch.uint8, device=DEV)
    for r0, r1, v in _activations(rows, K, seed):
        q[r0:r1], sf[r0:r1] = _mxfp4(v)
    return q, sf


def _routes(case, seed):
    """Top-k routing: int32 dst [M, fanout], the position of every copy in the dispatch buffer, where the copies are
    grouped by expert and keep the token order inside an expert; and its inverse, the token of every copy."""
    M, F, E = case["M"], case["fanout"], case["experts"]
    p = torch.rand(M, E, generator=_gen(seed), device=DEV)
    p = p * (torch.arange(E, device=DEV) + 1.0) ** -0.3  # some experts are asked for more often
    expert = p.topk(F, dim=1).indices.reshape(-1)
    order = torch.sort(expert, stable=True).indices  # copy (token * F + j) at every position
    dst = torch.empty(M * F, dtype=torch.int32, device=DEV)
    dst[order] = torch.arange(M * F, dtype=torch.int32, device=DEV)
    return dst.view(M, F), (order // F).to(torch.int32)


def _record(K):
    """Bytes from one per-token record to the next: its nibbles and scale bytes, on a 16-byte boundary."""
    return -(-(K // 2 + K // 32) // 16) * 16


def _packed(rows, K, records):
    """Output buffers of the quantizers: two planes, or one record of nibbles and scale bytes per row.
    Returns (q, sf, ld_q, ld_sf, what to give back)."""
    if records:
        ld = _record(K)
        rec = torch.empty(rows, ld, dtype=torch.uint8, device=DEV)
        flat = rec.view(-1)
        return flat, flat[K // 2:], ld, ld, rec[:, : K // 2 + K // 32]
    q = torch.empty(rows, K // 2, dtype=torch.uint8, device=DEV)
    sf = torch.empty(rows, K // 32, dtype=torch.uint8, device=DEV)
    return q, sf, K // 2, K // 32, (q, sf)


def _inputs(case, seed):
    op, M, K = case["op"], case["M"], case["K"]
    s = {"op": op, "M": M, "K": K}
    if op in ("quant", "step", "quant_gather", "quant_scatter"):
        s["x"], s["x_scale"] = _fp8_input(M, K, seed)
        if op in ("quant_gather", "quant_scatter"):
            s["dst"], s["gather"] = _routes(case, seed)
    elif op == "quant_bf16":
        s["x"] = torch.empty(M, K, dtype=torch.bfloat16, device=DEV)
        for r0, r1, v in _activations(M, K, seed):
            s["x"][r0:r1] = v.to(torch.bfloat16)
    elif op in ("row_to_col_experts", "fp8_col_experts"):
        t = _splits(case)
        order = torch.randperm(len(t), generator=torch.Generator().manual_seed(int(seed))).tolist()
        s["rows"] = [t[i] for i in order]  # which expert is the busy one changes from batch to batch
        s["q"], s["sf"] = _mxfp4_input(sum(t), K, seed)
    else:
        s["q"], s["sf"] = _mxfp4_input(M, K, seed)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    op, M, K = s["op"], s["M"], s["K"]
    if op in ("quant_gather", "quant_scatter"):
        s["out"] = _packed(M * case["fanout"], K, case["records"])
        del s["gather" if op == "quant_scatter" else "dst"]
    elif op == "dequant_records":
        rec = torch.zeros(M, _record(K), dtype=torch.uint8, device=DEV)
        rec[:, : K // 2] = s.pop("q")
        rec[:, K // 2: K // 2 + K // 32] = s.pop("sf")
        s["rec"] = rec.view(-1)
    elif op in ("row_to_col_experts", "fp8_col_experts"):
        rows, E = s["rows"], len(s["rows"])
        off = [0]
        for n in rows:
            off.append(off[-1] + n)
        s["offsets"] = torch.tensor(off, dtype=torch.int32, device=DEV)
        # the documented upper bounds; what is written is handed back
        if op == "row_to_col_experts":
            s["n"] = [K * sum(-(-n // u) for n in rows) for u in (2, 32)]
            s["out"] = [torch.empty(K * (off[-1] // u + E), dtype=torch.uint8, device=DEV) for u in (2, 32)]
        else:
            s["requant"] = case["requant"]
            s["n"] = [K * off[-1], K * sum(-(-n // 128) for n in rows)]
            s["out"] = [torch.empty(K * off[-1], dtype=torch.uint8, device=DEV),
                        torch.empty(K * (off[-1] // 128 + E), device=DEV)]
    elif op == "fp8_col":
        s["requant"] = case["requant"]
    return s


def run(s):
    op = s["op"]
    if op == "quant":
        return mx.mxfp4_quant_from_fp8(s["x"], s["x_scale"])
    if op == "quant_bf16":
        return mx.mxfp4_quant_from_bf16(s["x"])
    if op == "quant_gather":
        q, sf, ld_q, ld_sf, out = s["out"]
        mx.mxfp4_quant_from_fp8(s["x"], s["x_scale"], s["gather"], q=q, sf=sf, ld_q=ld_q, ld_sf=ld_sf)
        return out
    if op == "quant_scatter":
        q, sf, ld_q, ld_sf, out = s["out"]
        mx.mxfp4_quant_from_fp8_scatter(s["x"], s["x_scale"], s["dst"], s["dst"].numel(), q=q, sf=sf, ld_q=ld_q,
                                        ld_sf=ld_sf)
        return out
    if op == "dequant":
        return mx.mxfp4_dequant_to_fp8(s["q"], s["sf"])
    if op == "dequant_records":
        K, ld = s["K"], _record(s["K"])
        return mx.mxfp4_dequant_to_fp8(s["rec"], s["rec"][K // 2:], M=s["M"], K=K, ld_q=ld, ld_sf=ld)
    if op == "step":
        q, sf = mx.mxfp4_quant_from_fp8(s["x"], s["x_scale"])
        return (q, sf), mx.mxfp4_dequant_to_fp8(q, sf), mx.mxfp4_row_to_col(q, sf)
    if op == "row_to_col":
        return mx.mxfp4_row_to_col(s["q"], s["sf"])
    if op == "fp8_col":
        return mx.mxfp4_row_to_fp8_col(s["q"], s["sf"], requant=s["requant"])
    a, b = s["out"]
    if op == "row_to_col_experts":
        mx.mxfp4_row_to_col_grouped(s["q"], s["sf"], s["offsets"], q_col=a, sf_col=b)
    else:
        mx.mxfp4_row_to_fp8_col_grouped(s["q"], s["sf"], s["offsets"], x_col=a, x_col_scale=b, requant=s["requant"])
    return a[: s["n"][0]], b[: s["n"][1]]


def work(case):
    op, M, K = case["op"], case["M"], case["K"]
    fp8, mxb = K + K // 32, K // 2 + K // 32  # bytes of a row in either format (4 bytes of scale per 128)
    if op == "quant":
        n = M * (fp8 + mxb)
    elif op == "quant_bf16":
        n = M * (2 * K + mxb)
    elif op in ("quant_gather", "quant_scatter"):
        n = M * fp8 + M * case["fanout"] * (mxb + 4)
    elif op in ("dequant", "dequant_records"):
        n = M * (mxb + fp8)
    elif op == "step":
        n = M * (fp8 + mxb) + M * (mxb + fp8) + 2 * M * mxb
    elif op == "row_to_col":
        n = 2 * M * mxb
    elif op == "fp8_col":
        n = M * (mxb + fp8)
    else:
        t = _splits(case)
        n = sum(t) * mxb + 4 * (len(t) + 1)
        if op == "row_to_col_experts":
            n += K * sum(-(-r // 2) + -(-r // 32) for r in t)
        else:
            n += K * sum(r + 4 * -(-r // 128) for r in t)
    return {"bytes": n, "flops": 0}


def tolerance(case):
    return "exact"  # bytes, and FP32 scales that are powers of two


# ---- the same results in 64 bits


def _values(q, sf):
    """float64 [rows, K] of packed codes and scale bytes."""
    lut = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6, -0., -.5, -1, -1.5, -2, -3, -4, -6], dtype=torch.float64, device=DEV)
    code = torch.stack((q & 15, q >> 4), dim=-1).view(q.shape[0], -1).long()
    return lut[code] * _power(sf.int() - 127).repeat_interleave(32, dim=1)


def _e4m3(v):
    return v.float().to(torch.float8_e4m3fn).view(torch.uint8)


def _exact_quant(x, s):
    q, sf = [], []
    for r0, r1 in _chunks(x.shape[0], x.shape[1]):
        # an element's value is its FP32 product with the tile scale
        v = x[r0:r1].view(torch.float8_e4m3fn).float() * s[r0:r1].repeat_interleave(128, dim=1)
        for out, part in zip((q, sf), _mxfp4(v.double())):
            out.append(part)
    return torch.cat(q), torch.cat(sf)


def _exact_dequant(q, sf):
    M, K = q.shape[0], 2 * q.shape[1]
    x = torch.empty(M, K, dtype=torch.uint8, device=DEV)
    s = torch.empty(M, K // 128, dtype=torch.float64, device=DEV)
    for r0, r1 in _chunks(M, K):
        s[r0:r1] = _power(sf[r0:r1].view(r1 - r0, K // 128, 4).amax(-1).int() - 133)
        x[r0:r1] = _e4m3(_values(q[r0:r1], sf[r0:r1]) / s[r0:r1].repeat_interleave(128, dim=1))
    return x, s


def _exact_row_to_col(q, sf):
    """One matrix of any number of rows; a last block of fewer than 32 rows is quantized over the rows it has."""
    M, K = q.shape[0], 2 * q.shape[1]
    qc = torch.empty(K, -(-M // 2), dtype=torch.uint8, device=DEV)
    sc = torch.empty(K, -(-M // 32), dtype=torch.uint8, device=DEV)
    for r0, r1 in _chunks(M, K, 32):
        v = _values(q[r0:r1], sf[r0:r1]).t()
        v = torch.nn.functional.pad(v, (0, -(r1 - r0) % 32)).contiguous()
        a, b = _mxfp4(v)
        qc[:, r0 // 2: -(-r1 // 2)] = a[:, : -(-(r1 - r0) // 2)]
        sc[:, r0 // 32: -(-r1 // 32)] = b
    return qc, sc


def _exact_fp8_col(q, sf, requant):
    M, K = q.shape[0], 2 * q.shape[1]
    x = torch.empty(K, M, dtype=torch.uint8, device=DEV)
    s = torch.empty(K, -(-M // 128), dtype=torch.float64, device=DEV)
    for r0, r1 in _chunks(M, K, 128):
        n, pad = r1 - r0, -(r1 - r0) % 128
        v = torch.nn.functional.pad(_values(q[r0:r1], sf[r0:r1]).t(), (0, pad)).reshape(K, -1, 128)
        if requant:  # the smallest power of two S with max|v| <= 448 * S; 1 for a group of zeros
            mant, e = torch.frexp(v.abs().amax(-1))
            g = torch.where(mant > 0, _power(e - 9 + (mant > 0.875).int()), torch.ones_like(mant))
        else:        # the largest scale of the group, minus 6 binades
            b = torch.nn.functional.pad(sf[r0:r1].t().int(), (0, pad)).reshape(K // 32, -1, 128).amax(-1)
            g = _power(b - 133).repeat_interleave(32, dim=0)
        x[:, r0:r1] = _e4m3(v / g.unsqueeze(-1)).reshape(K, -1)[:, :n]
        s[:, r0 // 128: -(-r1 // 128)] = g
    return x, s


def exact(case, seed):
    s = _inputs(case, seed)
    op = s["op"]
    if op == "quant":
        return _exact_quant(s["x"], s["x_scale"])
    if op == "quant_bf16":
        parts = [_mxfp4(s["x"][r0:r1].double()) for r0, r1 in _chunks(s["M"], s["K"])]
        return torch.cat([a for a, _ in parts]), torch.cat([b for _, b in parts])
    if op in ("quant_gather", "quant_scatter"):
        q, sf = _exact_quant(s["x"], s["x_scale"])
        at = s["gather"].long()
        return torch.cat((q, sf), dim=1)[at] if case["records"] else (q[at], sf[at])
    if op in ("dequant", "dequant_records"):
        return _exact_dequant(s["q"], s["sf"])
    if op == "step":
        q, sf = _exact_quant(s["x"], s["x_scale"])
        return (q, sf), _exact_dequant(q, sf), _exact_row_to_col(q, sf)
    if op == "row_to_col":
        return _exact_row_to_col(s["q"], s["sf"])
    if op == "fp8_col":
        return _exact_fp8_col(s["q"], s["sf"], case["requant"])
    parts, r = [], 0
    for n in s["rows"]:
        if n:
            q, sf = s["q"][r: r + n], s["sf"][r: r + n]
            parts.append(_exact_row_to_col(q, sf) if op == "row_to_col_experts" else
                         _exact_fp8_col(q, sf, case["requant"]))
        r += n
    return torch.cat([a.reshape(-1) for a, _ in parts]), torch.cat([b.reshape(-1) for _, b in parts])
