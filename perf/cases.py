"""The work a program hands to this library: attention softmax, GELU and requantization of
integer vision transformers, from one image at a time to large batches.

Sizes are those of DeiT-T, ViT-S/B and Swin-B at their usual resolutions (the benchmark's own
workloads), of shifted windows and token maps of other sides, and of rows up to the interface's
limit.  Scores are exact integer products of int8 queries and keys; scales are log-uniform in
[2^-10, 2^-4]; every output is whole bytes, so results must be identical.
"""
import math

import torch

import paper_2511_15369_amd as ip

I32_MIN = -(2 ** 31)


# ----------------------------------------------------------------------------- the cases
def listed():
    return [
        # one image through one transformer block: two small launches, latency only
        dict(name="deit_t_block_b1", kind="block", images=1, heads=3, tokens=197, width=768,
             s_delta=2.0 ** -7, s_in=2.0 ** -4, variant=1),
        # an attention layer at an ordinary and at a large batch
        dict(name="vit_s_attention_b64", kind="rows", rows=64 * 6 * 197, cols=197, s_delta=0.0071,
             variant=1, form="uint8", pre=False, offset=0),
        dict(name="vit_b_attention_b128", kind="rows", rows=128 * 12 * 197, cols=197, s_delta=0.019,
             variant=0, form="uint8", pre=False, offset=0),
        # the activation of an MLP, int8 codes in and out
        dict(name="vit_b_gelu_b128", kind="gelu", n=128 * 197 * 3072, s_in=0.021, variant=1),
        # an MLP that hands over int32 accumulators: GELU with the requantization in front, then
        # the requantization of the second product
        dict(name="vit_s_mlp_b64", kind="mlp", tokens=64 * 197, width=1536, dim=384, s_in=2.0 ** -5,
             variant=1),
        # the shifted block of each of the four stages of a Swin backbone, mask one bit per key
        dict(name="swin_b_shifted_stages_b64", kind="stages", images=64, heads=4, side=8, win=7,
             n_stages=4, mask="bits", s_delta=0.0048, variant=1),
        # a shifted block with windows of 8 x 8 tokens (256 x 256 images)
        dict(name="windows_8x8_shifted_b32", kind="stages", images=32, heads=4, side=8, win=8,
             n_stages=1, mask="bits", s_delta=0.0048, variant=0),
        # windows of 12 x 12 tokens (384 x 384 images), mask kept as int32 entries
        dict(name="windows_12x12_shifted_b16", kind="stages", images=16, heads=4, side=8, win=12,
             n_stages=1, mask="int32", s_delta=0.012, variant=1),
        # 20 x 20 tokens and a class token, scores requantized in front, codes p - 128 for a signed
        # 8-bit product with V
        dict(name="vit_b_401_requant_front_b32", kind="rows", rows=32 * 12 * 401, cols=401,
             s_delta=2.0 ** -4, variant=1, form="minus128", pre=True, offset=0),
        # the second-degree exponential (the degree ablation), 14 x 14 tokens without a class token
        dict(name="degree2_196_b64", kind="rows", rows=64 * 12 * 196, cols=196, s_delta=0.0057,
             variant=2, form="int8", pre=False, offset=0),
        # global attention over a 64 x 64 token map and a class token
        dict(name="global_attention_4097", kind="rows", rows=12 * 4097, cols=4097, s_delta=0.0033,
             variant=1, form="uint8", pre=False, offset=0),
        # a block of queries against a 224 x 224 map, every position a token
        dict(name="dense_map_50176", kind="rows", rows=2048, cols=224 * 224, s_delta=0.0083,
             variant=1, form="uint8", pre=False, offset=0),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    s_delta = _log_uniform(rng, 2.0 ** -10, 2.0 ** -4)
    s_in = _log_uniform(rng, 2.0 ** -10, 2.0 ** -4)
    variant = rng.choice((0, 0, 1, 1, 2))
    kind = rng.choice(("block", "rows", "rows", "rows", "stages", "stages", "stages", "layers", "gelu", "mlp"))
    if kind == "block":
        return dict(kind=kind, images=rng.randint(1, 16), heads=rng.choice((3, 6, 12)),
                    tokens=rng.choice((49, 145, 196, 197, 198, 257, 401, 577)),
                    width=rng.choice((768, 1536, 3072)), s_delta=s_delta, s_in=s_in, variant=min(variant, 1))
    if kind == "rows":
        cols = int(_log_uniform(rng, 4, 65536))
        elements = _log_uniform(rng, 1e5, 5e7)
        pre = cols <= 4097 and rng.random() < 0.3     # 8-bit codes cannot rank longer rows
        return dict(kind=kind, rows=max(1, int(elements / cols)), cols=cols,
                    s_delta=_log_uniform(rng, 2.0 ** -5, 2.0 ** -4) if pre else s_delta, variant=variant,
                    form=rng.choice(("uint8", "int8", "minus128")), pre=pre,
                    offset=rng.choice((0, 0, 0, 1, 2, 3)))
    if kind == "stages":
        win = rng.randint(5, 16)
        side = rng.randint(2, 8)
        heads = rng.choice((2, 3, 4, 6, 8, 16))
        per_image = heads * (side * win * win) ** 2
        images = int(_log_uniform(rng, 1, 64))
        return dict(kind=kind, images=max(1, min(images, int(5e7 / per_image))), heads=heads, side=side, win=win,
                    n_stages=1, mask=rng.choice(("none", "int32", "bits", "bits")), s_delta=s_delta, variant=variant)
    if kind == "layers":
        cols = rng.choice((49, 145, 196, 197, 257, 577))
        rows = max(1, int(_log_uniform(rng, 1e5, 4e6) / cols))
        return dict(kind=kind, n_layers=rng.randint(2, 12), rows=rows, cols=cols,
                    width=rng.choice((384, 768, 1536)), s_delta=s_delta, s_in=s_in)
    if kind == "gelu":
        return dict(kind=kind, n=int(_log_uniform(rng, 1e5, 7e7)), s_in=s_in, variant=min(variant, 1))
    return dict(kind=kind, tokens=int(_log_uniform(rng, 100, 25000)), width=rng.choice((384, 768, 1536)),
                dim=rng.choice((96, 192, 384)), s_in=s_in, variant=min(variant, 1))


def work(case):
    """Every score, code and table entry read once, every output byte written once; integer
    arithmetic only, so no floating-point operations."""
    k = case["kind"]
    if k == "block":
        n = case["images"] * case["heads"] * case["tokens"] ** 2
        b = 5 * n + 2 * case["images"] * case["tokens"] * case["width"]
    elif k == "rows":
        b = 5 * case["rows"] * case["cols"]
    elif k == "stages":
        b = 0
        for side, heads, tokens, masked in _stages(case):
            b += 5 * case["images"] * side * side * heads * tokens * tokens + 4 * heads * tokens * tokens
            if masked and case["mask"] != "none":
                b += side * side * tokens * (4 * tokens if case["mask"] == "int32" else 8 * _words(tokens))
    elif k == "layers":
        b = case["n_layers"] * (5 * case["rows"] * case["cols"] + 2 * case["rows"] * case["width"])
    elif k == "gelu":
        b = 2 * case["n"]
    else:
        b = 5 * case["tokens"] * (case["width"] + case["dim"])
    return {"bytes": b, "flops": 0}


def tolerance(case):
    return "exact"


# ----------------------------------------------------------------------------- inputs
def _words(tokens):
    return (tokens + 63) // 64


def _stages(case):
    """(windows per side, heads, tokens of a window, whether the shifted mask applies) of each stage:
    the map halves and the heads double from stage to stage; a map of one window has no mask."""
    return [(case["side"] >> s, case["heads"] << s, case["win"] ** 2, (case["side"] >> s) > 1)
            for s in range(case["n_stages"])]


def _scores(gen, rows, cols, head_dim=64):
    """int32 [rows, cols]: products of int8 queries and keys, round(N(0, 25)) (exact in float32:
    every partial sum is an integer below 2^24), one pair of factors per attention matrix."""
    q_rows = min(rows, cols)
    lead = -(-rows // q_rows)
    q = (torch.randn((lead, q_rows, head_dim), device="cuda", generator=gen) * 25).round().clamp(-127, 127)
    k = (torch.randn((lead, head_dim, cols), device="cuda", generator=gen) * 25).round().clamp(-127, 127)
    s = torch.empty((lead * q_rows, cols), dtype=torch.int32, device="cuda")
    step = max(1, int(2e8) // (q_rows * cols))
    for a in range(0, lead, step):
        part = torch.bmm(q[a:a + step], k[a:a + step])
        s[a * q_rows:a * q_rows + part.shape[0] * q_rows] = part.view(-1, cols)
    return s[:rows]


def _codes(gen, n):
    """int8 activations with long tails: 0.9 N(0, 20) + 0.1 Laplace(0, 60)."""
    x = torch.randn(n, device="cuda", generator=gen) * 20
    u = torch.rand(n, device="cuda", generator=gen) - 0.5
    tail = -60 * torch.sign(u) * torch.log1p(-2 * u.abs() + 1e-6)
    x = torch.where(torch.rand(n, device="cuda", generator=gen) < 0.1, tail, x)
    return x.round().clamp(-127, 127).to(torch.int8)


def _accumulators(gen, n):
    return (torch.randn(n, device="cuda", generator=gen) * 30000).round().to(torch.int32)


def _gelu_range(s_in):
    """Output quantizer over the GELU's range on int8 inputs: (s_out, zp_out)."""
    v = [0.5 * s_in * q * (1 + math.erf(s_in * q / math.sqrt(2))) for q in range(-128, 128)]
    s_out = (max(v) - min(v)) / 255
    return s_out, int(round(-128 - min(v) / s_out))


def _shifted_mask(side, win):
    """int32 [windows, win^2, win^2]: 0 where query and key were neighbours before the shift by half
    a window, INT32_MIN elsewhere."""
    n, shift = side * win, win // 2
    at = torch.arange(n, device="cuda")
    region = (at >= n - win).long() + (at >= n - shift).long()
    region = region[:, None] * 3 + region[None, :]
    r = region.view(side, win, side, win).permute(0, 2, 1, 3).reshape(side * side, win * win)
    return torch.where(r[:, :, None] == r[:, None, :], 0, I32_MIN).to(torch.int32)


def _softmax_params(case, cols, variant=None):
    form = case.get("form", "uint8")
    p = ip.softmax_prepare(case["s_delta"], cols, case["variant"] if variant is None else variant,
                           0 if form == "uint8" else 1)
    if form == "minus128":
        p.post = ip.Dyadic(1, 0, -128, -128, 127)
    if case.get("pre"):
        p.pre_m, p.pre_s = 20000, 21              # scores of about +-15000 to 8-bit codes
    return p


def _gelu_params(case, max_abs_q, variant=None, pre=False):
    s_out, zp = _gelu_range(case["s_in"])
    p = ip.gelu_prepare(case["s_in"], s_out, 0, zp, case["variant"] if variant is None else variant, max_abs_q)
    if pre:
        p.pre_m, p.pre_s = 20000, 24
    return p


def _requant_params():
    return ip.Dyadic(20480, 25, 0, -128, 127)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    k = case["kind"]
    st = dict(case=case)
    if k == "block":
        st["rows"] = case["images"] * case["heads"] * case["tokens"]
        st["n"] = case["images"] * case["tokens"] * case["width"]
        st["scores"] = _scores(gen, st["rows"], case["tokens"])
        st["probs"] = torch.empty((st["rows"], case["tokens"]), dtype=torch.uint8, device="cuda")
        st["x"] = _codes(gen, st["n"])
        st["y"] = torch.empty(st["n"], dtype=torch.int8, device="cuda")
        st["sp"], st["gp"] = _softmax_params(case, case["tokens"]), _gelu_params(case, 255)
    elif k == "rows":
        n, off = case["rows"] * case["cols"], case["offset"]
        scores = _scores(gen, case["rows"], case["cols"])
        if off:                                       # a view into a larger tensor, off the 16-byte grid
            larger = torch.zeros(n + 4, dtype=torch.int32, device="cuda")
            larger[off:off + n] = scores.view(-1)
            scores = larger[off:off + n].view(case["rows"], case["cols"])
        st["scores"] = scores
        st["probs"] = torch.empty(n + 4, dtype=torch.uint8 if case["form"] == "uint8" else torch.int8,
                                  device="cuda")[off:off + n].view(case["rows"], case["cols"])
        st["sp"] = _softmax_params(case, case["cols"])
    elif k == "stages":
        st["stages"] = []
        for side, heads, tokens, masked in _stages(case):
            rows = case["images"] * side * side * heads * tokens
            bias = (torch.randn((heads * tokens, tokens), device="cuda", generator=gen) * 8).round().to(torch.int32)
            mask = _shifted_mask(side, case["win"]) if masked and case["mask"] != "none" else None
            bits = None
            if mask is not None and case["mask"] == "bits":
                bits = torch.empty((side * side, tokens, _words(tokens)), dtype=torch.int64, device="cuda")
                ip.pack_window_mask(mask, side * side, tokens, bits)
            st["stages"].append(dict(
                rows=rows, windows=side * side, heads=heads, tokens=tokens, bias=bias, mask=mask, bits=bits,
                scores=_scores(gen, rows, tokens, 32), sp=_softmax_params(case, tokens),
                probs=torch.empty((rows, tokens), dtype=torch.uint8, device="cuda")))
    elif k == "layers":
        n, rows, cols = case["n_layers"], case["rows"], case["cols"]
        st["scores"] = _scores(gen, n * rows, cols)
        st["probs"] = torch.empty((n * rows, cols), dtype=torch.uint8, device="cuda")
        st["x"] = _codes(gen, n * rows * case["width"])
        st["y"] = torch.empty(n * rows * case["width"], dtype=torch.int8, device="cuda")
        st["sps"] = [_softmax_params(case, cols, layer % 2) for layer in range(n)]
        st["gps"] = [_gelu_params(case, 255, layer % 2) for layer in range(n)]
    elif k == "gelu":
        st["x"] = _codes(gen, case["n"])
        st["y"] = torch.empty(case["n"], dtype=torch.int8, device="cuda")
        st["gp"] = _gelu_params(case, 255)
    else:
        st["acc1"] = _accumulators(gen, case["tokens"] * case["width"])
        st["acc2"] = _accumulators(gen, case["tokens"] * case["dim"])
        st["hidden"] = torch.empty(case["tokens"] * case["width"], dtype=torch.int8, device="cuda")
        st["codes"] = torch.empty(case["tokens"] * case["dim"], dtype=torch.int8, device="cuda")
        st["gp"], st["rp"] = _gelu_params(case, 127, pre=True), _requant_params()
    return st


# ----------------------------------------------------------------------------- one pass
def run(st):
    case = st["case"]
    k = case["kind"]
    if k == "block":
        ip.softmax_i32(st["scores"], None, 0, st["probs"], st["rows"], case["tokens"], st["sp"])
        ip.gelu_i8(st["x"], st["y"], st["n"], st["gp"])
        return st["probs"], st["y"]
    if k == "rows":
        ip.softmax_i32(st["scores"], None, 0, st["probs"], case["rows"], case["cols"], st["sp"])
        return st["probs"]
    if k == "stages":
        for s in st["stages"]:
            period = s["heads"] * s["tokens"]
            if s["bits"] is not None:
                ip.softmax_i32_windowed_bits(s["scores"], s["bias"], period, s["bits"], s["windows"], s["heads"],
                                             s["probs"], s["rows"], s["tokens"], s["sp"])
            elif s["mask"] is not None:
                ip.softmax_i32_windowed(s["scores"], s["bias"], period, s["mask"], s["windows"], s["heads"],
                                        s["probs"], s["rows"], s["tokens"], s["sp"])
            else:
                ip.softmax_i32(s["scores"], s["bias"], period, s["probs"], s["rows"], s["tokens"], s["sp"])
        return [s["probs"] for s in st["stages"]]
    if k == "layers":
        n, el, width = case["n_layers"], case["rows"] * case["cols"], case["rows"] * case["width"]
        ip.softmax_i32_layers(st["scores"], el, st["probs"], el, case["rows"], case["cols"], n, st["sps"])
        ip.gelu_i8_layers(st["x"], width, st["y"], width, width, n, st["gps"])
        return st["probs"], st["y"]
    if k == "gelu":
        ip.gelu_i8(st["x"], st["y"], case["n"], st["gp"])
        return st["y"]
    ip.gelu_i32(st["acc1"], st["hidden"], case["tokens"] * case["width"], st["gp"])
    ip.requant(st["acc2"], st["codes"], case["tokens"] * case["dim"], 1, st["rp"])
    return st["hidden"], st["codes"]


# ----------------------------------------------------------------------------- the same in 64 bits
def _exact_softmax(scores, s_delta, variant, form="uint8", pre=False, tables=()):
    """The steps of the softmax in int64, a few million scores at a time.  tables: functions from
    the row indices to [rows, cols] additive entries; INT32_MIN anywhere is minus infinity."""
    rows, cols = scores.shape
    i0 = int(math.floor(1.0 / s_delta))
    n = max(0, 15 - i0.bit_length())
    while n > 0 and cols * (i0 << n) > 1 << 30:
        n -= 1
    out = torch.empty((rows, cols), dtype=torch.uint8 if form == "uint8" else torch.int8, device=scores.device)
    step = max(1, int(8e6) // cols)
    for a in range(0, rows, step):
        x = scores[a:a + step].long()
        r = torch.arange(a, a + x.shape[0], device=x.device)
        masked = x == I32_MIN
        for table in tables:
            t = table(r)
            masked |= t == I32_MIN
            x = (x + t).clamp(I32_MIN, 2 ** 31 - 1)
        if pre:
            x = (x * 20000 + (1 << 20)) >> 21
        x = torch.where(masked, I32_MIN, x)
        d = (x - x.max(dim=1, keepdim=True).values).clamp(min=-(1 << 30))
        m = -(d + (d >> 1) - (d >> 4))
        q = torch.div(m, i0, rounding_mode="floor")
        f = -(m - q * i0)
        y = f >> 1
        if variant >= 1:
            y = y + (f >> 3) + (f >> 4)
        if variant == 2:
            y = y + torch.div(y * y, 2 * i0, rounding_mode="floor")
        e = torch.where(masked | (q >= 32), 0, ((i0 + y) << n) >> q.clamp(max=32))
        total = e.sum(dim=1, keepdim=True)
        factor = torch.where(total > 0, torch.div(torch.full_like(total, 1 << 30), total.clamp(min=1),
                                                  rounding_mode="floor"), 0)
        p = (factor * e) >> 23
        if form == "int8":
            p = p.clamp(max=127)
        elif form == "minus128":
            p = p - 128
        out[a:a + step] = p.to(out.dtype)
    return out


def _exact_gelu(codes, s_in, variant, max_abs_q):
    """The polynomial GELU of centred codes in int64 with constants from the real scales."""
    s_out, zp = _gelu_range(s_in)
    p, a, b = (4, -0.019913, -2.698088) if variant else (2, -0.2888, -1.769)
    s_e = s_in / math.sqrt(2.0)
    sq = s_e * s_e
    s_l = a * (sq if p == 2 else sq * sq)
    q_b, q_c = int(math.floor(b / s_e)), int(math.floor(1.0 / s_l))
    top, k = (-q_b) ** p + 2 * -q_c, 0
    while k < 62 and -(-top >> k) * max_abs_q >= 1 << 31:
        k += 1
    ratio = ((s_in * s_l) * 2.0 ** k / 2.0) / s_out
    frac, e = math.frexp(abs(ratio))
    m, s = int(math.floor(frac * 32768 + 0.5)), 15 - e
    if m == 32768:
        m, s = 16384, s - 1
    if s > 62:
        m, s = int(math.floor(math.ldexp(abs(ratio), 62) + 0.5)), 62
    m = -m if ratio < 0 else m
    # one value per distinct input, then a gather
    q = torch.arange(-max_abs_q, max_abs_q + 1, device=codes.device)
    t = q.abs().clamp(max=-q_b) + q_b
    u = t * t
    u = (u * u if p == 4 else u) + q_c
    v = (torch.sign(q) * u + q_c) >> k
    y = (((q * v * m + ((1 << s) >> 1)) >> s) + zp).clamp(-128, 127).to(torch.int8)
    out = torch.empty(codes.shape, dtype=torch.int8, device=codes.device)
    step = int(3e7)
    for i in range(0, codes.numel(), step):
        out[i:i + step] = y[codes[i:i + step].long().clamp(-max_abs_q, max_abs_q) + max_abs_q]
    return out


def exact(case, seed):
    st = prepare(case, seed)
    k = case["kind"]
    if k == "block":
        return (_exact_softmax(st["scores"], case["s_delta"], case["variant"]),
                _exact_gelu(st["x"], case["s_in"], case["variant"], 255))
    if k == "rows":
        return _exact_softmax(st["scores"], case["s_delta"], case["variant"], case["form"], case["pre"])
    if k == "stages":
        outs = []
        for s in st["stages"]:
            heads, tokens, windows = s["heads"], s["tokens"], s["windows"]
            tables = [lambda r, b=s["bias"].long(): b[r % b.shape[0]]]
            if s["mask"] is not None:
                tables.append(lambda r, m=s["mask"].long(), h=heads, t=tokens, w=windows:
                              m[(r // (h * t)) % w, r % t])
            outs.append(_exact_softmax(s["scores"], case["s_delta"], case["variant"], tables=tables))
        return outs
    if k == "layers":
        n, rows, width = case["n_layers"], case["rows"], case["rows"] * case["width"]
        return (torch.cat([_exact_softmax(st["scores"][i * rows:(i + 1) * rows], case["s_delta"], i % 2)
                           for i in range(n)]),
                torch.cat([_exact_gelu(st["x"][i * width:(i + 1) * width], case["s_in"], i % 2, 255)
                           for i in range(n)]))
    if k == "gelu":
        return _exact_gelu(st["x"], case["s_in"], case["variant"], 255)
    codes = (st["acc1"].long() * 20000 + (1 << 23)) >> 24
    r = (((st["acc2"].long() * 20480 + (1 << 24)) >> 25)).clamp(-128, 127).to(torch.int8)
    return _exact_gelu(codes, case["s_in"], case["variant"], 127), r
