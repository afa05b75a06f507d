"""The work that a program has this library do, as timed cases: fused MLP chains (include/ogc_mlp.h) and the fused
attention subgraph (include/ogc_mha.h), each through its public entry point on tensors that are already in HBM.

A case is a dict of plain values.  kind "mlp": dtype, m (batch rows), dims (layer widths, "13-64-32-16"), acts (one
letter a layer: n none, r ReLU, g GELU, s sigmoid), bias, residual, in_zp (zero point of the u8 input), out_f32 (a
quantized chain's last layer gives fp32).  An E4M3 chain ("f8") starts from fp32 rows and ends in them: the quantize and
dequantize nodes at the boundary of a low-precision graph are part of the pass.  kind "mha": dtype, batch, heads, seq,
head_dim, mask (padding mask), softmax, layout ("bshd": what a projection leaves, "bhsd": one block per head).
"""
import math

import torch

from paper_2301_01333_amd import binding

ACT = {"n": binding.OGC_ACT_NONE, "r": binding.OGC_ACT_RELU, "g": binding.OGC_ACT_GELU_TANH, "s": binding.OGC_ACT_SIGMOID}
TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "i8": torch.uint8, "f8": torch.uint8}
SIZE = {"f32": 4, "bf16": 2, "i8": 1, "f8": 1}


def _mlp(dtype, m, dims, acts, bias=True, residual=False, in_zp=128, out_f32=False, **more):
    return dict(more, kind="mlp", dtype=dtype, m=m, dims=dims, acts=acts, bias=bias, residual=residual, in_zp=in_zp,
                out_f32=out_f32)


def _mha(dtype, batch, heads, seq, head_dim, mask=True, softmax="stable", layout="bshd", **more):
    return dict(more, kind="mha", dtype=dtype, batch=batch, heads=heads, seq=seq, head_dim=head_dim, mask=mask, softmax=softmax,
                layout=layout)


def listed():
    top = "479-1024-1024-512-256-1"
    return [
        # the smallest chain there is: one launch, all latency
        _mlp("f32", 32, "13-64-32-16", "rrr", name="mlp_f32_b32"),
        # a recommendation model's bottom MLP on an online batch
        _mlp("bf16", 128, "13-512-256-128-64", "rrrr", name="mlp_bf16_b128"),
        # its top MLP, quantized, online batch: 479 features (rows that are not 16-byte aligned), one probability out
        _mlp("i8", 256, top, "rrrrs", out_f32=True, name="top_mlp_i8_b256"),
        # the same in fp32 at the largest batch of the paper's Table I
        _mlp("f32", 512, top, "rrrrn", name="top_mlp_f32_b512"),
        # the same, quantized, scoring offline: a large batch of odd size
        _mlp("i8", 8191, top, "rrrrs", out_f32=True, name="top_mlp_i8_b8191"),
        # a transformer's feed-forward block in bf16 with its residual, 32 sequences of 128 tokens
        _mlp("bf16", 4096, "1024-4096-1024", "gn", residual=True, name="ffn_bf16_t4096"),
        # the compute-bound quantized chain: the largest of all
        _mlp("i8", 32768, "1024-1024-1024-1024-1024", "rrrr", bias=False, name="mlp_i8_b32768"),
        # an 8-bit-float chain between fp32 neighbours: quantize, four layers, dequantize
        _mlp("f8", 8192, "1024-1024-1024-1024-1024", "rrrr", name="mlp_f8_b8192"),
        # attention of a BERT-large encoder (Table I, MHA-4) in fp32, a serving batch
        _mha("f32", 32, 16, 512, 64, name="mha_f32_s512_b32"),
        # the same in bf16 at the largest batch of Table I
        _mha("bf16", 128, 16, 512, 64, name="mha_bf16_s512_b128"),
        # quantized attention with wide heads (Table I, MHA-3), largest batch
        _mha("i8", 128, 8, 384, 128, name="mha_i8_s384_b128"),
        # a small batch of an odd length (an image encoder's patches and class token): no mask, one block per head
        _mha("bf16", 8, 12, 197, 64, mask=False, layout="bhsd", name="mha_bf16_s197_b8"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    if rng.random() < 0.4:
        dtype = rng.choice(["f32", "bf16", "i8"])
        head_dim, heads, seq = rng.choice([32, 64, 96, 128]), rng.choice([4, 8, 12, 16]), _log_int(rng, 48, 1024)
        if rng.random() < 0.4:
            seq = max(64, seq // 64 * 64)
        # operations of both products at most: what the listed attention cases take about a millisecond for
        most = {"f32": 3.4e10, "bf16": 1.3e11, "i8": 7.0e10}[dtype]
        cap = max(1, min(128, int(most / (4.0 * heads * seq * seq * head_dim))))
        softmax = "fast" if dtype != "i8" and rng.random() < 0.25 else "stable"
        return _mha(dtype, _log_int(rng, 1, cap), heads, seq, head_dim, rng.random() < 0.6, softmax, rng.choice(["bshd", "bshd", "bhsd"]))
    dtype = rng.choice(["f32", "bf16", "i8", "i8", "f8"])
    quant = dtype in ("i8", "f8")
    shape = rng.choice(["bottom", "top", "ffn", "square", "free"])
    residual, out_f32, in_zp, bias = False, False, 128, True
    if shape == "bottom":
        dims, acts = [13, 512, 256, 128] + [64] * rng.randrange(2), None
    elif shape == "top":
        dims, acts = [479, 1024, 1024, 512, 256, 1], "rrrrs" if quant else "rrrrn"
        out_f32 = quant
    elif shape == "ffn":
        h = rng.choice([256, 384, 512, 768, 1024])
        dims, acts, residual = [h, 4 * h, h], "gn", not quant
    elif shape == "square":
        dims, acts, bias = [rng.choice([256, 512, 1024])] * rng.randrange(3, 6), None, rng.random() < 0.5
    else:
        dims, acts = [_log_int(rng, 16, 1536) for _ in range(rng.randrange(3, 6))], None
        in_zp = 128 if rng.random() < 0.7 else rng.randrange(256)
    acts = acts or "r" * (len(dims) - 1)
    per_row = 2.0 * sum(a * b for a, b in zip(dims, dims[1:]))
    most = {"f32": 3.4e10, "bf16": 1.0e11, "i8": 1.3e11, "f8": 1.3e11}[dtype]
    m = _log_int(rng, 1, max(1, min(32768, int(most / per_row))))
    if m > 64 and rng.random() < 0.5:
        m = m // 32 * 32
    return _mlp(dtype, m, "-".join(str(d) for d in dims), acts, bias, residual, in_zp if dtype == "i8" else 128, out_f32)


# ---- inputs ---------------------------------------------------------------------------------------------------------
def _dims(case):
    return [int(v) for v in case["dims"].split("-")]


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _gen(seed):
    return torch.Generator(device=_device()).manual_seed(int(seed))


def _normal(g, shape, std=1.0):
    return torch.randn(shape, generator=g, device=g.device, dtype=torch.float32) * std


def _uniform(g, shape, lo, hi):
    return torch.rand(shape, generator=g, device=g.device, dtype=torch.float32) * (hi - lo) + lo


def _f32(v):
    return float(torch.tensor(v, dtype=torch.float32))


def _mlp_inputs(case, seed):
    """x, weights [K,N], biases, per-channel weight scales and the layers' descriptions."""
    g, dims, dtype = _gen(seed), _dims(case), case["dtype"]
    last = len(dims) - 2
    if dtype == "i8":
        x = torch.randint(0, 256, (case["m"], dims[0]), generator=g, device=g.device, dtype=torch.uint8)
    elif dtype == "f8":
        x = _normal(g, (case["m"], dims[0]))
    else:
        x = _normal(g, (case["m"], dims[0]), 1.0 / math.sqrt(dims[0]) if dtype == "f32" else 1.0).to(TORCH[dtype])
    ws, bs, scales, layers = [], [], [], []
    # static activation scales from the distributions alone: three (u8) or four (E4M3) standard deviations of the
    # pre-activation on the largest code
    in_scale = 0.05 if dtype == "i8" else _f32(4.0 / 448.0)
    in_zp = case["in_zp"] if dtype == "i8" else 0
    var = in_scale ** 2 * ((256.0 ** 2 - 1) / 12.0 + (127.5 - in_zp) ** 2) if dtype == "i8" else 1.0
    for l, (k, n) in enumerate(zip(dims, dims[1:])):
        f32_out = case["out_f32"] and l == last
        scale = None
        if dtype == "i8":
            w = torch.randint(-127, 128, (k, n), generator=g, device=g.device, dtype=torch.int8)
            scale = _uniform(g, (n,), 0.005, 0.02)
            var = var * k * (127.0 * 128.0 / 3.0) * (0.005 ** 2 + 0.005 * 0.02 + 0.02 ** 2) / 3.0
            out_scale, out_zp = _f32(3.0 * math.sqrt(var) / 127.0), 128
        elif dtype == "f8":
            wf = _normal(g, (k, n), 1.0 / math.sqrt(k))
            scale = wf.abs().amax(0) / 448.0
            w = _e4m3_codes(wf / scale)
            out_scale, out_zp = _f32(4.0 * math.sqrt(var) / 448.0), 0
        else:
            std = 0.02 if "g" in case["acts"] else 1.0 / math.sqrt(k)
            w = _normal(g, (k, n), std).to(TORCH[dtype])
            out_scale, out_zp = 0.0, 0
        if case["acts"][l] == "r":
            var = var / 2.0
        ws.append(w)
        bs.append(_uniform(g, (n,), -0.1, 0.1) if case["bias"] else None)
        scales.append(scale)
        layers.append(dict(k=k, n=n, has_bias=int(case["bias"]), act=ACT[case["acts"][l]], in_scale=in_scale, in_zp=in_zp,
                           out_scale=1.0 if f32_out else out_scale, out_zp=0 if f32_out else out_zp,
                           out=binding.OGC_OUT_F32 if f32_out else binding.OGC_OUT_SAME))
        in_scale, in_zp = out_scale, out_zp
    return x, ws, bs, scales, layers


def _mha_inputs(case, seed):
    """q, k, v (in memory order of the layout), the padding mask or None, the quantization scales or None."""
    g = _gen(seed)
    b, h, s, d = case["batch"], case["heads"], case["seq"], case["head_dim"]
    shape = (b, s, h, d) if case["layout"] == "bshd" else (b, h, s, d)
    step = _f32(4.0 / 127.0)
    ts = []
    for _ in range(3):
        t = _normal(g, shape)
        ts.append((t / step).round().clamp(-127, 127).to(torch.int8) if case["dtype"] == "i8" else t.to(TORCH[case["dtype"]]))
    mask = None
    if case["mask"]:  # every sequence of the batch fills at least half of its row
        lens = torch.randint(max(s // 2, 1), s + 1, (b, 1), generator=g, device=g.device)
        pos = torch.arange(s, device=g.device)[None, :]
        mask = torch.where(pos < lens, 0.0, -10000.0).to(torch.float32).contiguous()
    return ts, mask, (step, step, step, _f32(1.0 / 127.0)) if case["dtype"] == "i8" else None


# ---- what a program holds before the call, and the call ----------------------------------------------------------------
def prepare(case, seed):
    if case["kind"] == "mlp":
        x, ws, bs, scales, layers = _mlp_inputs(case, seed)
        dtype, m, n = case["dtype"], case["m"], layers[-1]["n"]
        mlp = binding.FusedMLP(dtype, m, layers, residual=case["residual"])
        mlp.prepack(ws, bs if case["bias"] else None, scales if dtype in ("i8", "f8") else None)
        y = torch.empty((m, n), device="cuda", dtype=torch.float32 if case["out_f32"] else TORCH[dtype])
        st = dict(kind="mlp", mlp=mlp, x=x, y=y)
        if dtype == "f8":
            st.update(kind="f8", xq=torch.empty((m, layers[0]["k"]), device="cuda", dtype=torch.uint8), in_scale=layers[0]["in_scale"],
                      out_scale=None if case["out_f32"] else layers[-1]["out_scale"],
                      yf=None if case["out_f32"] else torch.empty((m, n), device="cuda", dtype=torch.float32))
        torch.cuda.synchronize()  # the raw weights go out of scope here
        return st
    (q, k, v), mask, quant = _mha_inputs(case, seed)
    b, h, s, d = case["batch"], case["heads"], case["seq"], case["head_dim"]
    stride = (s * h * d, d, h * d) if case["layout"] == "bshd" else (h * s * d, s * d, d)
    desc = binding.mha_desc(binding.DTYPES[case["dtype"]], b, h, s, d, _f32(1.0 / math.sqrt(d)),
                            binding.OGC_SOFTMAX_FAST if case["softmax"] == "fast" else binding.OGC_SOFTMAX_STABLE,
                            stride, stride, stride, stride)
    return dict(kind="mha8" if quant else "mha", desc=desc, q=q, k=k, v=v, mask=mask, o=torch.empty_like(q),
                quant=binding.ogc_mha_quant(*quant) if quant else None)


def run(st):
    if st["kind"] == "mlp":
        st["mlp"].run(st["x"], st["y"])
        return st["y"]
    stream = int(torch.cuda.current_stream().cuda_stream)
    if st["kind"] == "f8":
        binding.ogc_quantize_e4m3(st["x"].data_ptr(), st["xq"].data_ptr(), st["x"].numel(), st["in_scale"], stream)
        st["mlp"].run(st["xq"], st["y"])
        if st["yf"] is None:
            return st["y"]
        binding.ogc_dequantize_e4m3(st["y"].data_ptr(), st["yf"].data_ptr(), st["y"].numel(), st["out_scale"], stream)
        return st["yf"]
    mask = st["mask"].data_ptr() if st["mask"] is not None else 0
    args = (st["q"].data_ptr(), st["k"].data_ptr(), st["v"].data_ptr(), mask, st["o"].data_ptr(), stream)
    if st["kind"] == "mha8":
        binding.ogc_mha_run_i8(st["desc"], st["quant"], *args)
    else:
        binding.ogc_mha_run(st["desc"], *args)
    return st["o"]


def work(case):
    """Each input read once, each output written once; the activations between layers and the attention scores count
    nothing."""
    e = SIZE[case["dtype"]]
    if case["kind"] == "mha":
        b, h, s, d = case["batch"], case["heads"], case["seq"], case["head_dim"]
        return {"bytes": 4 * b * s * h * d * e + (4 * b * s if case["mask"] else 0), "flops": 4 * b * h * s * s * d}
    dims, m = _dims(case), case["m"]
    pairs = list(zip(dims, dims[1:]))
    ends = 4 if case["dtype"] == "f8" else e  # E4M3 chains: fp32 rows on both sides
    params = sum(n for _, n in pairs) * (4 * bool(case["bias"]) + (4 if case["dtype"] in ("i8", "f8") else 0))
    return {"bytes": e * sum(k * n for k, n in pairs) + params + m * dims[0] * ends + m * dims[-1] * (4 if case["out_f32"] else ends),
            "flops": 2 * m * sum(k * n for k, n in pairs)}


def tolerance(case):
    dtype = case["dtype"]
    if case["kind"] == "mha":
        if dtype == "i8":  # a numerator within rounding error of a tie moves a byte by one step
            return {"rel": 0.0, "differ": 0.01}
        return {"rel": 1e-5} if dtype == "f32" else {"rel": 1e-2}
    if dtype == "i8":
        # integer sums and one order of fp32 operations: bytes are the same, a probability within its exponential's
        # error; a GELU that is not evaluated the same moves a byte at a rounding boundary
        return {"rel": 1e-5} if case["out_f32"] else ({"rel": 0.0, "differ": 0.01} if "g" in case["acts"] else "exact")
    # E4M3: the order of the sums moves a code at a rounding boundary, one code is 6 %
    return {"rel": {"f32": 1e-5, "bf16": 1e-2, "f8": 2e-2}[dtype]}


# ---- the same results in 64 bits ---------------------------------------------------------------------------------------
def _e4m3_codes(t):
    return t.clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)


def _e4m3_values(codes):
    return codes.view(torch.float8_e4m3fn).to(torch.float32).double()


def _act(y, act):
    if act == "r":
        return y.clamp(min=0.0)
    if act == "g":
        return 0.5 * y * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (y + 0.044715 * y ** 3)))
    return torch.sigmoid(y) if act == "s" else y


def _exact_mlp(case, seed):
    x, ws, bs, scales, layers = _mlp_inputs(case, seed)
    dtype = case["dtype"]
    if dtype in ("f32", "bf16"):
        y = x.double()
        for w, b, act in zip(ws, bs, case["acts"]):
            y = y @ w.double()
            y = _act(y + b.double() if b is not None else y, act)
        return y + x.double() if case["residual"] else y
    # quantized: the codes between the layers are part of the definition, and so is the fp32 arithmetic that decides them
    codes = x if dtype == "i8" else _e4m3_codes(x * (1.0 / torch.tensor(layers[0]["in_scale"], dtype=torch.float32, device=x.device)))
    for w, b, s, ly, act in zip(ws, bs, scales, layers, case["acts"]):
        vals = codes.double() - ly["in_zp"] if dtype == "i8" else _e4m3_values(codes)
        acc = (vals @ (w.double() if dtype == "i8" else _e4m3_values(w))).float()
        comb = (torch.tensor(ly["in_scale"], dtype=torch.float32, device=x.device) * s).double()
        y = acc.double() * comb + (b.double() if b is not None else 0.0)
        if ly["out"] == binding.OGC_OUT_F32:
            return _act(y, act)
        t = _act(y.float().double(), act).float() * (1.0 / torch.tensor(ly["out_scale"], dtype=torch.float32, device=x.device))
        codes = (t.round() + ly["out_zp"]).clamp(0, 255).to(torch.uint8) if dtype == "i8" else _e4m3_codes(t)
    return codes if dtype == "i8" else _e4m3_values(codes) * layers[-1]["out_scale"]


def _exact_mha(case, seed):
    (q, k, v), mask, quant = _mha_inputs(case, seed)
    out = torch.empty(q.shape, device=q.device, dtype=torch.float64)
    scale = _f32(1.0 / math.sqrt(case["head_dim"]))
    for i in range(case["batch"]):
        for j in range(case["heads"]):
            at = (i, slice(None), j) if case["layout"] == "bshd" else (i, j)
            s = q[at].double().contiguous() @ k[at].double().t().contiguous()
            s = s * (scale * quant[0] * quant[1] if quant else scale)
            if mask is not None:
                s = s + mask[i].double()
            p = torch.exp(s - s.amax(1, keepdim=True))
            if quant:
                p = (127.0 * p).round()
                out[at] = ((p @ v[at].double().contiguous()).float() / p.sum(1, keepdim=True).float()).double() * (quant[2] / quant[3])
            else:
                out[at] = (p / p.sum(1, keepdim=True)) @ v[at].double().contiguous()
    return out.round().clamp(-128, 127).to(torch.int8) if quant else out


def exact(case, seed):
    return _exact_mlp(case, seed) if case["kind"] == "mlp" else _exact_mha(case, seed)
