"""Workloads of the multi-bitwidth additive-codebook linear layer, for timing.

Each case is something a program does with a quantized model on one GPU: decode steps over the
linear layers of a few transformer blocks (recorded once in a HIP graph, as a serving loop does),
single layers called eagerly at token counts from one row to a long prompt, explicit
dequantization, and the quantizer's two data-parallel pieces (prefix distortions and the code
search). Inputs are synthetic, drawn on the GPU from the seed: N(0, 1) activations with 0.1 % of
the entries 20 times larger, uniform codes, codebooks that add up to weights of standard deviation
0.02, scales U(0.5, 1.5).

``exact`` is the same arithmetic in plain torch in 64 bits: the product with the exactly rebuilt
weights, and the same search with every error in 64 bits.
"""
import math

import torch

import paper_2606_12876_amd as aq

_DT = {"fp16": torch.float16, "bf16": torch.bfloat16, "fp32": torch.float32}
_AQ = {"fp16": aq.DType.F16, "bf16": aq.DType.BF16, "fp32": aq.DType.F32}


def listed():
    return [
        # the smallest call: one 1024 x 1024 projection, one row, eager (latency of a call)
        dict(name="linear_1row_1024", op="linear", d_out=1024, d_in=1024, bits=8, M=4, k=4, n=1, dtype="fp16"),
        # single-stream decoding of a 7B-class model: q/k/v, o, gate/up, down of four blocks
        dict(name="decode_b1", op="decode", hidden=4096, kv=4096, ffn=11008, blocks=4, bits=8, M=4, k=4, batch=1,
             dtype="bf16"),
        # batched decoding at a lower precision level, an odd number of streams
        dict(name="decode_b11", op="decode", hidden=4096, kv=4096, ffn=11008, blocks=4, bits=8, M=4, k=3, batch=11,
             dtype="bf16"),
        # decoding with the large-codebook format (2^16 codewords per book), one row
        dict(name="linear_1row_16bit", op="linear", d_out=14336, d_in=4096, bits=16, M=2, k=2, n=1, dtype="fp16"),
        # one decode step of 64 streams through a square projection
        dict(name="linear_64rows", op="linear", d_out=4096, d_in=4096, bits=8, M=4, k=4, n=64, dtype="bf16"),
        # a chunk of a prompt (or speculative tokens of many streams) of ragged length through an up projection
        dict(name="linear_333rows", op="linear", d_out=11008, d_in=4096, bits=8, M=4, k=3, n=333, dtype="bf16"),
        # prefill of a 2048-token prompt, with the workspace that such a program keeps
        dict(name="prefill_2048", op="prefill", d_out=4096, d_in=4096, bits=8, M=4, k=4, n=2048),
        # several prompts prefilled together through an up projection, no workspace
        dict(name="linear_8192rows", op="linear", d_out=11008, d_in=4096, bits=8, M=4, k=2, n=8192, dtype="bf16"),
        # explicit weights of a down projection
        dict(name="dequant_down", op="dequant", d_out=4096, d_in=11008, bits=8, M=4, k=4, dtype="bf16"),
        # quality of every prefix of a quantized layer over 1024 calibration inputs
        dict(name="distortion_1024", op="distortion", d_out=4096, d_in=4096, bits=8, M=4, n=1024),
        # code search for every group of a layer, squared error
        dict(name="beam_4096", op="beam", d_out=4096, d_in=4096, bits=8, k=4, beam=8),
        # data-aware code search of a smaller model's projection, ragged rows
        dict(name="beam_weighted", op="beam_weighted", d_out=2000, d_in=2304, bits=8, k=3, beam=5),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _d8(rng, lo, hi):
    return max(8, 8 * int(round(_log(rng, lo, hi) / 8)))


def draw(rng):
    op = rng.choice(["linear1", "decode", "decode", "wide", "rows", "rows", "prompt", "prefill", "dequant",
                     "distortion", "beam", "beam_weighted"])
    if op == "linear1":
        return dict(op="linear", d_out=_log(rng, 700, 12000), d_in=_d8(rng, 700, 12000), bits=rng.choice([8, 8, 4]),
                    M=4, k=rng.randint(1, 4), n=rng.choice([1, 1, 2, rng.randint(3, 16)]),
                    dtype=rng.choice(["fp16", "bf16"]))
    if op == "decode":
        hidden = _d8(rng, 1024, 4096)
        kv = rng.choice([hidden, max(128, hidden // 32 * 8)])
        return dict(op="decode", hidden=hidden, kv=kv, ffn=8 * int(hidden * rng.uniform(2.5, 3.5) / 8),
                    blocks=rng.randint(2, 4), bits=rng.choice([8, 8, 8, 4]), M=4, k=rng.randint(1, 4),
                    batch=rng.choice([1, 1, rng.randint(2, 16), rng.randint(2, 16)]),
                    dtype=rng.choice(["bf16", "bf16", "fp16"]))
    if op == "wide":
        return dict(op="linear", d_out=_log(rng, 2048, 14336), d_in=_d8(rng, 2048, 8192), bits=16, M=2,
                    k=rng.randint(1, 2), n=rng.choice([1, 1, rng.randint(2, 8)]), dtype=rng.choice(["fp16", "bf16"]))
    if op == "rows":
        return dict(op="linear", d_out=_log(rng, 1024, 11008), d_in=_d8(rng, 1024, 11008),
                    bits=rng.choice([8, 8, 8, 4]), M=4, k=rng.randint(1, 4), n=_log(rng, 17, 1500), dtype="bf16")
    if op == "prompt":
        return dict(op="linear", d_out=_log(rng, 1024, 11008), d_in=_d8(rng, 1024, 4096), bits=8, M=4,
                    k=rng.randint(1, 4), n=_log(rng, 1500, 8000), dtype="bf16")
    if op == "prefill":
        return dict(op="prefill", d_out=_log(rng, 1024, 11008), d_in=_d8(rng, 1024, 4096),
                    bits=rng.choice([8, 8, 8, 4]), M=4, k=rng.randint(1, 4), n=_log(rng, 256, 8000))
    if op == "dequant":
        return dict(op="dequant", d_out=_log(rng, 1024, 11008), d_in=_d8(rng, 1024, 11008),
                    bits=rng.choice([8, 8, 4]), M=4, k=rng.randint(1, 4), dtype=rng.choice(["bf16", "fp16", "fp32"]))
    if op == "distortion":
        return dict(op="distortion", d_out=_log(rng, 1024, 8192), d_in=_d8(rng, 1024, 4096),
                    bits=rng.choice([8, 8, 8, 4]), M=rng.randint(3, 5), n=_log(rng, 256, 2048))
    if op == "beam":
        return dict(op="beam", d_out=_log(rng, 500, 4096), d_in=_d8(rng, 500, 4096), bits=rng.choice([8, 8, 8, 4]),
                    k=rng.randint(2, 4), beam=rng.randint(2, 8))
    return dict(op="beam_weighted", d_out=_log(rng, 500, 4096), d_in=_d8(rng, 500, 3000), bits=8, k=rng.randint(2, 4),
                beam=rng.randint(2, 8))


# ---------------------------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _format(g, d_out, d_in, M, bits):
    """The stored format of a layer: codes, codebooks, scales."""
    shape = (M, d_out, d_in // 8)
    if bits == 16:
        codes = torch.randint(-32768, 32768, shape, dtype=torch.int16, device="cuda", generator=g)
    else:
        codes = torch.randint(0, 1 << bits, shape, dtype=torch.uint8, device="cuda", generator=g)
    books = torch.randn((M, 1 << bits, 8), device="cuda", generator=g) * (0.02 / math.sqrt(M))
    scales = torch.rand((d_out,), device="cuda", generator=g) + 0.5
    return codes, books.half(), scales.half()


def _rows(g, shape, dtype):
    x = torch.randn(shape, device="cuda", generator=g)
    big = torch.rand(shape, device="cuda", generator=g) < 0.001
    return torch.where(big, x * 20, x).to(dtype)


def _weights(g, d_out, d_in):
    return (torch.randn((d_out, d_in), device="cuda", generator=g) * 0.02).half()


def _search_inputs(case, g):
    """Dense weights, codebooks and scales of a code search: each codebook half as large as the one
    before, as the stages of a trained prefix code are."""
    d_out, d_in, k, ncw = case["d_out"], case["d_in"], case["k"], 1 << case["bits"]
    W = _weights(g, d_out, d_in)
    books = torch.randn((k, ncw, 8), device="cuda", generator=g) * 0.02
    books *= (0.5 ** torch.arange(k, device="cuda"))[:, None, None]
    scales = torch.rand((d_out,), device="cuda", generator=g) + 0.5
    H = None
    if case["op"] == "beam_weighted":
        n, G = 512, d_in // 8
        X = torch.randn((n, d_in), device="cuda", generator=g)
        X *= torch.exp(0.5 * torch.randn((d_in,), device="cuda", generator=g))
        X = X.half().float().reshape(n, G, 8).permute(1, 2, 0).contiguous()
        H = torch.bmm(X, X.transpose(1, 2).contiguous()) / n
        H = ((H + H.transpose(1, 2)) / 2).contiguous()
    return W, books.half(), scales.half(), H


def _block_shapes(case):
    """(name, d_out, d_in, which input) of a block's layers."""
    h, kv, f = case["hidden"], case["kv"], case["ffn"]
    return [("q", h, h, 0), ("k", kv, h, 0), ("v", kv, h, 0), ("o", h, h, 1), ("gate", f, h, 2), ("up", f, h, 2),
            ("down", h, f, 3)]


def _decode_inputs(case, g):
    widths = [case["hidden"], case["hidden"], case["hidden"], case["ffn"]]
    return [_rows(g, (case["blocks"], case["batch"], w), _DT[case["dtype"]]) for w in widths]


def prepare(case, seed):
    g, op = _gen(seed), case["op"]
    s = {"case": case}
    if op == "linear":
        s["layer"] = aq.QuantLinear(*_format(g, case["d_out"], case["d_in"], case["M"], case["bits"]))
        s["x"] = _rows(g, (case["n"], case["d_in"]), _DT[case["dtype"]])
    elif op == "prefill":
        s["layer"] = aq.QuantLinear(*_format(g, case["d_out"], case["d_in"], case["M"], case["bits"]))
        s["x"] = _rows(g, (case["n"], case["d_in"]), torch.bfloat16)
        s["y"] = torch.empty((case["n"], case["d_out"]), dtype=torch.bfloat16, device="cuda")
        nb = aq.gemm_workspace_bytes(s["layer"].handle, case["k"], case["n"])
        s["ws"] = torch.empty((nb,), dtype=torch.uint8, device="cuda") if nb else None
    elif op == "decode":
        s["layers"] = [[aq.QuantLinear(*_format(g, o, i, case["M"], case["bits"])) for _, o, i, _ in _block_shapes(case)]
                       for _ in range(case["blocks"])]
        s["x"] = _decode_inputs(case, g)
        s["y"] = [torch.empty((case["blocks"], case["batch"], o), dtype=_DT[case["dtype"]], device="cuda")
                  for _, o, _, _ in _block_shapes(case)]
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _decode_step(s)                       # first launches outside the recording
        torch.cuda.current_stream().wait_stream(side)
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            _decode_step(s)
    elif op == "dequant":
        s["layer"] = aq.QuantLinear(*_format(g, case["d_out"], case["d_in"], case["M"], case["bits"]))
    elif op == "distortion":
        s["layer"] = aq.QuantLinear(*_format(g, case["d_out"], case["d_in"], case["M"], case["bits"]))
        s["W"] = _weights(g, case["d_out"], case["d_in"])
        s["X"] = torch.randn((case["n"], case["d_in"]), device="cuda", generator=g).half()
        s["D"] = torch.empty((case["M"],), dtype=torch.float64, device="cuda")
    else:
        s["W"], s["books"], s["scales"], s["H"] = _search_inputs(case, g)
        G = case["d_in"] // 8
        s["desc"] = aq.make_desc(case["d_out"], case["d_in"], case["k"], case["bits"])
        s["codes"] = torch.empty((case["k"], case["d_out"], G), dtype=torch.uint8, device="cuda")
        s["errors"] = torch.empty((case["d_out"], G), dtype=torch.float32, device="cuda")
    return s


# -------------------------------------------------------------------------------------- run
def _decode_step(s):
    """One token of every stream through the linear layers of the blocks."""
    c = s["case"]
    k, b, dt = c["k"], c["batch"], _AQ[c["dtype"]]
    xs, ys = s["x"], s["y"]
    for i, (q, kk, v, o, gate, up, down) in enumerate(s["layers"]):
        aq.gemv_multi([q.handle, kk.handle, v.handle], k, xs[0][i], dt, b, [ys[0][i], ys[1][i], ys[2][i]], dt)
        aq.gemv(o.handle, k, xs[1][i], dt, b, ys[3][i], dt)
        aq.gemv_multi([gate.handle, up.handle], k, xs[2][i], dt, b, [ys[4][i], ys[5][i]], dt)
        aq.gemv(down.handle, k, xs[3][i], dt, b, ys[6][i], dt)


def run(s):
    c = s["case"]
    op = c["op"]
    if op == "linear":
        return s["layer"](s["x"], c["k"])
    if op == "prefill":
        aq.gemm_ws(s["layer"].handle, c["k"], s["x"], c["n"], s["y"], aq.DType.BF16, s["ws"])
        return s["y"]
    if op == "decode":
        s["graph"].replay()
        return s["y"]
    if op == "dequant":
        return s["layer"].dequant(c["k"], _DT[c["dtype"]])
    if op == "distortion":
        aq.prefix_distortion(s["layer"].handle, s["W"], aq.DType.F16, s["X"], aq.DType.F16, c["n"], s["D"])
        return s["D"]
    if op == "beam":
        aq.beam_search(s["desc"], c["k"], c["beam"], s["W"], s["books"], s["scales"], s["codes"], s["errors"])
    else:
        aq.beam_search_weighted(s["desc"], c["k"], c["beam"], s["W"], s["books"], s["scales"], s["H"], s["codes"],
                                s["errors"])
    return {"codes": s["codes"], "errors": s["errors"]}


# ------------------------------------------------------------------------- work and exactness
def _layer_bytes(d_out, d_in, bits, k):
    return k * d_out * (d_in // 8) * bits / 8 + k * (1 << bits) * 16 + 2 * d_out


def work(case):
    op, bits, k = case["op"], case["bits"], case.get("k", case.get("M"))
    if op == "decode":
        nb = fl = 0
        for _, o, i, _ in _block_shapes(case):
            nb += _layer_bytes(o, i, bits, k) + 2 * case["batch"] * o
            fl += 2 * case["batch"] * o * i
        nb += 2 * case["batch"] * (3 * case["hidden"] + case["ffn"])
        return {"bytes": case["blocks"] * nb, "flops": case["blocks"] * fl}
    o, i = case["d_out"], case["d_in"]
    if op in ("linear", "prefill"):
        return {"bytes": _layer_bytes(o, i, bits, k) + 2 * case["n"] * (o + i), "flops": 2 * case["n"] * o * i}
    if op == "dequant":
        return {"bytes": _layer_bytes(o, i, bits, k) + o * i * (4 if case["dtype"] == "fp32" else 2),
                "flops": k * o * i}
    if op == "distortion":                        # the products with W and with every plane's codewords
        return {"bytes": _layer_bytes(o, i, bits, k) + 2 * o * i + 2 * case["n"] * i + 8 * k,
                "flops": 2 * (k + 1) * case["n"] * o * i}
    ncw, groups = 1 << bits, o * (i // 8)         # one 8-term product per candidate
    return {"bytes": 2 * o * i + k * ncw * 16 + 2 * o + groups * (k + 4) + (256 * (i // 8) if op != "beam" else 0),
            "flops": groups * ncw * (1 + (k - 1) * case["beam"]) * 16}


def tolerance(case):
    op = case["op"]
    if op in ("dequant", "beam", "beam_weighted"):
        return "exact"                            # a stated order of 32-bit operations
    if op == "distortion":
        return {"rel": 1e-5}                      # 32-bit sums
    if case.get("dtype", "bf16") == "fp16":
        return {"rel": 1.2e-3}                    # rounding of the output
    return {"rel": 1e-2}


def _exact_weights(codes, books, scales, k):
    idx = codes[:k].to(torch.int64)
    if codes.dtype == torch.int16:
        idx = idx & 0xFFFF
    W = torch.zeros((codes.shape[1], codes.shape[2], 8), dtype=torch.float64, device="cuda")
    for m in range(k):
        W += books[m].double()[idx[m]]
    return W.reshape(codes.shape[1], -1) * scales.double()[:, None]


def _product(x, W):
    return torch.cat([p.double() @ W.t().contiguous() for p in x.split(2048)])


def _exact_search(case, g):
    """Errors of the beam search with every error in 64 bits."""
    W, books, scales, H = _search_inputs(case, g)
    k, beam, G, ncw = case["k"], case["beam"], case["d_in"] // 8, 1 << case["bits"]
    out = torch.empty((case["d_out"], G), dtype=torch.float64, device="cuda")
    rows = max(1, 4096 * 256 // (G * ncw) * 4)
    for r0 in range(0, case["d_out"], rows):
        w = W[r0:r0 + rows].double().reshape(-1, G, 8)
        s = scales[r0:r0 + rows].double()
        R = w.shape[0]
        res = w[:, :, None, :]                    # [R, G, kept, 8]
        for m in range(k):
            C = books[m].double()                 # [ncw, 8]
            if H is None:
                b, Q = res, (C * C).sum(-1)[None].expand(G, ncw)
            else:
                Hd = H.double()
                b = torch.matmul(res.permute(1, 0, 2, 3).reshape(G, -1, 8), Hd).reshape(G, R, -1, 8)
                b = b.permute(1, 0, 2, 3)
                Q = (torch.matmul(C, Hd) * C).sum(-1)             # [G, ncw]
            A = (b * res).sum(-1)                 # [R, G, kept]
            T = torch.matmul(b.reshape(-1, 8), C.t().contiguous()).reshape(R, G, -1, ncw)
            e = A[..., None] - 2 * s[:, None, None, None] * T + (s * s)[:, None, None, None] * Q[None, :, None, :]
            e = e.reshape(R, G, -1)
            keep = 1 if m == k - 1 else min(beam, e.shape[-1])
            idx = torch.topk(e, keep, dim=-1, largest=False).indices
            par, c = idx // ncw, idx % ncw
            res = torch.gather(res, 2, par[..., None].expand(-1, -1, -1, 8)) - s[:, None, None, None] * C[c]
        r = res[:, :, 0, :]
        if H is None:
            out[r0:r0 + rows] = (r * r).sum(-1)
        else:
            Hr = torch.matmul(r.permute(1, 0, 2).contiguous(), H.double()).permute(1, 0, 2)
            out[r0:r0 + rows] = (Hr * r).sum(-1)
    return out


def exact(case, seed):
    g, op = _gen(seed), case["op"]
    if op in ("beam", "beam_weighted"):
        return {"codes": None, "errors": _exact_search(case, g)}
    if op == "decode":
        fmt = [[_format(g, o, i, case["M"], case["bits"]) for _, o, i, _ in _block_shapes(case)]
               for _ in range(case["blocks"])]
        xs = _decode_inputs(case, g)
        return [torch.stack([_product(xs[sh[3]][b], _exact_weights(*fmt[b][j], case["k"]))
                             for b in range(case["blocks"])]) for j, sh in enumerate(_block_shapes(case))]
    fmt = _format(g, case["d_out"], case["d_in"], case["M"], case["bits"])
    if op == "dequant":
        return _exact_weights(*fmt, case["k"])
    if op == "distortion":
        W = _weights(g, case["d_out"], case["d_in"]).double()
        X = torch.randn((case["n"], case["d_in"]), device="cuda", generator=g).half()
        return torch.stack([_product(X, W - _exact_weights(*fmt, k)).square().sum() / (case["d_out"] * case["n"])
                            for k in range(1, case["M"] + 1)])
    x = _rows(g, (case["n"], case["d_in"]), _DT[case.get("dtype", "bf16")])
    return _product(x, _exact_weights(*fmt, case["k"]))
