"""The work that a user of this library has it do, as cases to measure.

A case is one pass of a kind of work at given sizes, through the public entry
points, with what a user's program holds beforehand (repacked weights,
descriptors, routing tables, output buffers) made by prepare():

  linear  one weight, or the four projections of a Llama-3.1-70B-shaped layer
          (one tensor-parallel share of them), applied to M rows: decode
          (M <= 64) and prefill (M > 64); bf16 or FP8 weights, tile-major or
          in a conventional layout
  moe     the expert half of a mixture-of-experts layer over routed tokens:
          grouped gate+up with the gated activation, then grouped down
  repack  a weight to tile-major and back (checkpoint load and export)
"""
import math

import torch

import paper_2607_04031_amd as tl

# Llama-3.1-70B-class projections [N, K]: qkv, o, gate+up, down
LLAMA70B = ((10240, 8192), (8192, 8192), (57344, 8192), (8192, 28672))
W_SIGMA = 0.02

KIND = {"tile": tl.TL_LAYOUT_TILE, "nk": tl.TL_LAYOUT_NK_ROW, "kn": tl.TL_LAYOUT_KN_ROW}
OUT = {"f32": tl.TL_OUT_F32, "bf16": tl.TL_OUT_BF16}
TORCH_OUT = {"f32": torch.float32, "bf16": torch.bfloat16}


def listed():
    return [
        # the smallest call: one token through one small projection, where
        # launches and latency are everything
        linear("decode_tiny", M=1, N=1024, K=1024, out="bf16"),
        # the ordinary decode step of a dense layer at a small batch
        layer("decode_layer_m8", M=8, out="f32"),
        # the same layer at a large decode batch (a batch of sequences)
        layer("decode_layer_m48", M=48, out="bf16"),
        # one GPU's share of the layer under 8-way tensor parallelism
        layer("decode_tp8_m4", M=4, tp=8, out="bf16"),
        # a language-model head with a vocabulary that no tile divides
        linear("decode_head_m5", M=5, N=50257, K=768, out="f32"),
        # the layer with 8-bit weights and per-channel scales
        layer("decode_fp8_m16", M=16, weight="fp8", G=4096, block_rows=64, out="bf16"),
        # a weight used as the checkpoint stores it, [K][N]
        linear("decode_kn_m8", M=8, N=8192, K=28672, layout="kn", out="f32"),
        # a whole prompt through the dense layer
        layer("prefill_layer_m2048", M=2048, out="bf16"),
        # a short prompt, or a few of them packed together: ragged M
        layer("prefill_layer_m300", M=300, out="bf16"),
        # Qwen-3-30B-A3B-shaped experts: a decode batch and a prompt
        moe("moe_decode_64", tokens=64, experts=128, topk=8, hidden=2048, inter=768),
        moe("moe_prefill_2048", tokens=2048, experts=128, topk=8, hidden=2048, inter=768),
        # loading a weight and writing it back out
        repack("repack_down", rows=8192, cols=28672, elem=2, G=4096, block_rows=32),
    ]


def linear(name, M, N, K, out, layout="tile", weight="bf16", G=4096, block_rows=32):
    c = {"kind": "linear", "M": M, "N": N, "K": K, "out": out, "layout": layout, "weight": weight, "G": G,
         "block_rows": block_rows}
    return dict(c, name=name) if name else c


def layer(name, M, out, tp=1, weight="bf16", G=4096, block_rows=32):
    return {"name": name, "kind": "layer", "M": M, "tp": tp, "out": out, "layout": "tile", "weight": weight, "G": G,
            "block_rows": block_rows}


def moe(name, tokens, experts, topk, hidden, inter):
    c = {"kind": "moe", "tokens": tokens, "experts": experts, "topk": topk, "hidden": hidden, "inter": inter}
    return dict(c, name=name) if name else c


def repack(name, rows, cols, elem, G, block_rows):
    c = {"kind": "repack", "rows": rows, "cols": cols, "elem": elem, "G": G, "block_rows": block_rows}
    return dict(c, name=name) if name else c


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _dim(rng, lo, hi, step):
    """A size of [lo, hi], spread over its logarithm: a multiple of 256, of 32 or of step."""
    m = rng.choice((256, 32, step))
    m = max(m, step)
    return max(lo, _log(rng, lo, hi) // m * m)


def draw(rng):
    kind = rng.choice(("decode", "decode", "decode", "prefill", "prefill", "moe", "repack"))
    if kind == "decode":
        weight = rng.choice(("bf16", "bf16", "fp8"))
        layout = rng.choice(("tile", "tile", "nk", "kn")) if weight == "bf16" else "tile"
        while True:
            N = _dim(rng, 256, 57344, 8 if layout == "kn" else 1)
            K = _dim(rng, 512, 28672, 64 if layout == "kn" else 16)
            if N * K <= 57344 * 8192:
                break
        G, br = rng.choice(((4096, 32), (4096, 16), (1024, 8), (16384, 32))) if weight == "bf16" else (4096, 64)
        return linear(None, M=_log(rng, 1, 64), N=N, K=K, out=rng.choice(("f32", "bf16")), layout=layout,
                      weight=weight, G=G, block_rows=br)
    if kind == "prefill":
        while True:
            M, N, K = _log(rng, 65, 2048), _dim(rng, 512, 57344, 1), _dim(rng, 512, 28672, 64)
            if M * N * K <= 2048 * 57344 * 8192:
                break
        G, br = rng.choice(((4096, 32), (4096, 32), (4096, 16), (16384, 32)))
        return linear(None, M=M, N=N, K=K, out=rng.choice(("f32", "bf16", "bf16")),
                      layout=rng.choice(("tile", "tile", "nk")), G=G, block_rows=br)
    if kind == "moe":
        while True:
            experts, topk = rng.choice((16, 32, 64, 128)), rng.choice((1, 2, 4, 8))
            hidden, inter = _dim(rng, 512, 4096, 64), _dim(rng, 256, 2048, 32)
            if experts * hidden * inter <= 128 * 2048 * 768 and topk * hidden * inter <= 8 * 2048 * 768:
                break
        return moe(None, tokens=_log(rng, 1, 2048), experts=experts, topk=topk, hidden=hidden, inter=inter)
    elem = rng.choice((1, 2, 2, 4))
    while True:
        rows, cols = _dim(rng, 256, 57344, 1), _dim(rng, 256, 28672, 8)
        if rows * cols * elem <= 57344 * 8192:
            break
    G, br = rng.choice(((4096, 32), (4096, 16), (1024, 8), (16384, 64)))
    return repack(None, rows=rows, cols=cols, elem=elem, G=G, block_rows=br)


# ---------------------------------------------------------------------------
# Inputs, from the seed alone
# ---------------------------------------------------------------------------

def _gen(seed, i):
    return torch.Generator(device="cuda").manual_seed(seed * 1009 + i)


def _normal(shape, seed, i, sigma=1.0):
    return (torch.randn(shape, generator=_gen(seed, i), device="cuda", dtype=torch.float32) * sigma).to(torch.bfloat16)


def _shapes(case):
    if case["kind"] == "linear":
        return [(case["N"], case["K"])]
    t = case["tp"]   # column-parallel qkv and gate+up, row-parallel o and down
    (qn, qk), (on, ok), (gn, gk), (dn, dk) = LLAMA70B
    return [(qn // t, qk), (on, ok // t), (gn // t, gk), (dn, dk // t)]


def _activations(case, seed, i, K):
    return _normal((case["M"], K), seed, 2 * i, 1.0)


def _weight(case, seed, i, N, K):
    """A weight [N, K]: bf16, or FP8 E4M3 with per-channel scales (float32 [N])."""
    w = _normal((N, K), seed, 2 * i + 1, W_SIGMA)
    if case["weight"] == "bf16":
        return w, None
    amax = w.abs().amax(dim=1).float()
    scales = torch.where(amax > 0, amax / 448.0, torch.ones_like(amax))
    return (w.float() / scales[:, None]).to(torch.float8_e4m3fn), scales


def _routing(case, seed):
    """Per token topk distinct experts: group offsets [E + 1], the token of each row (rows sorted by expert), and the
    largest group."""
    scores = torch.rand((case["tokens"], case["experts"]), generator=_gen(seed, 0), device="cuda")
    chosen = scores.topk(case["topk"], dim=1).indices.flatten()
    order = torch.sort(chosen, stable=True).indices
    counts = torch.bincount(chosen, minlength=case["experts"])
    offsets = torch.zeros(case["experts"] + 1, dtype=torch.int32, device="cuda")
    offsets[1:] = counts.cumsum(0)
    return offsets, (order // case["topk"]).to(torch.int32), int(counts.max())


def _experts(case, seed):
    E, H, I = case["experts"], case["hidden"], case["inter"]
    return _normal((case["tokens"], H), seed, 1), _normal((E, 2 * I, H), seed, 2, W_SIGMA), _normal((E, H, I), seed, 3, W_SIGMA)


def _stack(ws, G, block_rows):
    """The experts' weights, repacked one by one into one stack."""
    out = torch.empty((ws.shape[0],) + tl.padded_shape(ws.shape[1], ws.shape[2], 2, G, block_rows), dtype=ws.dtype, device="cuda")
    for e in range(ws.shape[0]):
        tl.repack(ws[e], G, block_rows, out=out[e])
    return out


def _matrix(case, seed):
    dt = {1: torch.uint8, 2: torch.int16, 4: torch.int32}[case["elem"]]
    info = torch.iinfo(dt)
    return torch.randint(info.min, info.max, (case["rows"], case["cols"]), generator=_gen(seed, 0), device="cuda", dtype=dt)


def prepare(case, seed):
    if case["kind"] in ("linear", "layer"):
        calls = []
        for i, (N, K) in enumerate(_shapes(case)):
            a = _activations(case, seed, i, K)
            w, scales = _weight(case, seed, i, N, K)
            if case["layout"] == "tile":
                raw = w.view(torch.uint8) if case["weight"] == "fp8" else w
                w = tl.repack(raw, case["G"], case["block_rows"])
            elif case["layout"] == "kn":
                w = w.t().contiguous()
            desc = tl.layout(kind=KIND[case["layout"]], G=case["G"], block_rows=case["block_rows"],
                             out_dtype=OUT[case["out"]], elem_bytes=1 if case["weight"] == "fp8" else 2)
            c = torch.empty((case["M"], N), dtype=TORCH_OUT[case["out"]], device="cuda")
            calls.append((a, w, scales, c, N, K, desc))
        fetch = tl.TL_FETCH_BLOCK if case["layout"] == "tile" else tl.TL_FETCH_NATIVE
        return {"kind": "linear", "M": case["M"], "calls": calls, "fetch": fetch}
    if case["kind"] == "moe":
        E, H, I = case["experts"], case["hidden"], case["inter"]
        x, gate_up, down = _experts(case, seed)
        offsets, ids, most = _routing(case, seed)
        rows = case["tokens"] * case["topk"]
        gate_up, down = _stack(gate_up, 4096, 32), _stack(down, 4096, 32)
        return {"kind": "moe", "x": x, "gate_up": gate_up, "down": down, "offsets": offsets, "ids": ids, "most": most,
                "rows": rows, "E": E, "H": H, "I": I,
                "gate_up_stride": gate_up.stride(0) * 2, "down_stride": down.stride(0) * 2,
                "h": torch.empty((rows, I), dtype=torch.bfloat16, device="cuda"),
                "y": torch.empty((rows, H), dtype=torch.bfloat16, device="cuda"),
                "desc": tl.layout(G=4096, block_rows=32, out_dtype=tl.TL_OUT_BF16)}
    w = _matrix(case, seed)
    G, br = case["G"], case["block_rows"]
    packed = torch.empty(tl.padded_shape(case["rows"], case["cols"], case["elem"], G, br), dtype=w.dtype, device="cuda")
    return {"kind": "repack", "w": w, "packed": packed, "back": torch.empty_like(w), "G": G, "block_rows": br}


def run(s):
    if s["kind"] == "linear":
        for a, w, scales, c, N, K, desc in s["calls"]:
            if scales is None:
                tl.tl_gemm(a, w, c, s["M"], N, K, desc, s["fetch"])
            else:
                tl.tl_gemm_w8(a, w, scales, c, s["M"], N, K, desc, s["fetch"])
        return [call[3] for call in s["calls"]]
    if s["kind"] == "moe":
        tl.tl_gemm_grouped_swiglu(s["x"], s["x"].shape[0], s["ids"], s["offsets"], s["E"], s["rows"], s["most"],
                                  s["gate_up"], s["gate_up_stride"], s["h"], s["I"], s["H"], s["desc"])
        tl.tl_gemm_grouped(s["h"], s["rows"], None, s["offsets"], s["E"], s["rows"], s["most"], s["down"],
                           s["down_stride"], s["y"], s["H"], s["I"], s["desc"])
        return [s["h"], s["y"]]
    rows, cols = s["w"].shape
    tl.repack(s["w"], s["G"], s["block_rows"], out=s["packed"])
    tl.unpack(s["packed"], s["G"], s["block_rows"], rows, cols, out=s["back"])
    return [s["packed"], s["back"]]


def work(case):
    if case["kind"] in ("linear", "layer"):
        M, cb = case["M"], 4 if case["out"] == "f32" else 2
        wb = 1 if case["weight"] == "fp8" else 2
        shapes = _shapes(case)
        extra = sum(4 * N for N, _ in shapes) if wb == 1 else 0
        return {"bytes": sum(wb * N * K + 2 * M * K + cb * M * N for N, K in shapes) + extra,
                "flops": sum(2 * M * N * K for N, K in shapes)}
    if case["kind"] == "moe":
        E, H, I, T, k = case["experts"], case["hidden"], case["inter"], case["tokens"], case["topk"]
        read = E * (1 - (1 - k / E) ** T)   # experts that get a token, on average
        rows = T * k
        return {"bytes": read * 3 * I * H * 2 + T * H * 2 + 2 * rows * I * 2 + rows * H * 2 + rows * 4,
                "flops": 2 * rows * 3 * I * H}
    rows, cols, s = case["rows"], case["cols"], case["elem"]
    r, c = tl.padded_shape(rows, cols, s, case["G"], case["block_rows"])
    return {"bytes": 2 * rows * cols * s + 2 * r * c * s, "flops": 0}


def tolerance(case):
    if case["kind"] == "repack":
        return "exact"
    if case["kind"] == "moe":
        # bf16 rounding of both outputs and of the activation between them
        return {"rel": 8e-3, "max": 2e-2}
    if case["out"] == "bf16":
        # one rounding to bf16 (1.7e-3 of the result); a sum near a rounding boundary may land one unit away
        return {"rel": 7e-3, "max": 1.6e-2}
    # fp32 sums of up to 28672 products in another order
    return {"rel": 4e-6, "max": 2e-5}


def exact(case, seed):
    if case["kind"] in ("linear", "layer"):
        got = []
        for i, (N, K) in enumerate(_shapes(case)):
            a = _activations(case, seed, i, K).double()
            w, scales = _weight(case, seed, i, N, K)
            c = torch.empty((case["M"], N), dtype=torch.float64, device="cuda")
            for n in range(0, N, 8192):
                part = w[n:n + 8192].float().double()
                if scales is not None:
                    part = part * scales[n:n + 8192, None].double()
                c[:, n:n + 8192] = a @ part.t().contiguous()
            got.append(c)
        return got
    if case["kind"] == "moe":
        I = case["inter"]
        x, gate_up, down = _experts(case, seed)
        offsets, ids, _ = _routing(case, seed)
        at = offsets.tolist()
        hs, ys = [], []
        for e in range(case["experts"]):
            if at[e] == at[e + 1]:
                continue
            rows = x[ids[at[e]:at[e + 1]].long()].double()
            g = rows @ gate_up[e].double().t().contiguous()
            h = torch.nn.functional.silu(g[:, :I]) * g[:, I:]
            hs.append(h)
            ys.append(h @ down[e].double().t().contiguous())
        return [torch.cat(hs), torch.cat(ys)]
    w = _matrix(case, seed)
    rows, cols, s, G, br = case["rows"], case["cols"], case["elem"], case["G"], case["block_rows"]
    bc = G // (s * br)
    r, c = -(-rows // br) * br, -(-cols // bc) * bc
    padded = torch.zeros((r, c), dtype=w.dtype, device="cuda")
    padded[:rows, :cols] = w
    tiles = padded.view(r // br, br, c // bc, bc).transpose(1, 2).contiguous()
    return [tiles.view(r, c), w]
