"""Performance cases: the calls a program makes that keeps INT8 weights compressed in GPU memory.

The work is the runtime half of the method and the compression that feeds it, all on device buffers: decoding chunks
into a buffer (both coders, all coded or partly raw), the decode fused with the conversion to bf16 and with the batch-1
products, the products on decoded weights, and the compression itself.  Shapes are those of Llama-7B and Llama-13B
decoder layers, single matrices, and odd sizes; chunk sizes, sub-stream counts and policies are the ones the library
takes.  The weights are normal with one row in a hundred eight times larger, quantised per row to INT8 with |q| <= 1
pruned, optionally after the per-input-channel rescale of the compression stage.
"""
import math

import numpy as np
import torch

import paper_2502_15443_amd as dc

CODECS = {"huffman": dc.CODEC_HUFFMAN, "tans": dc.CODEC_TANS}
POLICIES = {"all": dc.POLICY_ALL_HUFF, "auto": dc.POLICY_AUTO, "raw_fraction": dc.POLICY_RAW_FRACTION,
            "block_last": dc.POLICY_BLOCK_LAST}

# (rows, cols) of the matrices of a decoder layer: q k v o gate up down
LAYERS = {
    "llama7b": [(4096, 4096)] * 4 + [(11008, 4096)] * 2 + [(4096, 11008)],
    "llama13b": [(5120, 5120)] * 4 + [(13824, 5120)] * 2 + [(5120, 13824)],
    "llama7b_attention": [(4096, 4096)] * 4,
}
# entropy of the weights in bits a byte, without and with the rescale
ENTROPY_BITS = {False: 7.06, True: 5.64}


def case(name, kind, shape="", rows=0, cols=0, layers=1, rescale=False, chunk_bytes=65536, n_streams=256, codec="huffman",
         policy="all", raw_fraction=0.0, block_chunks=0, act="bf16"):
    c = dict(kind=kind, shape=shape, rows=rows, cols=cols, layers=layers, rescale=rescale, chunk_bytes=chunk_bytes,
             n_streams=n_streams, codec=codec, policy=policy, raw_fraction=raw_fraction, block_chunks=block_chunks, act=act)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one small projection of odd size, a few dozen short chunks; a latency
        case("decode small odd", "decode", rows=1023, cols=1021, chunk_bytes=16384),
        # one matrix at the sub-stream count that gives the best compression ratio: long chains, few wavefronts
        case("decode matrix 32 streams", "decode", rows=4096, cols=4096, n_streams=32),
        # the layer about to be used, decoded into the decompression buffer: the ordinary call
        case("decode 7B layer", "decode", shape="llama7b", rescale=True),
        # several layers in one launch, as much as the buffer holds: the largest call
        case("decode four 7B layers", "decode", shape="llama7b", layers=4),
        # the speed-adaptive mix: half of the chunks stored raw
        case("decode 7B layer half raw", "decode", shape="llama7b", rescale=True, policy="raw_fraction", raw_fraction=0.5),
        # the container's second coder
        case("decode 7B layer tans", "decode", shape="llama7b", rescale=True, codec="tans"),
        # a layer decoded straight to bf16 for a GEMM over a batch (prefill)
        case("dequant 13B layer", "dequant", shape="llama13b"),
        # a layer's batch-1 products without writing the weights (token decode)
        case("gemv 13B layer", "gemv", shape="llama13b"),
        # the same in INT8 arithmetic on the attention projections, at a quarter of the sub-streams
        case("gemv w8a8 7B attention", "gemv", shape="llama7b_attention", rescale=True, n_streams=64, act="int8"),
        # the products of a layer whose weights already lie decoded in the buffer, one call a matrix
        case("resident products 7B layer", "resident", shape="llama7b"),
        # compressing a layer on the GPU, chunks that would grow kept raw
        case("compress 7B layer", "compress", shape="llama7b", rescale=True, policy="auto"),
        # compressing one projection with the second coder
        case("compress matrix tans", "compress", rows=11008, cols=4096, codec="tans", policy="auto"),
    ]


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "decode", "dequant", "gemv", "gemv", "resident", "compress", "compress"])
    limit = {"decode": 128 << 20, "dequant": 128 << 20, "gemv": 128 << 20, "resident": 64 << 20, "compress": 64 << 20}[kind]
    elements = math.exp(rng.uniform(math.log(1 << 18), math.log(limit)))
    cols = int(math.exp(rng.uniform(math.log(256), math.log(16384))))
    if kind in ("dequant", "gemv", "resident"):
        cols = max(16, cols // 16 * 16)
    rows = max(1, int(elements / cols))
    n_streams = rng.choice([32, 64, 128, 256, 256])
    codec = rng.choice(["huffman", "huffman", "huffman", "tans"]) if n_streams >= 64 and kind != "resident" else "huffman"
    if rng.random() < 0.6:
        chunk = rng.choice([8192, 16384, 32768, 65536, 65536, 131072, 262144])
    else:
        chunk = int(math.exp(rng.uniform(math.log(4096), math.log(131072)))) // 16 * 16
    policy = rng.choice(["all", "all", "auto", "raw_fraction", "block_last"])
    return case(None, kind, rows=rows, cols=cols, rescale=rng.random() < 0.5, chunk_bytes=chunk, n_streams=n_streams,
                codec=codec, policy=policy, raw_fraction=round(rng.uniform(0.05, 0.95), 2) if policy == "raw_fraction" else 0.0,
                block_chunks=rng.randint(2, 9) if policy == "block_last" else 0, act=rng.choice(["bf16", "int8"]))


def matrices(c):
    return (LAYERS[c["shape"]] if c["shape"] else [(c["rows"], c["cols"])]) * c["layers"]


def params(c):
    return dc.Params(c["chunk_bytes"], c["n_streams"], POLICIES[c["policy"]], c["raw_fraction"], c["block_chunks"],
                     codec=CODECS[c["codec"]])


def generator(seed, part):
    return torch.Generator(device="cuda").manual_seed(seed * 1009 + part)


def weight(c, seed, i, rows, cols):
    """Matrix i of the case: int8 q[rows, cols] and its fp32 row scales."""
    g = generator(seed, 4 * i)
    w = torch.randn(rows, cols, generator=g, device="cuda") * 0.02
    w[torch.randperm(rows, generator=g, device="cuda")[:round(rows * 0.01)]] *= 8.0
    if c["rescale"]:
        w *= torch.exp(torch.randn(cols, generator=g, device="cuda")).sqrt()
    top = w.abs().amax(1)
    scale = torch.where(top == 0, torch.ones_like(top), top / 127)
    q = torch.round(w / scale[:, None]).clamp_(-127, 127)
    q[q.abs() <= 1] = 0
    return q.to(torch.int8), scale


def activation(c, seed, i, cols):
    """Activations of matrix i: bf16 values, or int8 values and their scale."""
    x = torch.randn(cols, generator=generator(seed, 4 * i + 1), device="cuda")
    if c["act"] == "bf16":
        return x.to(torch.bfloat16), 0.0
    scale = float(np.float32(x.abs().max().item()) / np.float32(127))
    return torch.round(x / scale).clamp_(-127, 127).to(torch.int8), scale


def compressor(c, n, src):
    """Buffers of one compression of n bytes."""
    p = params(c)
    cap, nc = dc.compress_bound(n, p)
    ws = dc.compress_chunks_dev_workspace(n, p)
    return {"p": p, "n": n, "src": src, "cap": cap, "nc": nc, "ws_n": ws, "blob": torch.zeros(cap, dtype=torch.uint8, device="cuda"),
            "table": torch.zeros(nc, 2, dtype=torch.int64, device="cuda"), "ws": torch.empty(ws, dtype=torch.uint8, device="cuda"),
            "result": torch.zeros(2, dtype=torch.int64, device="cuda")}


def compress(b, stream):
    dc.compress_chunks_dev(b["src"], b["n"], b["p"], b["blob"], b["cap"], b["table"], b["nc"], b["ws"], b["ws_n"], b["result"], stream)


def compressed(c, src):
    """Blob and table of the bytes of one tensor."""
    b = compressor(c, src.numel(), src.reshape(-1))
    compress(b, torch.cuda.current_stream().cuda_stream)
    size, err = b["result"].tolist()
    if err:
        raise RuntimeError("the blob does not fit its bound")
    return b["blob"][:size].clone(), b["table"]


def flat_weights(c, seed):
    return torch.cat([weight(c, seed, i, r, k)[0].reshape(-1) for i, (r, k) in enumerate(matrices(c))])


def prepare(c, seed):
    s = {"kind": c["kind"], "p": params(c), "act": c["act"]}
    if c["kind"] == "compress":
        q = flat_weights(c, seed)
        return dict(s, **compressor(c, q.numel(), q))
    if c["kind"] == "decode":
        q = flat_weights(c, seed)
        blob, table = compressed(c, q)
        return dict(s, blob=blob, blob_n=blob.numel(), table=table, nc=table.shape[0], n=q.numel(),
                    dst=torch.zeros(q.numel(), dtype=torch.int8, device="cuda"))
    # the fused calls and the products: every matrix starts at a chunk of its own
    s.update(q=[], scale=[], x=[], x_scale=[], out=[], y_bf16=[], mats=[], rows=[], cols=[])
    blobs, tables, at, nc = [], [], 0, 0
    for i, (rows, cols) in enumerate(matrices(c)):
        q, scale = weight(c, seed, i, rows, cols)
        x, x_scale = activation(c, seed, i, cols)
        if c["kind"] == "dequant":
            out = torch.zeros(rows, cols, dtype=torch.bfloat16, device="cuda")
        else:
            out = torch.zeros(rows, dtype=torch.float32, device="cuda")
        # the INT8 product leaves bf16 results beside the fp32 ones
        y16 = torch.zeros(rows, dtype=torch.bfloat16, device="cuda") if c["act"] == "int8" and c["kind"] != "dequant" else None
        for k, v in (("scale", scale), ("x", x), ("x_scale", x_scale), ("out", out), ("y_bf16", y16), ("rows", rows), ("cols", cols)):
            s[k].append(v)
        if c["kind"] == "resident":
            s["q"].append(q)
            continue
        blob, table = compressed(c, q)
        table[:, 0] += at
        if c["kind"] == "dequant":
            s["mats"].append(dc.Matrix(nc, rows, cols, scale, dst_bf16_dev=out, dst_cap_elems=rows * cols))
        elif c["act"] == "bf16":
            s["mats"].append(dc.Matrix(nc, rows, cols, scale, x_bf16_dev=x, y_accum_dev=out))
        else:
            s["mats"].append(dc.Matrix(nc, rows, cols, scale, y_accum_dev=out, y_bf16_dev=y16, x_i8_dev=x, x_scale=x_scale))
        blobs.append(blob)
        tables.append(table)
        at += blob.numel()
        nc += table.shape[0]
    if c["kind"] != "resident":
        ws = dc.decompress_gemv_workspace(nc)
        s.update(blob=torch.cat(blobs), blob_n=at, table=torch.cat(tables), nc=nc, ws_n=ws,
                 ws=torch.empty(ws, dtype=torch.uint8, device="cuda"))
    return s


def run(s):
    stream = torch.cuda.current_stream().cuda_stream
    if s["kind"] == "compress":
        compress(s, stream)
        return {"blob": s["blob"], "table": s["table"], "result": s["result"]}
    if s["kind"] == "decode":
        dc.decompress_chunks(s["blob"], s["blob_n"], s["table"], s["nc"], s["p"], s["dst"], s["n"], stream)
        return s["dst"]
    if s["kind"] == "dequant":
        dc.decompress_dequant_bf16_layer(s["blob"], s["blob_n"], s["table"], s["nc"], s["p"], s["mats"], stream)
        return s["out"]
    if s["kind"] == "resident":
        for q, scale, rows, cols, x, x_scale, y, y16 in zip(s["q"], s["scale"], s["rows"], s["cols"], s["x"], s["x_scale"], s["out"], s["y_bf16"]):
            if s["act"] == "bf16":
                dc.gemv_i8(q, scale, rows, cols, x, y, y16, stream)
            else:
                dc.gemv_w8a8(q, scale, rows, cols, x, x_scale, y, y16, stream)
    elif s["act"] == "bf16":
        dc.decompress_gemv_layer(s["blob"], s["blob_n"], s["table"], s["nc"], s["p"], s["mats"], s["ws"], s["ws_n"], stream)
    else:
        dc.decompress_gemv_w8a8_layer(s["blob"], s["blob_n"], s["table"], s["nc"], s["p"], s["mats"], stream)
    return {"y": s["out"], "y_bf16": [y for y in s["y_bf16"] if y is not None]}


def work(c):
    n = sum(r * k for r, k in matrices(c))
    coded = {"raw_fraction": 1 - c["raw_fraction"], "block_last": 1 / max(1, c["block_chunks"])}.get(c["policy"], 1.0)
    stored = n * (1 - coded + coded * ENTROPY_BITS[c["rescale"]] / 8)
    vectors = sum(8 * r + 2 * k for r, k in matrices(c))
    if c["kind"] in ("decode", "compress"):
        return {"bytes": n + stored, "flops": 0}
    if c["kind"] == "dequant":
        return {"bytes": 2 * n + stored, "flops": n}
    return {"bytes": (n if c["kind"] == "resident" else stored) + vectors, "flops": 2 * n}


def tolerance(c):
    # decoded bytes, compressed bytes, scaled values rounded once and integer sums have one right value; the fp32 sums
    # of the bf16 product differ by their order (0.7e-7 against 64 bits for this kernel; a plain serial sum of 16384 terms shows some 2.5e-7)
    return {"rel": 1e-6} if c["kind"] in ("gemv", "resident") and c["act"] == "bf16" else "exact"


def exact(c, seed):
    if c["kind"] == "compress":
        return None
    if c["kind"] == "decode":
        return flat_weights(c, seed)
    if c["kind"] == "dequant":
        return [q.double() * scale.double()[:, None] for q, scale in (weight(c, seed, i, r, k) for i, (r, k) in enumerate(matrices(c)))]
    y = []
    for i, (rows, cols) in enumerate(matrices(c)):
        q, scale = weight(c, seed, i, rows, cols)
        x, x_scale = activation(c, seed, i, cols)
        y.append((q.double() @ x.double()) * scale.double() * (x_scale if c["act"] == "int8" else 1.0))
    return {"y": y, "y_bf16": [None] * (len(y) if c["act"] == "int8" else 0)}
