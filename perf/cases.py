"""What a user of this framework has it do, as cases that can be timed and compared.

A case is one call (or one batched call) of a public entry point of `paper_2604_03298_amd.enec`:

  op          compress, decompress, compress_per_block, decompress_per_block or tune
  kind        what the tensors hold: "norm" (weights around one), "gauss" (one standard deviation per tensor),
              "layer" (the nine tensors of a decoder layer, a scale per row and rare outliers) or "mix" (blocks of
              zeros, of one value, heavy tails, random bits)
  dtype       bf16, fp16 or fp32
  count       how many tensors the call takes; one tensor goes through the entry point for one, several through the batch
  elems       elements per tensor (kind "layer": unused, hidden and ffn give the shapes)
  L, block    group length and data-block size (0 = the library's default)
  every       tune: 1 = all exponents, k = every k-th chunk

Weights are compressed when a checkpoint is prepared and decompressed each time a layer is used, so both directions are
here at the size of a vector, a matrix, a layer and a stream of large matrices.  Everything the calls return is bytes or
counts, so outputs are compared exactly.
"""
import math

import numpy as np
import torch

from paper_2604_03298_amd import enec

DTYPES = {"bf16": (torch.bfloat16, torch.int16, enec.BF16, 2),
          "fp16": (torch.float16, torch.int16, enec.FP16, 2),
          "fp32": (torch.float32, torch.int32, enec.FP32, 4)}


def _case(name, op, kind, dtype="bf16", count=1, elems=0, hidden=0, ffn=0, L=16, block=0, every=1):
    c = {"op": op, "kind": kind, "dtype": dtype, "count": count, "elems": elems, "hidden": hidden, "ffn": ffn,
         "L": L, "block": block, "every": every}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the two norm vectors of a decoder layer: the smallest call, one data block each, latency only
        _case("norms-compress", "compress", "norm", count=2, elems=4096),
        # one 1024 x 4096 matrix (a key or value projection with grouped heads) needed right now
        _case("matrix-decompress", "decompress", "gauss", elems=1024 * 4096),
        # a whole 7B-style decoder layer, nine tensors with two different tuples, when a checkpoint is prepared ...
        _case("layer-compress", "compress", "layer", count=9, hidden=4096, ffn=11008),
        # ... and when the layer is about to be used
        _case("layer-decompress", "decompress", "layer", count=9, hidden=4096, ffn=11008),
        # matrices of a 70B-style feed-forward, 470 MB each: the long launches
        _case("large-compress", "compress", "gauss", count=2, elems=8192 * 28672),
        _case("large-decompress", "decompress", "gauss", count=2, elems=8192 * 28672),
        # half-precision checkpoint, an odd vocabulary: the last block is ragged
        _case("fp16-ragged-compress", "compress", "gauss", "fp16", count=2, elems=32003 * 2047),
        # single-precision checkpoint, ragged
        _case("fp32-ragged-decompress", "decompress", "gauss", "fp32", elems=11007 * 4099),
        # groups of eight, which Eq. 4's joint search picks for Gaussian weights: the best ratio
        _case("group8-compress", "compress", "gauss", count=4, elems=4096 * 4096, L=8),
        # one tuple per data block: a tensor whose blocks differ in kind
        _case("mix-per-block-compress", "compress_per_block", "mix", elems=4096 * 16384),
        # the layer coded with one tuple per data block, read back
        _case("layer-per-block-decompress", "decompress_per_block", "layer", count=9, hidden=4096, ffn=11008),
        # the parameter search for the whole layer (the caller waits for the tuples)
        _case("layer-tune", "tune", "layer", count=9, hidden=4096, ffn=11008),
    ]


def draw(rng):
    """One more case: any operation, format, group length and block size, 4096 elements to half a gigabyte of input."""
    op = rng.choice(["compress", "compress", "decompress", "decompress", "compress_per_block", "decompress_per_block", "tune"])
    kind = rng.choice(["gauss", "gauss", "gauss", "layer", "norm"] + (["mix"] if "per_block" in op else []))
    dtype = rng.choice(["bf16", "bf16", "fp16", "fp32"]) if kind in ("gauss", "norm") else "bf16"
    L, block = 16, 0
    if op != "tune" and rng.random() < 0.4:
        L, block = rng.choice([(8, 0), (32, 0), (16, 4096), (16, 8192), (16, 32768), (8, 8192), (32, 32768)])
    every = rng.choice([1, 1, 16]) if op == "tune" else 1
    if kind == "layer":
        hidden = 64 * int(round(2 ** rng.uniform(3, 6.3)))
        return _case(None, op, kind, dtype, 9, 0, hidden, 2 * (hidden * 43 // 32), L, block, every)
    count = rng.choice([1, 1, 2, 3, 7, 16, 20])
    if kind == "norm":
        return _case(None, op, kind, dtype, count, int(2 ** rng.uniform(12, 14)), L=L, block=block, every=every)
    top = 28 - (dtype == "fp32") - ("per_block" in op)
    total = 2 ** rng.uniform(14, top)
    elems = max(4096, int(total / count))
    if rng.random() < 0.5:
        elems |= 1
    return _case(None, op, kind, dtype, count, elems, L=L, block=block, every=every)


def _sizes(case):
    """(elements, rows) of the case's tensors; rows = 0: no rows."""
    if case["kind"] == "layer":
        h, f = case["hidden"], case["ffn"]
        return [(h * h, h)] * 4 + [(h * f, h)] * 2 + [(h * f, f)] + [(h, 0)] * 2
    return [(case["elems"], 0)] * case["count"]


def _values(case, seed):
    """The tensors' bit patterns on the GPU, from the seed alone.  Normals are drawn in 64 bits: single-precision samplers
    give exact zeros, which real weights hardly have and which would force the widest tuple."""
    real, bits, _, _ = DTYPES[case["dtype"]]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    out = []
    sizes = _sizes(case)
    stds = np.exp(np.random.RandomState(seed % (1 << 32)).uniform(math.log(0.003), math.log(0.03), len(sizes)))
    for i, (n, rows) in enumerate(sizes):
        x = torch.empty(n, dtype=real, device="cuda")
        if case["kind"] == "mix":
            x = _mix(n, g)
        elif case["kind"] == "norm" or (case["kind"] == "layer" and not rows):
            x.copy_(1 + 0.05 * torch.randn(n, generator=g, device="cuda", dtype=torch.float64))
        elif case["kind"] == "layer":
            cols = n // rows
            scale = torch.exp(math.log(0.005) + math.log(10) * torch.rand(rows, 1, generator=g, device="cuda", dtype=torch.float64))
            step = max(1, (1 << 25) // cols)
            for r in range(0, rows, step):
                s = scale[r:r + step]
                v = torch.randn(s.shape[0], cols, generator=g, device="cuda", dtype=torch.float64)
                u = torch.rand(s.shape[0], cols, generator=g, device="cuda")
                v = torch.where(u < 0.0005, 20.0, torch.where(u < 0.001, -20.0, v)) * s
                x[r * cols:(r + s.shape[0]) * cols] = v.reshape(-1).to(real)
        else:
            for s in range(0, n, 1 << 25):
                e = min(n, s + (1 << 25))
                x[s:e] = (torch.randn(e - s, generator=g, device="cuda", dtype=torch.float64) * float(stds[i])).to(real)
        out.append(x.view(bits))
    return out


def _mix(n, g):
    """Blocks of 16384: zeros, one repeated value, Student-t (three degrees of freedom) or random bits, a quarter each."""
    nb = -(-n // 16384)
    kind = torch.randperm(nb, generator=g, device="cuda") % 4
    out = torch.zeros(nb, 16384, dtype=torch.int16, device="cuda")
    one = (0.02 * torch.randn(nb, 1, generator=g, device="cuda")).to(torch.bfloat16).view(torch.int16)
    out = torch.where((kind == 1)[:, None], one, out)
    bits = torch.randint(-32768, 32768, (nb, 16384), generator=g, device="cuda", dtype=torch.int16)
    out = torch.where((kind == 3)[:, None], bits, out)
    del bits
    for s in range(0, nb, 512):
        v = torch.randn(4, min(512, nb - s), 16384, generator=g, device="cuda", dtype=torch.float64)
        t = v[0] / (v[1:].square().sum(0) / 3).sqrt()
        out[s:s + 512] = torch.where((kind[s:s + 512] == 2)[:, None], (0.02 * t).to(torch.bfloat16).view(torch.int16), out[s:s + 512])
    return out.reshape(-1)[:n].contiguous().view(torch.bfloat16)


def prepare(case, seed):
    """Tensors, tuples, workspace and output buffers; for the way back the streams, their headers and the item array."""
    _, _, code, _ = DTYPES[case["dtype"]]
    srcs = _values(case, seed)
    block, L = case["block"], case["L"]
    total, smallest = sum(s.numel() for s in srcs), min(s.numel() for s in srcs)
    st = {"op": case["op"], "dtype": code, "srcs": srcs, "every": case["every"], "L": L}
    st["ws"] = enec.new_workspace(total, block or enec.default_block_size(smallest))
    if case["op"] == "tune":
        return st
    # a group length that a short tensor's own block size does not admit is coded with the next block size that does
    st["blocks"] = [block or max(enec.default_block_size(s.numel()), 4096 if L == 32 else 2048) for s in srcs]
    per_block = case["op"].endswith("per_block")
    bound = enec.compress_bound_per_block if per_block else enec.compress_bound
    st["outs"] = [torch.zeros(bound(s.numel(), code, b), dtype=torch.uint8, device="cuda") for s, b in zip(srcs, st["blocks"])]
    st["sizes"] = torch.zeros(len(srcs), dtype=torch.int64, device="cuda")
    st["size_views"] = [st["sizes"][i:i + 1] for i in range(len(srcs))]
    if not per_block:
        st["params"] = [enec.tune(s, st["ws"], dtype=code, lengths=None if L == 16 else (L,), block_size=b)
                        for s, b in zip(srcs, st["blocks"])]
    if case["op"].startswith("decompress"):
        _compress(st, per_block)
        streams = [o[:int(n)].clone() for o, n in zip(st["outs"], st["sizes"].tolist())]
        st["streams"] = streams
        st["headers"] = [bytes(s[:enec.HEADER_BYTES].cpu().numpy()) for s in streams]
        st["backs"] = [torch.zeros_like(s) for s in srcs]
        st["items"] = enec.make_decompress_items(streams, st["headers"], st["backs"])
        for k in ("outs", "srcs", "sizes", "size_views", "ws"):
            del st[k]
    return st


def _done(rc):
    if rc != enec.OK:
        raise RuntimeError(enec.strerror(rc))


def _compress(st, per_block):
    if per_block and len(st["srcs"]) == 1:
        _done(enec.compress_per_block(st["srcs"][0], st["outs"][0], st["ws"], block_size=st["blocks"][0], out_bytes=st["size_views"][0],
                                      dtype=st["dtype"], group_length=st["L"]))
    elif per_block:
        _done(enec.compress_per_block_batch(st["srcs"], st["outs"], st["ws"], out_bytes=st["size_views"], dtype=st["dtype"],
                                            block_sizes=st["blocks"], group_length=st["L"]))
    elif len(st["srcs"]) == 1:
        _done(enec.compress(st["srcs"][0], st["params"][0], st["outs"][0], st["ws"], block_size=st["blocks"][0],
                            out_bytes=st["size_views"][0], dtype=st["dtype"]))
    else:
        _done(enec.compress_batch(st["srcs"], st["params"], st["outs"], st["ws"], block_sizes=st["blocks"],
                                  out_bytes=st["size_views"], dtype=st["dtype"]))


def run(st):
    if st["op"] == "tune":
        prm, hist = enec.tune_batch(st["srcs"], st["ws"], every=st["every"], dtype=st["dtype"], want_histograms=True)
        return {"params": np.array(prm, dtype=np.int64), "histograms": hist.view(np.int64)}
    if st["op"].startswith("compress"):
        _compress(st, st["op"] == "compress_per_block")
        return {"streams": st["outs"], "sizes": st["sizes"]}
    if len(st["streams"]) == 1:
        _done(enec.decompress_with_header(st["streams"][0], st["headers"][0], st["backs"][0]))
    else:
        _done(enec.decompress_batch(st["streams"], st["headers"], st["backs"], items=st["items"][0]))
    return st["backs"]


def exact(case, seed):
    """What the way back has to return is the tensors themselves, what the search counts is a plain count.  A stream has no
    such second form, and neither has the tuple that is found."""
    if case["op"].startswith("decompress"):
        return _values(case, seed)
    if case["op"] == "tune" and case["every"] == 1:
        shift, mask = {"bf16": (7, 255), "fp16": (10, 31), "fp32": (23, 255)}[case["dtype"]]
        h = [torch.bincount((v.to(torch.int32) >> shift) & mask, minlength=256) for v in _values(case, seed)]
        return {"params": None, "histograms": torch.stack(h).cpu()}
    return None


def tolerance(case):
    return "exact"


# stream bytes per input byte: what the coded exponents of such values take (paper: 1.33 to 1.38, 1.09 to 1.12 and 1.15)
SHARE = {"bf16": 1 / 1.37, "fp16": 1 / 1.11, "fp32": 1 / 1.16}


def work(case):
    """The tensor once and the stream once.  The arithmetic is a few whole-number operations per element."""
    size = DTYPES[case["dtype"]][3]
    raw = float(sum(n for n, _ in _sizes(case)) * size)
    if case["op"] == "tune":
        return {"bytes": raw / case["every"], "flops": 0.0}
    share = {"mix": 1 / 1.448, "layer": 1 / 1.32}.get(case["kind"], SHARE[case["dtype"]])
    return {"bytes": raw * (1 + share), "flops": 0.0}
