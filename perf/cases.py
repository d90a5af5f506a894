"""The codec's work as a user of this library has it do: the cases that are timed.

A case is one collective's device-side step: the tensor is on the GPU, the buffers and the workspace are allocated
once (as a training or serving loop keeps them), and one pass is the library calls of that step through
`paper_2604_27844_amd.binding`, on the current stream.

    op        compress   table given by sigma                              -> compressed slots, chunk_bytes
              compress_static  the same with the library's own workspace   -> the same
              auto       robust per-tensor table on the device, then compress with it
              auto_chunks  sampled per-chunk tables (stride), then compress with them
              decompress slots                                             -> tensor, status
              reduce     `chunks` peers' slots of n values each            -> FP32 sum (out: fp32 / bf16), status
              estimate   table from the sample standard deviation
              estimate_chunks  exact robust table of every chunk
    dtype     bf16 / fp32: type of the tensor
    n         values of the tensor (reduce: values of each peer's contribution)
    chunks    peer chunks of the call
    unit      values a chunk is a multiple of (a token's hidden size, a row; 1 = any element); 0 = equal split
    kind      what the values are like (fill())
"""
import math

import numpy as np
import torch

import paper_2604_27844_amd.binding as z

DTYPE = {"bf16": z.BF16, "fp32": z.FP32}
BYTES = {"bf16": 2, "fp32": 4}
# nominal scale of each kind, and the share of its values outside the seven-exponent window of that scale
SIGMA = {"normal": 0.02, "hidden": 0.5, "outliers": 1.0, "grads": 1e-4, "params": 0.02}
ESCAPES = {"normal": 0.025, "hidden": 0.025, "outliers": 0.027, "grads": 0.054, "params": 0.070}


def _case(name, op, dtype, n, chunks, unit, kind, **more):
    return {"name": name, "op": op, "dtype": dtype, "n": n, "chunks": chunks, "unit": unit, "kind": kind, **more}


def listed():
    return [
        # a decoding step's activations: 32 tokens x 4096 for 8 peers; latency and launches are all there is
        _case("decode_act_compress", "compress", "bf16", 32 * 4096, 8, 0, "outliers"),
        # the receiving side of a small uneven exchange: 8 odd pieces that start at any element
        _case("small_ragged_decompress", "decompress", "bf16", 200003, 8, 1, "hidden"),
        # one small tensor (2 MiB) as a single chunk, sent without a workspace of the caller's
        _case("small_static_compress", "compress_static", "bf16", 1 << 20, 1, 0, "normal"),
        # a small gradient bucket of odd length summed from 8 peers, kept in bf16
        _case("small_ragged_reduce", "reduce", "bf16", 1000003, 8, 0, "grads", out="bf16"),
        # tensor-parallel activations, 4096 x 4096 with outlier channels, 8 row blocks: table from the data, then compress
        _case("act_auto_compress", "auto", "bf16", 4096 * 4096, 8, 0, "outliers"),
        # the same tensor on the receiving side
        _case("act_decompress", "decompress", "bf16", 4096 * 4096, 8, 0, "outliers"),
        # expert dispatch buffer: 64 experts, about 512 tokens of 7168 each, one table per expert from a sample
        _case("moe_auto_compress", "auto_chunks", "bf16", 64 * 512 * 7168, 64, 7168, "hidden", stride=16),
        # the same buffer on the receiving side
        _case("moe_decompress", "decompress", "bf16", 64 * 512 * 7168, 64, 7168, "hidden"),
        # gradient bucket: the shard's contributions of 8 peers summed in FP32
        _case("grad_reduce", "reduce", "bf16", 1 << 25, 8, 0, "grads", out="fp32"),
        # fp32 contributions of 8 peers whose shard is no whole number of tiles
        _case("fp32_ragged_reduce", "reduce", "fp32", (1 << 24) - 12345, 8, 0, "params", out="fp32"),
        # fp32 master parameters, 64 chunks, receiving side
        _case("master_fp32_decompress", "decompress", "fp32", 1 << 27, 64, 0, "params"),
        # parameter shard of 1 GiB, 64 chunks, sending side
        _case("param_compress", "compress", "bf16", 1 << 29, 64, 0, "params"),
    ]


def draw(rng):
    """A case of the same ranges: any operation, size (over its logarithm), split, type and kind of values."""
    op = rng.choice(["compress", "compress", "compress_static", "auto", "auto_chunks", "decompress", "decompress",
                     "reduce", "reduce", "estimate", "estimate_chunks"])
    dtype = rng.choice(["bf16", "bf16", "fp32"])
    kind = rng.choice(sorted(SIGMA))
    lo, hi = (14, 29 if dtype == "bf16" else 27)
    more = {}
    if op == "reduce":
        chunks = rng.choice([2, 4, 8, 8, 16])
        lo, hi = 14, (hi - 1 - math.log2(chunks))
        more["out"] = rng.choice(["fp32", "fp32", "bf16"])
        unit = 0
    else:
        chunks = rng.choice([1, 2, 8, 8, 64, 64, 200])
        unit = rng.choice([0, 0, 1, 4096, 7168]) if chunks > 1 else 0
    if op == "auto_chunks":
        more["stride"] = rng.choice([4, 16, 16, 64])
    n = int(2.0 ** rng.uniform(lo, hi))
    if op != "reduce":
        n = max(n // chunks, 1) * chunks if unit == 0 else max(n // unit, 1) * unit     # what such a split can hold
    return {"op": op, "dtype": dtype, "n": n, "chunks": chunks, "unit": unit, "kind": kind, **more}


def fill(kind, n, gen):
    """n FP32 values on the GPU.  normal: initialised weights; hidden: token vectors; outliers: activations whose
    rows of 4096 hold 8 channels 50 times as large; grads: heavy-tailed (Student t with 5 degrees of freedom) with
    1 % exact zeros; params: rows of 4096, every 20th of them gains near 1."""
    x = torch.empty(n, dtype=torch.float32, device="cuda")
    block = 1 << 26
    for s in range(0, n, block):
        part = x[s:s + block]
        part.normal_(generator=gen)
        if kind == "grads":
            chi = torch.zeros_like(part)
            for _ in range(5):
                chi += torch.empty_like(part).normal_(generator=gen).square_()
            part.mul_(chi.mul_(1 / 5).rsqrt_()).mul_(SIGMA[kind] / math.sqrt(5 / 3))
            part.masked_fill_(torch.empty_like(part).uniform_(generator=gen) < 0.01, 0.0)
        else:
            part.mul_(SIGMA[kind])
    if kind == "outliers":
        at = torch.randperm(4096, generator=gen, device="cuda")[:8]
        rows = x[:n // 4096 * 4096].view(-1, 4096)
        rows[:, at] *= 50.0
    if kind == "params":
        rows = x[:n // 4096 * 4096].view(-1, 4096)[::20]
        rows.mul_(0.05 / SIGMA[kind]).add_(1.0)
    return x


def split(case, seed):
    """Element count of every chunk as the binding takes it; None = equal split."""
    if case["op"] == "reduce" or case["unit"] == 0:
        return None
    units = case["n"] // case["unit"]
    got = np.random.default_rng(seed).multinomial(units, [1 / case["chunks"]] * case["chunks"])
    return got.astype(np.uint64) * np.uint64(case["unit"])


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    op, dt, C = case["op"], DTYPE[case["dtype"]], case["chunks"]
    n = case["n"] * (C if op == "reduce" else 1)
    ce = split(case, seed)
    x = fill(case["kind"], n, gen)
    if dt == z.BF16:
        x = x.to(torch.bfloat16)
    zeros = lambda count, kind: torch.zeros(count, dtype=kind, device="cuda")
    table = z.zipccl_build_table(SIGMA[case["kind"]], dt)
    s = {"case": case, "dt": dt, "n": n, "ce": ce, "table": table, "x": x}
    if op not in ("estimate", "estimate_chunks"):
        # room for any split of n values into C chunks: every slot adds less than 1 KiB of header and padding
        s["out"] = zeros(z.zipccl_max_compressed_size(n, dt) + 1024 * C, torch.uint8)
        s["sizes"] = zeros(C, torch.int64)
        s["ws"] = torch.empty(z.zipccl_compress_workspace_size(n, dt, C, ce), dtype=torch.uint8, device="cuda")
    if op in ("decompress", "reduce"):
        z.zipccl_compress(x, n, dt, C, ce, table, s["out"], s["sizes"], s["ws"])
        s["status"] = zeros(1, torch.int32)
        if op == "reduce":
            s["sum"] = zeros(case["n"], torch.float32 if case["out"] == "fp32" else torch.bfloat16)
        else:
            s["back"] = torch.empty_like(x)
        torch.cuda.synchronize()
        del s["x"], s["ws"]
    else:
        s["tables"] = zeros(8 * C, torch.uint8)
        s["sigmas"] = zeros(C, torch.float64)
        need = {"auto": z.zipccl_estimate_robust_workspace_size(), "estimate": z.zipccl_estimate_workspace_size()}
        s["ews"] = torch.empty(need.get(op) or z.zipccl_estimate_chunk_tables_workspace_size(C), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    case = s["case"]
    op, dt, n, C, ce = case["op"], s["dt"], s["n"], case["chunks"], s["ce"]
    if op == "compress":
        z.zipccl_compress(s["x"], n, dt, C, ce, s["table"], s["out"], s["sizes"], s["ws"])
        return s["out"], s["sizes"]
    if op == "compress_static":
        z.zipccl_compress_static(s["x"], n, dt, C, ce, s["table"], s["out"], s["sizes"])
        return s["out"], s["sizes"]
    if op == "auto":
        z.zipccl_estimate_table_robust(s["x"], n, dt, s["tables"], s["sigmas"], s["ews"])
        z.zipccl_compress_device_table(s["x"], n, dt, C, ce, s["tables"], s["out"], s["sizes"], s["ws"])
        return s["tables"], s["sigmas"], s["out"], s["sizes"]
    if op == "auto_chunks":
        z.zipccl_estimate_chunk_tables_sampled(s["x"], n, dt, C, ce, case["stride"], s["tables"], s["sigmas"], s["ews"])
        z.zipccl_compress_chunk_tables(s["x"], n, dt, C, ce, s["tables"], s["out"], s["sizes"], s["ws"])
        return s["tables"], s["sigmas"], s["out"], s["sizes"]
    if op == "decompress":
        z.zipccl_decompress(s["out"], s["back"], n, dt, C, ce, s["status"])
        return s["back"], s["status"]
    if op == "reduce":
        z.zipccl_decompress_reduce(s["out"], s["sum"], case["n"], dt, C, DTYPE[case["out"]], s["status"])
        return s["sum"], s["status"]
    if op == "estimate":
        z.zipccl_estimate_table(s["x"], n, dt, s["tables"], s["sigmas"], s["ews"])
        return s["tables"], s["sigmas"]
    z.zipccl_estimate_chunk_tables(s["x"], n, dt, C, ce, s["tables"], s["sigmas"], s["ews"])
    return s["tables"], s["sigmas"]


def work(case):
    """Bytes that every implementation moves: the tensor once and its compressed form once (sign and mantissa byte,
    three code bits, a 32-bit index entry per 512 values, one byte per value outside the window; fp32: two low bytes
    more).  No arithmetic to speak of except the reduction's additions."""
    es = BYTES[case["dtype"]]
    packed = es - 1 + 3 / 8 + 4 / z.GROUP + ESCAPES[case["kind"]]
    n = case["n"]
    if case["op"] == "reduce":
        return {"bytes": n * (case["chunks"] * packed + BYTES[case["out"]]), "flops": n * case["chunks"]}
    if case["op"] in ("estimate", "estimate_chunks"):
        return {"bytes": n * es, "flops": 0}
    return {"bytes": n * (es + packed), "flops": 0}          # an estimate in front reads what the compress reads


def tolerance(case):
    """Everything is bytes, counts or FP32 sums in a fixed order, the same for every implementation, except the
    sample standard deviation: FP64 sums in another order differ by up to 1e-15 relative (measured against
    torch.std in FP64 on every kind of values, 20 000 to 2^26 of them)."""
    if case["op"] == "estimate":
        return {"rel": 4e-15, "max": 4e-15}
    return "exact"
