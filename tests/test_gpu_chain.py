"""The chained compress, in which a tile waits for the counts of the chunk's tiles before it: lengths at the edges of its
tiles and of the words it reads, workspaces in any state, calls side by side, and the bound of the wait.  Bytes
throughout, equal to the oracle's or to those of the captured call, which takes the form without a wait."""
import ctypes
import os

import impatient_lib
import numpy as np
import pytest
import torch

import paper_2604_27844_amd.binding as z
from paper_2604_27844_amd import workloads as W

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import DEV, check_parity, gpu_compress, replayed, to_device_words

TILE = 8192


@pytest.fixture(scope="module")
def impatient():
    return ctypes.CDLL(impatient_lib.LIB if os.path.exists(impatient_lib.LIB) else impatient_lib.build())


def _values(n, dtype, seed, sigma=0.02):
    rng = np.random.default_rng(seed)
    f = rng.standard_normal(n, dtype=np.float32) * np.float32(sigma)
    f[n // 3:n // 3 + 2 * TILE + 77] = 1.0                                # a stretch of zero-points
    return W.f32_to_bf16_words(f) if dtype == z.BF16 else f.view(np.uint32).copy()


# launches of up to 256, 640 and more tiles of 8192 values; whole, one value less and more; with the larger tiles chunks of as many
# as run at a time (bf16 1024, fp32 512) and 63, 64 and 65 more, where the first total stands for the counts far back
@pytest.mark.parametrize("dtype,sizes", [
    (z.BF16, [3 * TILE]), (z.BF16, [9 * TILE - 1, 8 * TILE + 1, 0, 1]), (z.BF16, [256 * TILE]), (z.BF16, [256 * TILE + 1]),
    (z.BF16, [64 * TILE + 5] * 10), (z.BF16, [641 * TILE - 8]), (z.BF16, [7, 600 * TILE, 41 * TILE + 8191]),
    (z.BF16, [2 * TILE * 1087 + 1]), (z.BF16, [2 * TILE * 1088]), (z.BF16, [2 * TILE * 1089 - 1, 2 * TILE * 1152 + 9]),
    (z.FP32, [3 * TILE]), (z.FP32, [256 * TILE - 3]), (z.FP32, [257 * TILE]), (z.FP32, [33 * TILE + 1] * 9),
    (z.FP32, [2 * TILE * 575 + 2]), (z.FP32, [2 * TILE * 576]), (z.FP32, [2 * TILE * 577 - 1, 2 * TILE * 640 + 3]),
], ids=str)
def test_edges_of_tiles_and_of_what_a_tile_reads(dtype, sizes):
    ce = np.array(sizes, dtype=np.uint64)
    print(f"[chain] dtype={dtype} sizes={sizes}", flush=True)
    check_parity(_values(int(ce.sum()), dtype, len(sizes)), dtype, 0.02, len(ce), ce, label=str(sizes))


def test_a_workspace_that_other_calls_have_left():
    """The same workspace for calls of several shapes in turn, each twice on other values, and for captured calls between them, which leave
    the counts and prefixes of the form with a stash and of the one that reads twice where the words are."""
    shapes = [[700 * TILE], [40 * TILE + 3] * 8, [9 * TILE], [2 * TILE * 600 + 1], [5 * TILE] * 20]
    ws = torch.full((max(z.zipccl_compress_workspace_size(sum(s), z.BF16, len(s), np.array(s, dtype=np.uint64)) for s in shapes),), 0xFF,
                    dtype=torch.uint8, device=DEV)
    table = z.zipccl_build_table(0.02, z.BF16)
    for rep in range(2):
        for s in shapes:
            ce = np.array(s, dtype=np.uint64)
            n = int(ce.sum())
            print(f"[chain workspace] {rep} {s[:2]}", flush=True)
            for seed in (1, 2):
                data = _values(n, z.BF16, 10 * rep + seed)
                want, want_cb, _ = gpu_compress(data, z.BF16, 0.02, len(ce), ce, captured=True, d_ws=ws, reread=seed == 2)
                got = torch.full_like(want, 0xA5)
                got_cb = torch.zeros_like(want_cb)
                z.zipccl_compress(to_device_words(data), n, z.BF16, len(ce), ce, table, got, got_cb, ws)
                torch.cuda.synchronize()
                assert torch.equal(got, want) and torch.equal(got_cb, want_cb), (rep, s, seed)


def test_calls_side_by_side_on_several_streams():
    sizes = [[1100 * TILE + 7], [150 * TILE] * 8, [12 * TILE] * 64, [3 * TILE + 1]]
    table = z.zipccl_build_table(0.02, z.BF16)
    work = []
    for k, s in enumerate(sizes):
        ce = np.array(s, dtype=np.uint64)
        n = int(ce.sum())
        data = _values(n, z.BF16, 40 + k)
        want, want_cb, _ = gpu_compress(data, z.BF16, 0.02, len(ce), ce, captured=True)
        ws = torch.empty(z.zipccl_compress_workspace_size(n, z.BF16, len(ce), ce), dtype=torch.uint8, device=DEV)
        work.append((torch.cuda.Stream(), to_device_words(data), n, ce, want, want_cb, torch.full_like(want, 0xA5), torch.zeros_like(want_cb), ws))
    torch.cuda.synchronize()
    print("[chain streams]", flush=True)
    for _ in range(10):
        for stream, d_in, n, ce, _, _, got, got_cb, ws in work:
            with torch.cuda.stream(stream):
                z.zipccl_compress(d_in, n, z.BF16, len(ce), ce, table, got, got_cb, ws)
    torch.cuda.synchronize()
    for _, _, n, _, want, want_cb, got, got_cb, _ in work:
        assert torch.equal(got, want) and torch.equal(got_cb, want_cb), n


@pytest.mark.parametrize("dtype,sizes", [
    (z.BF16, [3 * TILE]), (z.BF16, [40 * TILE + 3] * 3), (z.BF16, [300 * TILE - 1]), (z.BF16, [100 * TILE + 1] * 8),
    (z.BF16, [2 * TILE * 1160]), (z.FP32, [40 * TILE + 1, 100 * TILE]), (z.FP32, [2 * TILE * 650 + 1]),
], ids=str)
def test_workgroups_that_look_only_once(dtype, sizes, impatient):
    """A copy of the library built so that a workgroup looks once for the counts before it and then counts what is missing itself."""
    ce = np.array(sizes, dtype=np.uint64)
    n, C = int(ce.sum()), len(ce)
    print(f"[chain impatient] dtype={dtype} sizes={sizes}", flush=True)
    data = _values(n, dtype, 70)
    want, want_cb, table = gpu_compress(data, dtype, 0.02, C, ce, captured=True)
    d_in = to_device_words(data)
    ws = torch.full((z.zipccl_compress_workspace_size(n, dtype, C, ce),), 0x5A, dtype=torch.uint8, device=DEV)
    vp, size = ctypes.c_void_p, ctypes.c_size_t
    for _ in range(3):
        got = torch.full_like(want, 0xA5)
        got_cb = torch.zeros_like(want_cb)
        rc = impatient.zipccl_compress(vp(d_in.data_ptr()), size(n), ctypes.c_int(dtype), ctypes.c_uint32(C), ce.ctypes.data_as(vp), ctypes.byref(table),
                                       vp(got.data_ptr()), size(got.numel()), vp(got_cb.data_ptr()), vp(ws.data_ptr()), size(ws.numel()),
                                       vp(torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        assert rc == 0 and torch.equal(got, want) and torch.equal(got_cb, want_cb), sizes


def test_the_way_back_to_a_total_is_as_short_in_a_long_chunk(impatient):
    """Workgroups that look only once go back to the nearest total that was told, not to the chunk's start: a chunk of 16384 of the larger tiles
    takes them no longer than 16 of 1024 (1.1 times; going back to the start of the chunk it was 4.6)."""
    n = 1 << 28
    print("[chain impatient, long chunk]", flush=True)
    x = (torch.randn(n, device=DEV) * 0.02).bfloat16()
    table = z.zipccl_build_table(0.02, z.BF16)
    vp, size = ctypes.c_void_p, ctypes.c_size_t
    took = {}
    for C in (16, 1):
        want = torch.zeros(z.zipccl_max_compressed_size(n, z.BF16, C), dtype=torch.uint8, device=DEV)
        got, want_cb, got_cb = torch.zeros_like(want), torch.zeros(C, dtype=torch.int64, device=DEV), torch.zeros(C, dtype=torch.int64, device=DEV)
        ws = torch.empty(z.zipccl_compress_min_workspace_size(n, z.BF16, C), dtype=torch.uint8, device=DEV)
        z.zipccl_compress(x, n, z.BF16, C, None, table, want, want_cb, ws)
        took[C] = []
        for _ in range(7):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            rc = impatient.zipccl_compress(vp(x.data_ptr()), size(n), ctypes.c_int(z.BF16), ctypes.c_uint32(C), vp(0), ctypes.byref(table), vp(got.data_ptr()),
                                           size(got.numel()), vp(got_cb.data_ptr()), vp(ws.data_ptr()), size(ws.numel()), vp(torch.cuda.current_stream().cuda_stream))
            end.record()
            torch.cuda.synchronize()
            assert rc == 0
            took[C].append(start.elapsed_time(end))
        assert torch.equal(got, want) and torch.equal(got_cb, want_cb)
    assert sorted(took[1])[3] < 2 * sorted(took[16])[3], took


def _all_forms(n, dtype, ce, call, label):
    """call(out, sizes, workspace, its bytes), as it is and captured, with room for a stash and without, all in one workspace and twice over:
    the same bytes from all.  Returns them."""
    C = len(ce)
    ws = torch.full((z.zipccl_compress_workspace_size(n, dtype, C, ce),), 0x5A, dtype=torch.uint8, device=DEV)
    want = None
    for captured, some in ((True, ws.numel()), (False, ws.numel()), (True, None), (False, None), (False, ws.numel())):
        print(f"[chain forms] {label} captured={captured} workspace={'full' if some else 'least'}", flush=True)
        out = torch.full((z.zipccl_max_compressed_size(n, dtype, C, ce),), 0xA5, dtype=torch.uint8, device=DEV)
        sizes = torch.zeros(C, dtype=torch.int64, device=DEV)
        some = some or z.zipccl_compress_min_workspace_size(n, dtype, C, ce)
        if captured:
            replayed(lambda: call(out, sizes, ws, some))
        else:
            call(out, sizes, ws, some)
        torch.cuda.synchronize()
        if want is None:
            want = out, sizes
        assert torch.equal(out, want[0]) and torch.equal(sizes, want[1]), (label, captured, some)
    return want


def _device_values(n, dtype, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    x = torch.randn(n, generator=gen, device=DEV).mul_(0.02)
    x[n // 3:n // 3 + 2 * TILE + 77] = 1.0                                # a stretch of zero-points
    return x.bfloat16() if dtype == z.BF16 else x


# more than 8192 tiles of bf16 values in chunks that start off cache lines: with a stash, if there is room for one; and on lines
@pytest.mark.parametrize("dtype,sizes", [
    (z.BF16, [4096 * TILE + 1, 4096 * TILE + 63]), (z.BF16, [4096 * TILE + 64, 4096 * TILE + 64, 1]), (z.BF16, [8191 * TILE - 1, TILE]),
    (z.FP32, [4096 * TILE + 1, 4096 * TILE + 63]),
], ids=str)
def test_many_tiles_on_and_off_cache_lines(dtype, sizes):
    ce = np.array(sizes, dtype=np.uint64)
    n, C = int(ce.sum()), len(ce)
    x = _device_values(n, dtype, 5)
    table = z.zipccl_build_table(0.02, dtype)
    out, sizes_got = _all_forms(n, dtype, ce, lambda out, cb, ws, some: z.zipccl_compress(x, n, dtype, C, ce, table, out, cb, ws, workspace_bytes=some), str(sizes))
    once = torch.full_like(out, 0xA5), torch.zeros_like(sizes_got)
    z.zipccl_compress_static(x, n, dtype, C, ce, table, *once)
    assert torch.equal(once[0], out) and torch.equal(once[1], sizes_got)
    back, status = torch.zeros_like(x), torch.zeros(1, dtype=torch.int32, device=DEV)
    z.zipccl_decompress(out, back, n, dtype, C, ce, status)
    as_words = torch.int16 if dtype == z.BF16 else torch.int32
    assert int(status.item()) == 0 and torch.equal(back.view(as_words), x.view(as_words))


# a table in device memory, one for all chunks (which has the smaller tiles up to 2304 tiles of bf16 and 2048 of fp32 values) or one for each
@pytest.mark.parametrize("dtype,sizes", [
    (z.BF16, [9 * TILE + 3] * 3), (z.BF16, [1152 * TILE] * 2), (z.BF16, [1152 * TILE, 1151 * TILE + 1, 1]), (z.BF16, [77, 4097 * TILE + 9, 4000 * TILE]),
    (z.FP32, [5 * TILE + 1, 9 * TILE]), (z.FP32, [2048 * TILE - 2]), (z.FP32, [700 * TILE + 5, 1349 * TILE]),
], ids=str)
def test_tables_in_device_memory(dtype, sizes):
    ce = np.array(sizes, dtype=np.uint64)
    n, C = int(ce.sum()), len(ce)
    x = _device_values(n, dtype, 6)
    off = z.zipccl_chunk_slot_offsets(n, dtype, C, ce)
    sigmas = [0.02 * 3.0 ** c for c in range(C)]
    tables = [z.zipccl_build_table(s, dtype) for s in sigmas]
    d_tables = torch.tensor([list(bytes(t.dec)) for t in tables], dtype=torch.uint8, device=DEV)
    cases = {"one": lambda out, cb, ws, some: z.zipccl_compress_device_table(x, n, dtype, C, ce, d_tables, out, cb, ws, workspace_bytes=some),
             "each": lambda out, cb, ws, some: z.zipccl_compress_chunk_tables(x, n, dtype, C, ce, d_tables, out, cb, ws, workspace_bytes=some)}
    for name, call in cases.items():
        out, cb = _all_forms(n, dtype, ce, call, f"{name} {sizes}")
        start = 0
        for c in range(C):                                                # as a call of its own, with the table on the host, makes it
            m = int(ce[c])
            alone = torch.full((z.zipccl_max_compressed_size(m, dtype),), 0xA5, dtype=torch.uint8, device=DEV)
            alone_cb = torch.zeros(1, dtype=torch.int64, device=DEV)
            ws = torch.empty(z.zipccl_compress_workspace_size(m, dtype), dtype=torch.uint8, device=DEV)
            z.zipccl_compress(x[start:start + m], m, dtype, 1, None, tables[c if name == "each" else 0], alone, alone_cb, ws)
            assert int(alone_cb.item()) == int(cb[c].item()), (name, c)
            assert torch.equal(out[int(off[c]):int(off[c]) + int(alone_cb.item())], alone[:int(alone_cb.item())]), (name, c)
            start += m
