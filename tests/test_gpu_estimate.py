"""GPU parity of the device-side sigma estimates and table choice against the oracle.

sigma is floating point (FP64 sums in a different order): tolerance 1e-10 relative, derived from
N * 2^-53 growth of a recursive FP64 sum over <= 2^27 values with |mean| <= sigma.  The table is
an integer decision taken from sigma in FP64 on both sides; inputs are chosen away from the
decision boundaries (sigma = 0.82335 * 2^k) so the tolerance cannot flip it.  Compressing with
the device table must give exactly the bytes of compressing with the oracle's table.
The robust estimate (median of the magnitudes) is a count followed by one FP64 division by the same
constant on both sides: its sigma must be equal bit for bit.
"""
import math

import numpy as np
import pytest
import torch

import oracle
from oracle import sigma as osg
import paper_2604_27844_amd.binding as z
from paper_2604_27844_amd import workloads as W

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import DEV, replayed, to_device_words


def _estimate(d_in, n, dtype):
    d_tab = torch.full((8,), 0xEE, dtype=torch.uint8, device=DEV)
    d_sig = torch.zeros(1, dtype=torch.float64, device=DEV)
    d_ws = torch.empty(z.zipccl_estimate_workspace_size(), dtype=torch.uint8, device=DEV)
    z.zipccl_estimate_table(d_in, n, dtype, d_tab, d_sig, d_ws)
    torch.cuda.synchronize()
    return d_tab, list(d_tab.cpu().numpy()), float(d_sig.item())


def _estimate_robust(d_in, n, dtype):
    d_tab = torch.full((8,), 0xEE, dtype=torch.uint8, device=DEV)
    d_sig = torch.zeros(1, dtype=torch.float64, device=DEV)
    d_ws = torch.full((z.zipccl_estimate_robust_workspace_size(),), 0x77, dtype=torch.uint8, device=DEV)   # garbage in
    z.zipccl_estimate_table_robust(d_in, n, dtype, d_tab, d_sig, d_ws)
    torch.cuda.synchronize()
    return d_tab, list(d_tab.cpu().numpy()), float(d_sig.item())


def _compress_with_device_table_equals_oracle(w, d_in, d_tab, dec):
    cap = z.zipccl_max_compressed_size(w.n_elems, w.dtype, w.n_chunks, w.chunk_elems)
    d_out = torch.full((cap,), 0xA5, dtype=torch.uint8, device=DEV)
    d_cb = torch.zeros(w.n_chunks, dtype=torch.int64, device=DEV)
    d_ws = torch.empty(z.zipccl_compress_workspace_size(w.n_elems, w.dtype, w.n_chunks, w.chunk_elems),
                       dtype=torch.uint8, device=DEV)
    z.zipccl_compress_device_table(d_in, w.n_elems, w.dtype, w.n_chunks, w.chunk_elems, d_tab, d_out, d_cb, d_ws)
    torch.cuda.synchronize()
    ref, ref_cb, off = oracle.compress(w.data, w.dtype, dec, w.n_chunks, w.chunk_elems)
    got = d_out.cpu().numpy()
    assert np.array_equal(d_cb.cpu().numpy().astype(np.uint64), ref_cb)
    for c in range(w.n_chunks):
        a, b = int(off[c]), int(off[c]) + int(ref_cb[c])
        assert np.array_equal(got[a:b], ref[a:b]), c
    return w.nbytes / float(ref_cb.sum())


def _away_from_boundary(s):
    frac = (math.log2(s / 0.82335)) % 1.0
    return min(frac, 1 - frac) > 1e-6


@pytest.mark.parametrize("name,scale", [("c1", 1.0), ("c2", 1 / 8), ("c3", 1 / 32), ("c4", 1 / 64), ("c5", 1 / 64),
                                        ("c5_fp32", 1 / 32)])
def test_estimate_matches_oracle_on_workloads(name, scale):
    w = W.make(name, scale)
    dec, s = osg.estimate_table(w.data, w.dtype)
    assert _away_from_boundary(s)
    d_in = to_device_words(w.data)
    d_tab, got_dec, got_s = _estimate(d_in, w.n_elems, w.dtype)
    assert got_s == pytest.approx(s, rel=1e-10)
    assert got_dec == list(dec)
    _compress_with_device_table_equals_oracle(w, d_in, d_tab, dec)


def test_estimate_edge_cases():
    rng = np.random.default_rng(3)
    cases = {
        "two values": np.array([0x3F80, 0x4040], dtype=np.uint16),
        "odd start / tail": W.f32_to_bf16_words(rng.standard_normal(12345, dtype=np.float32) * np.float32(3.0)),
        "nonzero mean": W.f32_to_bf16_words(rng.standard_normal(50000, dtype=np.float32) * np.float32(0.05) + np.float32(1.0)),
        "constant": np.full(1000, 0x3F80, dtype=np.uint16),
        "one value": np.array([0x3F80], dtype=np.uint16),
        "with inf": np.array([0x3F80, 0x7F80, 0x3F80, 0x0000], dtype=np.uint16),
        "empty": np.zeros(0, dtype=np.uint16),
    }
    for label, x in cases.items():
        dec, s = osg.estimate_table(x, z.BF16)
        d_in = to_device_words(x)
        # a view that starts 2 bytes into an allocation
        d_off = torch.zeros(x.size + 1, dtype=torch.int16, device=DEV)
        d_off[1:] = d_in
        for d in (d_in, d_off[1:]):
            _, got_dec, got_s = _estimate(d, x.size, z.BF16)
            assert got_dec == list(dec), label
            if math.isnan(s):
                assert math.isnan(got_s), label
            else:
                assert got_s == pytest.approx(s, rel=1e-10, abs=1e-300), label


@pytest.mark.parametrize("dtype", [z.BF16, z.FP32])
@pytest.mark.parametrize("n", [3, 7, 8, 9, 4095, 4096, 4097, 4 * 4096 + 13, 2048 * 4096 - 1, 2048 * 4096 + 5, 3 * 2048 * 4096 + 7, (1 << 25) + 3])
def test_estimate_at_the_edges_of_pieces_and_workgroups(dtype, n):
    """Remainders of a 16-byte piece, of a thread's pieces in flight and of the grid, at every alignment of the start."""
    rng = np.random.default_rng(n)
    x = (rng.standard_normal(n, dtype=np.float32) * np.float32(0.3) + np.float32(0.7)).astype(np.float32)
    words = W.f32_to_bf16_words(x) if dtype == z.BF16 else x.view(np.uint32)
    dec, s = osg.estimate_table(words, dtype)
    d_in = to_device_words(words)
    for off in (0, 1, 2, 3):
        d = torch.full((n + 8,), -1, dtype=d_in.dtype, device=DEV)                # NaNs around it
        d[off:off + n] = d_in
        _, got_dec, got_s = _estimate(d[off:off + n], n, dtype)
        assert got_s == pytest.approx(s, rel=1e-10), off
        assert got_dec == list(dec) or not _away_from_boundary(s)


def test_plain_estimate_far_from_zero_mean_does_not_cancel():
    """Sums are taken of x minus the first value, so a tensor whose mean dwarfs its spread keeps its sigma:
    a constant that is not a power of two gives exactly 0 (lowest window), mean 1000 with sigma 0.001 in fp32
    gives the oracle's two-pass value."""
    const = np.full(100000, 0x3DCD, dtype=np.uint16)                      # bf16 0.1
    dec, s = osg.estimate_table(const, z.BF16)
    assert s == 0.0 and list(dec) == [0, 1, 2, 3, 4, 5, 6, 7]
    _, got_dec, got_s = _estimate(to_device_words(const), const.size, z.BF16)
    assert got_s == 0.0 and got_dec == list(dec)
    rng = np.random.default_rng(8)
    far = (np.float32(1000.0) + rng.standard_normal(1 << 20, dtype=np.float32) * np.float32(1e-3)).astype(np.float32)
    dec, s = osg.estimate_table(far.view(np.uint32), z.FP32)
    assert 0.9e-3 < s < 1.1e-3 and _away_from_boundary(s)
    _, got_dec, got_s = _estimate(to_device_words(far.view(np.uint32)), far.size, z.FP32)
    assert got_s == pytest.approx(s, rel=1e-9) and got_dec == list(dec)


@pytest.mark.parametrize("name,scale", [("c1", 1.0), ("c2", 1 / 8), ("c3", 1 / 32), ("c4", 1 / 64), ("c5", 1 / 64),
                                        ("c5_fp32", 1 / 32)])
def test_robust_estimate_matches_oracle_on_workloads(name, scale):
    w = W.make(name, scale)
    print(f"[robust] {w.name} n={w.n_elems}", flush=True)
    dec, s = osg.robust_table(w.data, w.dtype)
    d_in = to_device_words(w.data)
    d_tab, got_dec, got_s = _estimate_robust(d_in, w.n_elems, w.dtype)
    assert got_s == s                                          # exact: a count and one division
    assert got_dec == list(dec)
    ratio = _compress_with_device_table_equals_oracle(w, d_in, d_tab, dec)
    nominal = w.nbytes / float(oracle.compress(w.data, w.dtype, oracle.build_table(w.sigma), w.n_chunks, w.chunk_elems)[1].sum())
    assert ratio >= nominal * 0.99, (ratio, nominal)           # the window of the nominal sigma, or as good


def test_robust_estimate_edge_cases():
    rng = np.random.default_rng(9)
    allpat = np.arange(65536, dtype=np.uint16)
    cases = {
        "empty": np.zeros(0, dtype=np.uint16),
        "zeros only": np.array([0x0000, 0x8000] * 50, dtype=np.uint16),
        "inf and nan only": np.array([0x7F80, 0xFF80, 0x7FC0, 0xFFFF], dtype=np.uint16),
        "one value": np.array([0xC0A0], dtype=np.uint16),
        "two values": np.array([0x3F80, 0x4040], dtype=np.uint16),
        "subnormals": np.array([0x0001, 0x0002, 0x0003, 0x8004], dtype=np.uint16),
        "every pattern": allpat,
        "every pattern, shuffled, odd length": rng.permutation(allpat)[:65001],
        "tail after vector part": W.f32_to_bf16_words(rng.standard_normal(300007, dtype=np.float32) * np.float32(3.0)),
        "mostly zeros": np.where(rng.random(200000) < 0.9, 0, W.f32_to_bf16_words(rng.standard_normal(200000, dtype=np.float32))).astype(np.uint16),
    }
    for label, x in cases.items():
        print(f"[robust edge] {label} n={x.size}", flush=True)
        dec, s = osg.robust_table(x, z.BF16)
        d_in = to_device_words(x)
        d_off = torch.zeros(x.size + 1, dtype=torch.int16, device=DEV)     # a view 2 bytes into an allocation
        d_off[1:] = d_in
        for d in (d_in, d_off[1:]):
            _, got_dec, got_s = _estimate_robust(d, x.size, z.BF16)
            assert got_dec == list(dec), label
            assert (math.isnan(s) and math.isnan(got_s)) or got_s == s, (label, got_s, s)
    f = rng.integers(0, 2 ** 32, 100003, dtype=np.uint64).astype(np.uint32)                  # fp32 bit patterns
    dec, s = osg.robust_table(f, z.FP32)
    _, got_dec, got_s = _estimate_robust(to_device_words(f), f.size, z.FP32)
    assert got_dec == list(dec) and got_s == s
    with pytest.raises(z.ZipcclError) as ei:
        d_small = torch.zeros(1024, dtype=torch.uint8, device=DEV)
        z.zipccl_estimate_table_robust(to_device_words(f), f.size, z.FP32, torch.zeros(8, dtype=torch.uint8, device=DEV),
                                       None, d_small)
    assert ei.value.code == 3


def _chunk_tables_case(x, dtype, ce, label):
    """Device per-chunk tables == oracle per-chunk tables (sigma bit-equal), and compressing with them gives, slot
    by slot, the bytes the oracle produces for that chunk alone with that chunk's table."""
    C = len(ce)
    n = int(x.size)
    print(f"[chunk tables] {label}: n={n} chunks={C}", flush=True)
    decs, sig = osg.robust_chunk_tables(x, dtype, C, ce)
    d_in = to_device_words(x)
    d_tabs = torch.full((8 * C,), 0xEE, dtype=torch.uint8, device=DEV)
    d_sig = torch.zeros(C, dtype=torch.float64, device=DEV)
    d_ews = torch.full((z.zipccl_estimate_chunk_tables_workspace_size(C),), 0x77, dtype=torch.uint8, device=DEV)
    z.zipccl_estimate_chunk_tables(d_in, n, dtype, C, ce, d_tabs, d_sig, d_ews)
    torch.cuda.synchronize()
    assert np.array_equal(d_tabs.cpu().numpy().reshape(C, 8), decs), label
    got_sig = d_sig.cpu().numpy()
    assert np.array_equal(np.isnan(got_sig), np.isnan(sig)) and np.array_equal(got_sig[~np.isnan(sig)], sig[~np.isnan(sig)]), label
    cap = z.zipccl_max_compressed_size(n, dtype, C, ce)
    off = z.zipccl_chunk_slot_offsets(n, dtype, C, ce)
    for captured, reread in ((False, False), (False, True), (True, False), (True, True)):
        d_out = torch.full((cap,), 0xA5, dtype=torch.uint8, device=DEV)
        d_cb = torch.zeros(C, dtype=torch.int64, device=DEV)
        d_ws = torch.empty(z.zipccl_compress_workspace_size(n, dtype, C, ce), dtype=torch.uint8, device=DEV)
        wsb = z.zipccl_compress_min_workspace_size(n, dtype, C, ce) if reread else None
        call = lambda: z.zipccl_compress_chunk_tables(d_in, n, dtype, C, ce, d_tabs, d_out, d_cb, d_ws, workspace_bytes=wsb)
        if captured:
            replayed(call)
        else:
            call()
        torch.cuda.synchronize()
        got, got_cb = d_out.cpu().numpy(), d_cb.cpu().numpy()
        start = 0
        for c in range(C):
            ref, ref_cb, _ = oracle.compress(x[start:start + int(ce[c])], dtype, decs[c])
            assert int(got_cb[c]) == int(ref_cb[0]), (label, c)
            a = int(off[c])
            assert np.array_equal(got[a:a + int(ref_cb[0])], ref[:int(ref_cb[0])]), (label, c)
            start += int(ce[c])
        d_back = torch.zeros_like(d_in)
        d_st = torch.zeros(1, dtype=torch.int32, device=DEV)
        z.zipccl_decompress(d_out, d_back, n, dtype, C, ce, d_st)
        torch.cuda.synchronize()
        assert int(d_st.item()) == 0 and torch.equal(d_back, d_in), label
    return x.nbytes / float(got_cb.sum())


def test_chunk_tables_match_oracle_and_follow_each_chunks_scale():
    rng = np.random.default_rng(10)
    sigmas = [1e-4, 0.02, 1.0, 37.0, 0.02]
    ce = np.array([30000, 8192 * 3 + 1, 50001, 0, 12345], dtype=np.uint64)      # odd sizes: unaligned chunk starts; one empty
    x = np.concatenate([W.f32_to_bf16_words(rng.standard_normal(int(n), dtype=np.float32) * np.float32(s)) for n, s in zip(ce, sigmas)])
    ratio = _chunk_tables_case(x, z.BF16, ce, "scales 1e-4 .. 37, bf16")
    assert ratio > 1.38
    f = np.concatenate([(rng.standard_normal(int(n), dtype=np.float32) * np.float32(s)).view(np.uint32) for n, s in zip(ce, sigmas)])
    _chunk_tables_case(f, z.FP32, ce, "scales 1e-4 .. 37, fp32")
    w = W.make("c3", 1 / 32)                                                     # 64 ragged chunks
    _chunk_tables_case(w.data, w.dtype, w.chunk_elems, w.name)
    many = W.f32_to_bf16_words(rng.standard_normal(300 * 700, dtype=np.float32))  # more chunks than one launch holds
    _chunk_tables_case(many, z.BF16, np.full(300, 700, dtype=np.uint64), "300 chunks")
    tiny = np.array([0x3F80, 0x0000, 0x7F80, 0x4000, 0xC000, 0x0001, 0x4040], dtype=np.uint16)
    _chunk_tables_case(tiny, z.BF16, np.array([1, 2, 0, 4], dtype=np.uint64), "tiny chunks")
    # chunks of more than 508 groups: several workgroups per chunk, a finish kernel, a zeroed histogram in the workspace
    ce_big = np.array([700_001, 0, 1024 * 512 + 1, 1024 * 512, 40_000], dtype=np.uint64)
    sig_big = [0.02, 1.0, 3.0, 1e-3, 0.5]
    big = np.concatenate([W.f32_to_bf16_words(rng.standard_normal(int(n), dtype=np.float32) * np.float32(s)) for n, s in zip(ce_big, sig_big)])
    _chunk_tables_case(big, z.BF16, ce_big, "chunks past one workgroup's share")


def _sampled_case(x, dtype, ce, stride, label):
    """Tables and sigmas from the sample of every chunk must be the oracle's, bit for bit (the estimate is a count)."""
    C = len(ce)
    n = int(x.size)
    print(f"[sampled tables] {label}: n={n} chunks={C} stride={stride}", flush=True)
    decs, sig = osg.robust_chunk_tables_sampled(x, dtype, C, [int(v) for v in ce], stride=stride)
    d_in = to_device_words(x)
    d_tabs = torch.full((8 * C,), 0xEE, dtype=torch.uint8, device=DEV)
    d_sig = torch.zeros(C, dtype=torch.float64, device=DEV)
    d_ews = torch.full((z.zipccl_estimate_chunk_tables_workspace_size(C),), 0x77, dtype=torch.uint8, device=DEV)
    z.zipccl_estimate_chunk_tables_sampled(d_in, n, dtype, C, ce, stride, d_tabs, d_sig, d_ews)
    torch.cuda.synchronize()
    got_sig = d_sig.cpu().numpy()
    assert np.array_equal(np.isnan(got_sig), np.isnan(sig)), (label, got_sig, sig)
    assert np.array_equal(got_sig[~np.isnan(sig)], sig[~np.isnan(sig)]), (label, got_sig, sig)
    assert np.array_equal(d_tabs.cpu().numpy().reshape(C, 8), decs), label


def test_sampled_chunk_tables_match_oracle():
    rng = np.random.default_rng(12)
    # chunk lengths around the group and block sizes, odd lengths (chunk starts that are only element-aligned: read
    # value by value), an empty chunk, a chunk shorter than one group, a last group cut short, a last block whose
    # group lies past the end
    ce = np.array([512 * 64 + 7, 0, 300, 512 * 16 * 5, 512 * 23 + 100, 512 * 23, 99_999, 8], dtype=np.uint64)
    sig = [1e-3, 1.0, 5.0, 0.3, 0.02, 0.02, 2.0, 1.0]
    for dtype in (z.BF16, z.FP32):
        f = [rng.standard_normal(int(n), dtype=np.float32) * np.float32(s) for n, s in zip(ce, sig)]
        x = np.concatenate([W.f32_to_bf16_words(v) if dtype == z.BF16 else v.view(np.uint32) for v in f])
        for stride in (1, 2, 16, 64, 4096):
            _sampled_case(x, dtype, ce, stride, f"ragged dtype={dtype}")
    # one chunk, aligned: the vector path, several workgroups, four groups in flight per wave and a ragged end
    for dtype, n in ((z.BF16, 512 * 16 * 700 + 512 * 5 + 33), (z.FP32, 512 * 16 * 300 + 17)):
        f = rng.standard_normal(n, dtype=np.float32) * np.float32(0.02)
        f[::997] = 0.0
        f[5::4001] = np.inf
        x = W.f32_to_bf16_words(f) if dtype == z.BF16 else f.view(np.uint32).copy()
        for stride in (4, 16):
            _sampled_case(x, dtype, np.array([n], dtype=np.uint64), stride, f"one chunk dtype={dtype}")
    # more chunks than one launch holds
    many = W.f32_to_bf16_words(rng.standard_normal(300 * 2048, dtype=np.float32))
    _sampled_case(many, z.BF16, np.full(300, 2048, dtype=np.uint64), 2, "300 chunks")
    # either side of the size up to which one workgroup takes a chunk's sample on its own (512 sampled groups)
    edge = W.f32_to_bf16_words(rng.standard_normal(4 * 512 * 512 + 600, dtype=np.float32) * np.float32(0.3))
    for n in (512 * 512, 512 * 512 + 1):
        _sampled_case(edge[:n], z.BF16, np.array([n], dtype=np.uint64), 1, f"one chunk of {n} values")
        _sampled_case(edge[:4 * n], z.BF16, np.array([4 * n], dtype=np.uint64), 4, f"one chunk of {4 * n} values")


@pytest.mark.parametrize("name,scale", [("c2", 1 / 8), ("c3", 1 / 32), ("c4", 1 / 64), ("c5", 1 / 64), ("c5_fp32", 1 / 32)])
def test_sampled_tables_on_workloads_are_the_full_estimates(name, scale):
    """On the benchmark's workloads (outlier columns, gain rows, heavy tails, ragged chunks) a sample of one group
    in 16 picks the window the whole tensor picks, per chunk and for the tensor as one chunk."""
    w = W.make(name, scale)
    ce = w.chunk_elems if w.chunk_elems is not None else np.full(w.n_chunks, w.n_elems // w.n_chunks, dtype=np.uint64)
    _sampled_case(w.data, w.dtype, ce, 16, w.name)
    _sampled_case(w.data, w.dtype, np.array([w.n_elems], dtype=np.uint64), 16, w.name + " as one chunk")
    d_in = to_device_words(w.data)
    d_tab = torch.zeros(8, dtype=torch.uint8, device=DEV)
    d_full = torch.zeros(8, dtype=torch.uint8, device=DEV)
    d_ews = torch.empty(z.zipccl_estimate_robust_workspace_size(), dtype=torch.uint8, device=DEV)
    z.zipccl_estimate_chunk_tables_sampled(d_in, w.n_elems, w.dtype, 1, None, 16, d_tab, None, d_ews)
    z.zipccl_estimate_table_robust(d_in, w.n_elems, w.dtype, d_full, None, d_ews)
    torch.cuda.synchronize()
    assert torch.equal(d_tab, d_full), w.name


def test_sampled_estimate_seeded_fuzz():
    """Random splits (empty, tiny, around the group, block and one-workgroup sizes), strides, scales, zeros and
    infinities, both dtypes, inputs that are only element-aligned: tables and sigmas bit-equal to the oracle's."""
    rng = np.random.default_rng(77)
    sizes = [0, 1, 7, 511, 512, 513, 1000, 4096, 8191, 8193, 40000, 100003, 262144, 262145, 300001, 1_000_003]
    for case in range(80):
        dtype = int(rng.integers(0, 2))
        C = int(rng.integers(1, 7))
        ce = rng.choice(sizes, size=C).astype(np.uint64)
        n = int(ce.sum())
        stride = int(2 ** rng.integers(0, 13))
        f = np.concatenate([rng.standard_normal(int(k), dtype=np.float32) * np.float32(np.exp(rng.uniform(-12, 6))) for k in ce])
        if n and rng.integers(0, 3) == 0:
            f[rng.integers(0, n, max(1, n // 20))] = 0.0
        if n and rng.integers(0, 4) == 0:
            f[rng.integers(0, n, max(1, n // 100))] = np.inf
        x = W.f32_to_bf16_words(f) if dtype == z.BF16 else f.view(np.uint32).copy()
        off = int(rng.integers(0, 2))
        print(f"[sampled fuzz {case}] dtype={dtype} chunks={[int(v) for v in ce]} stride={stride} offset={off}", flush=True)
        decs, sig = osg.robust_chunk_tables_sampled(x, dtype, C, [int(v) for v in ce], stride=stride)
        d_all = torch.zeros(n + 1, dtype=torch.int16 if dtype == z.BF16 else torch.int32, device=DEV)
        if n:
            d_all[off:off + n] = to_device_words(x)
        d_in = d_all[off:off + max(n, 1)]
        d_tabs = torch.full((8 * C,), 0xEE, dtype=torch.uint8, device=DEV)
        d_sig = torch.zeros(C, dtype=torch.float64, device=DEV)
        d_ews = torch.full((z.zipccl_estimate_chunk_tables_workspace_size(C),), 0x77, dtype=torch.uint8, device=DEV)
        z.zipccl_estimate_chunk_tables_sampled(d_in, n, dtype, C, ce, stride, d_tabs, d_sig, d_ews)
        torch.cuda.synchronize()
        got = d_sig.cpu().numpy()
        assert np.array_equal(np.isnan(got), np.isnan(sig)) and np.array_equal(got[~np.isnan(sig)], sig[~np.isnan(sig)]), case
        assert np.array_equal(d_tabs.cpu().numpy().reshape(C, 8), decs), case


@pytest.mark.parametrize("n", [5000, 200_007, 300_007])       # one kernel; the wide window; the narrow one
def test_robust_rank_at_the_edges_of_the_bins(n):
    """The rank's bin at the ends of what counts and of every unit the search works in (4 bins of a thread, 256 of a
    wave, 4096 of a step), alone and between neighbours: sigma bit-equal to the oracle's (a count)."""
    rng = np.random.default_rng(21)
    for b in (1, 2, 3, 4, 5, 255, 256, 257, 1023, 1024, 4095, 4096, 4097, 0x3F80, 0x7EFF, 0x7F00, 0x7F7E, 0x7F7F):
        for below, above in ((0, 0), (0.3, 0.1), (0.4999, 0.4999)):
            r = rng.random(n)
            x = np.where(r < below, max(b - 1, 1), np.where(r > 1 - above, min(b + 1, 0x7F7F), b)).astype(np.uint16)
            x[rng.integers(0, n, n // 50)] = 0x8000
            x[rng.integers(0, n, n // 50)] = 0x7F80
            x ^= (rng.integers(0, 2, n).astype(np.uint16) << np.uint16(15))
            print(f"[rank edges] n={n} bin={b:#x} below={below} above={above}", flush=True)
            dec, s = osg.robust_table(x, z.BF16)
            _, got_dec, got_s = _estimate_robust(to_device_words(x), n, z.BF16)
            assert got_s == s and got_dec == list(dec), (b, below, above)


def test_robust_counts_past_32_bits():
    """2^32 + 7 equal values and three smaller ones: the count of their bin does not fit 32 bits.  The median is the
    value itself, whatever else rounds."""
    n = 2 ** 32 + 10
    d_in = torch.full((n,), 0x3F81, dtype=torch.int16, device=DEV)            # bf16 1.0078125
    d_in[5:8] = 0x3C00
    print(f"[robust wide] n={n}", flush=True)
    _, dec, s = _estimate_robust(d_in, n, z.BF16)
    assert s == 1.0078125 / 0.6744897501960817
    assert dec == list(bytes(z.zipccl_build_table(s).dec))


@pytest.mark.parametrize("dtype", [z.BF16, z.FP32])
def test_estimate_of_chunks_shared_by_a_few_workgroups(dtype):
    """Chunks of one workgroup to a few (32 groups to count each, up to 508 in all without a shared histogram for a second
    count), counts all in one bin, ragged and element-aligned chunks beside empty ones: bit-equal to the oracle."""
    rng = np.random.default_rng(31)
    G = 512
    for stride, groups in ((1, (159, 160, 161, 254, 255)), (1, (381, 382, 507, 508)), (1, (509, 3)), (4, (4 * 160, 4 * 508 - 1, 4 * 508))):
        ce = np.array([g * G for g in groups] + [0, 5, 160 * G - 7], dtype=np.uint64)
        x = np.concatenate([rng.standard_normal(int(k), dtype=np.float32) * np.float32(np.exp(rng.uniform(-8, 4))) for k in ce])
        x = W.f32_to_bf16_words(x) if dtype == z.BF16 else x.view(np.uint32).copy()
        _sampled_case(x, dtype, ce, stride, f"sizes {groups} dtype={dtype}")
        _sampled_case(x[1:], dtype, np.concatenate([[ce[0] - 1], ce[1:]]).astype(np.uint64), stride, f"sizes {groups} skewed dtype={dtype}")
    for word in (0x3F80, 0x0000, 0x7F7F, 0x0001):                    # all counts in one bin, or in none
        x = np.full(508 * G, word, dtype=np.uint16) if dtype == z.BF16 else np.full(508 * G, word << 16, dtype=np.uint32)
        x[7], x[1000] = 0, 0
        _sampled_case(x, dtype, np.array([x.size], dtype=np.uint64), 1, f"one value {word:#x} dtype={dtype}")
    many = rng.standard_normal(100 * 200 * G, dtype=np.float32)      # 100 chunks: two workgroups each
    _sampled_case(W.f32_to_bf16_words(many) if dtype == z.BF16 else many.view(np.uint32).copy(), dtype,
                  np.full(100, 200 * G, dtype=np.uint64), 1, f"100 chunks dtype={dtype}")


@pytest.mark.parametrize("dtype", [z.BF16, z.FP32])
@pytest.mark.parametrize("ce,stride", [((200 * 512 - 3,), 1), ((508 * 512 + 1,), 1), ((1 << 21,), 1), ((1 << 21, 5, 0, 300_000), 4),
                                       ((600 * 512, 70_001, 1 << 20), 1), ((90 * 512,) * 20 + (181 * 512,), 1),
                                       ((2048 * 512,) + (70_001,) * 8, 1), ((2048 * 512,) + (20_001,) * 31, 1), ((2049 * 512,) + (20_001,) * 31, 1)])
def test_estimate_of_chunks_whose_small_sample_misleads(dtype, ce, stride):
    """The windowed count looks at 16 values of each of 64 strata before it counts: chunks where those say nothing about
    the median.  The sampled values alone at another scale, above or below the rest; everything zero but a short run; two
    halves far apart, so that the median is the largest value of the one or the smallest of the other; chunks that do
    not mislead beside them.  Bit-equal to the oracle."""
    rng = np.random.default_rng(71)
    base = rng.standard_normal(sum(ce), dtype=np.float32)
    starts = np.concatenate([[0], np.cumsum(ce)])
    def sampled(n):
        length = (n - 16) // 64
        k = np.arange(64, dtype=np.uint64)
        at = k * np.uint64(length) + ((k * np.uint64(2654435761) % np.uint64(2 ** 32)) * np.uint64(length) >> np.uint64(32))
        return (at.astype(np.int64)[:, None] + np.arange(16)).ravel()
    for kind in ("high", "low", "run", "halves"):
        x = base.copy()
        for c, n in enumerate(ce):
            if n < 1024 or c % 2:
                continue
            part = x[starts[c]:starts[c] + n]
            if kind in ("high", "low"):
                part[sampled(n)] *= np.float32(1e6 if kind == "high" else 1e-6)
            elif kind == "run":
                part[:n // 3] = 0.0
                part[n // 3 + 700:] = 0.0
            else:
                part[::2] = np.abs(part[::2]) * np.float32(1e6) + 1
        words = W.f32_to_bf16_words(x) if dtype == z.BF16 else x.view(np.uint32).copy()
        _sampled_case(words, dtype, np.array(ce, dtype=np.uint64), stride, f"misled {kind} {ce[:3]} dtype={dtype}")


@pytest.mark.parametrize("dtype", [z.BF16, z.FP32])
def test_estimate_of_rows_of_different_scales_is_counted_once(dtype):
    """Rows of 4096 values whose scales are log-normal, spread by e^1 to e^3, sparse ones, and tokens of 7168 sampled per chunk: the
    windowed count looks again where its sample's values lie far apart, so that the window holds the rank and nothing
    is counted a second time.  A second count leaves its workgroups' number behind the chunk's first window of counts."""
    rng = np.random.default_rng(73)
    def scaled(n, row, s):
        return rng.standard_normal(n, dtype=np.float32) * np.repeat(np.exp(s * rng.standard_normal(n // row)), row).astype(np.float32)
    recounted = lambda ws, wide: int((ws.view(torch.int32).view(-1, 65536)[:, 500 if wide else 116] != 0).sum())       # 256 KiB per chunk
    words = lambda x: W.f32_to_bf16_words(x) if dtype == z.BF16 else x.view(np.uint32).copy()
    cases = [(scaled(1 << 21, 4096, s), 1, 1) for s in (1, 1, 1.5, 1.5, 2, 2, 2, 2, 3, 3, 3, 3)]
    cases += [(scaled(1 << 18, 4096, 2), 1, 1), (scaled(8 * 192 * 7168, 7168, 2), 8, 4), (scaled(16 * 640 * 1024, 1024, 2), 16, 2)]
    sparse = rng.standard_normal(1 << 21, dtype=np.float32)
    sparse[rng.random(1 << 21) < 0.93] = 0.0
    cases.append((sparse, 1, 1))
    again = 0
    for x, chunks, stride in cases:
        x = words(x)
        d_tabs = torch.zeros(8 * chunks, dtype=torch.uint8, device=DEV)
        d_sig = torch.zeros(chunks, dtype=torch.float64, device=DEV)
        d_ews = torch.full((z.zipccl_estimate_chunk_tables_workspace_size(chunks),), 0x77, dtype=torch.uint8, device=DEV)
        z.zipccl_estimate_chunk_tables_sampled(to_device_words(x), x.size, dtype, chunks, None, stride, d_tabs, d_sig, d_ews)
        torch.cuda.synchronize()
        groups = -(-(x.size // chunks) // (512 * stride))
        again += recounted(d_ews, min(-(-groups // 32), 256 // chunks) <= 16)              # workgroups per chunk
        decs, sig = osg.robust_chunk_tables_sampled(x, dtype, chunks, [x.size // chunks] * chunks, stride=stride)
        assert np.array_equal(d_sig.cpu().numpy(), sig) and np.array_equal(d_tabs.cpu().numpy().reshape(chunks, 8), decs)
    assert again == 0


def test_estimate_of_a_tensor_of_zero_rows_mostly_takes_a_few_times_the_usual():
    """One group in a thousand of 2^24 values holds any: the sample misses them and everything is counted a second time.  What
    that takes must not grow with the zeros, which do not count but would all be added to one word: 3 times the same call on normal
    values, 34 times when they were.  (10: the device's own events, an average of 20 calls.)"""
    n = 1 << 24
    g = torch.Generator(device=DEV)
    g.manual_seed(79)
    x = torch.empty(n, dtype=torch.float32, device=DEV).normal_(generator=g)
    sparse = x.clone()
    sparse.view(-1, 512)[torch.rand(n // 512, device=DEV, generator=g) < 0.999] = 0.0
    tab, ws = torch.zeros(8, dtype=torch.uint8, device=DEV), torch.empty(z.zipccl_estimate_robust_workspace_size(), dtype=torch.uint8, device=DEV)
    def time_of(d):
        d = d.to(torch.bfloat16)
        call = lambda: z.zipccl_estimate_table_robust(d, n, z.BF16, tab, None, ws)
        call()
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        for _ in range(20):
            call()
        end.record()
        end.synchronize()
        return start.elapsed_time(end)
    assert time_of(sparse) < 10 * time_of(x)
    words = sparse.to(torch.bfloat16).view(torch.int16).cpu().numpy().view(np.uint16)
    dec, s = osg.robust_table(words, z.BF16)
    _, got_dec, got_s = _estimate_robust(to_device_words(words), n, z.BF16)
    assert got_s == s and got_dec == list(dec)
