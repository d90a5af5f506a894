/*
 * Auxiliary kernels of libzipccl.so: the sigma estimates / table choice on the device (paper section 4.1).
 */
#include <algorithm>

#include "zipccl_device.h"

namespace zipccl {
namespace {

/* The table for a given sigma by Eq.5 / Eq.2 (erf in FP64), exactly as the host builder does; a sigma that is
 * not positive and finite selects the lowest window.  Called by all 64 lanes of one wave with the same sigma: the
 * four values of erf are independent, so lanes 0..3 take one each (one after the other in a single lane they
 * are most of a small estimate's last microseconds). */
__device__ void table_from_sigma(double sigma, uint8_t* table, double* sigma_out)
{
    uint32_t e0 = 1;
    if (sigma > 0.0 && sigma < __longlong_as_double(0x7FF0000000000000ll)) {
        const double x_opt = log2(sigma) + 0.5 * log2(14.0 * log(2.0) / 16383.0);     /* Eq.5 */
        const int lo = (int)floor(x_opt), hi = (int)ceil(x_opt);
        const double s2 = sigma * sqrt(2.0);
        const uint32_t l = lane_id();
        const double v = erf(ldexp(1.0, ((l & 2u) ? hi : lo) + ((l & 1u) ? 0 : 7)) / s2);
        const double p_lo = __shfl(v, 0, 64) - __shfl(v, 1, 64);                      /* Eq.2 */
        const double p_hi = __shfl(v, 2, 64) - __shfl(v, 3, 64);
        int e = (p_hi > p_lo ? hi : lo) + 127;
        e = e < 1 ? 1 : (e > 248 ? 248 : e);
        e0 = (uint32_t)e;
    }
    if (lane_id() != 0) return;
    table[0] = 0;
    for (uint32_t k = 1; k <= 7; ++k) table[k] = (uint8_t)(e0 + k - 1);
    if (sigma_out) *sigma_out = sigma;
}

/* Value of element i as a double (bf16 widened exactly). */
template <int DT>
__device__ __forceinline__ double value_at(const uint8_t* in, uint64_t i)
{
    uint32_t bits;
    if (DT == ZIPCCL_BF16) bits = (uint32_t)(*reinterpret_cast<const uint16_t*>(in + i * 2)) << 16;
    else bits = *reinterpret_cast<const uint32_t*>(in + i * 4);
    return (double)__uint_as_float(bits);
}

/*
 * sigma of a tensor as the paper takes it (section 4.1: torch.std = unbiased sample standard
 * deviation), in FP64.  Sums are taken of d = x - pivot, the pivot being the tensor's first value (0 if that
 * is not finite): sum d^2 - (sum d)^2 / N then cancels only as far as the pivot is from the mean, not as far
 * as the mean is from zero.  Every workgroup writes its partial sums; k_estimate_finish adds the partials in a
 * fixed order, forms sigma, and picks the window (table_from_sigma).
 *
 * Large tensors are bound by reading (2^29 bf16 values 166 us, 6.5 TB/s), with one streamed load in flight per thread: with four the call takes
 * 5 % longer.  Up to 64 MiB, where ramps and latencies count, a thread requests four pieces at a time and does not stream, so that
 * the compress that usually follows finds the tensor in the caches, and workgroups take 4096 values instead of 16384 until
 * there are 2048.  (Of a bf16 tensor of up to 2^23 values a thread has two pieces; it requests the first of them twice more.)  us,
 * before / after, the call: bf16 2^17 6.7 / 5.8, 2^20 6.8 / 5.9, 2^24 12.5 / 11.5, with the compress 28.7 / 26.5; fp32 2^20
 * 7.6 / 5.8, 2^22 10.7 / 8.5, with the compress 24.3 / 19.2.  The 16-byte loads are issued at the tensor's own alignment, which the
 * hardware takes (value by value off a 16-byte boundary: 2^24 bf16 values 25 us, 10.6 now; 2^26 51, 31).
 */
template <int DT, bool STREAM>
__global__ __launch_bounds__(kThreads) void k_moments(const MomentArgs a)
{
    constexpr uint32_t NF = STREAM ? 1u : 4u;          /* pieces in flight per thread */
    constexpr uint32_t ES = DT == ZIPCCL_BF16 ? 2u : 4u;
    constexpr uint32_t PER16 = 16u / ES;               /* values per 16-byte load */
    __shared__ double s_sum[kWavesPerBlock], s_sq[kWavesPerBlock];
    double sum = 0.0, sq = 0.0;
    double pivot = a.n ? value_at<DT>(a.in, 0) : 0.0;
    if (!(fabs(pivot) < __longlong_as_double(0x7FF0000000000000ll))) pivot = 0.0;
    const uint64_t n16 = a.n / PER16, stride = (uint64_t)gridDim.x * kThreads;        /* 16-byte pieces */
    auto load = [&](uint64_t i) { return STREAM ? ld_stream_a2(a.in + i * 16) : (u32x4)*reinterpret_cast<const u32x4_a2*>(a.in + i * 16); };
    auto add = [&](const u32x4& v) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (DT == ZIPCCL_BF16) {
                const double x0 = (double)__uint_as_float(w[k] << 16) - pivot, x1 = (double)__uint_as_float(w[k] & 0xFFFF0000u) - pivot;
                sum += x0; sq += x0 * x0;
                sum += x1; sq += x1 * x1;
            } else {
                const double x = (double)__uint_as_float(w[k]) - pivot;
                sum += x; sq += x * x;
            }
        }
    };
    for (uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < n16; i += NF * stride) {
        u32x4 v[NF];                                   /* past the end the first of them again, not added */
#pragma unroll
        for (uint32_t u = 0; u < NF; ++u) v[u] = load(i + u * stride < n16 ? i + u * stride : i);
#pragma unroll
        for (uint32_t u = 0; u < NF; ++u)
            if (i + u * stride < n16) add(v[u]);
    }
    /* fewer than 16 bytes are left */
    const uint64_t tail = n16 * PER16 + (uint64_t)blockIdx.x * kThreads + threadIdx.x;
    if (tail < a.n) {
        const double x = value_at<DT>(a.in, tail) - pivot;
        sum += x; sq += x * x;
    }
    /* fixed-order reduction: lanes by butterfly, waves in order */
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        sum += __shfl_xor(sum, d, 64);
        sq += __shfl_xor(sq, d, 64);
    }
    const uint32_t wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63u) == 0) { s_sum[wave] = sum; s_sq[wave] = sq; }
    __syncthreads();
    if (threadIdx.x == 0) {
        double ts = 0.0, tq = 0.0;
        for (uint32_t w = 0; w < kWavesPerBlock; ++w) { ts += s_sum[w]; tq += s_sq[w]; }
        a.partial[2 * blockIdx.x] = ts;
        a.partial[2 * blockIdx.x + 1] = tq;
    }
}

__global__ __launch_bounds__(kThreads) void k_estimate_finish(const MomentArgs a)
{
    /* all of a thread's partial sums are requested together */
    constexpr uint32_t PER = kMomentBlocks / kThreads;
    __shared__ double s_sum[kWavesPerBlock], s_sq[kWavesPerBlock];
    double p[PER][2], sum = 0.0, sq = 0.0;
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
        const uint32_t i = min(threadIdx.x + k * kThreads, a.n_blocks - 1u);
        p[k][0] = a.partial[2 * i];
        p[k][1] = a.partial[2 * i + 1];
    }
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k)
        if (threadIdx.x + k * kThreads < a.n_blocks) { sum += p[k][0]; sq += p[k][1]; }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        sum += __shfl_xor(sum, d, 64);
        sq += __shfl_xor(sq, d, 64);
    }
    if ((threadIdx.x & 63u) == 0) { s_sum[threadIdx.x >> 6] = sum; s_sq[threadIdx.x >> 6] = sq; }
    __syncthreads();
    if (threadIdx.x >= 64) return;
    const double N = (double)a.n;
    double sigma = __longlong_as_double(0x7FF8000000000000ll);          /* NaN for fewer than two values */
    if (a.n >= 2) {
        const double ts = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]), tq = (s_sq[0] + s_sq[1]) + (s_sq[2] + s_sq[3]);
        const double var = (tq - ts * ts / N) / (N - 1.0);                       /* sums of x - pivot */
        sigma = sqrt(var > 0.0 ? var : (var == var ? 0.0 : var));
    }
    table_from_sigma(sigma, a.table, a.sigma);
}

/*
 * Robust sigma (for Eq.5 / Eq.2 when the tensor is not the zero-mean Gaussian of section 4.1: outlier
 * channels, LayerNorm gains among matrix weights): the median of |w| over Phi^-1(3/4).  The median is taken
 * over the 15-bit magnitudes of the values' high 16-bit words, so it is a count: the magnitude of rank (K - 1) / 2
 * among the K magnitudes that are neither zero nor Inf/NaN.  Integer work until the final division: the result does
 * not depend on any order.  Three forms, the first two for one or more chunks at once (one table per chunk; the whole
 * tensor is one chunk):
 *   windowed k_window_count: a few workgroups per chunk; each looks for the median of the same small sample of the
 *            chunk, counts only a window of magnitudes around that one by one, and how many there are below and in all,
 *            and stores its own counts.  k_window_finish adds them up; if the rank lies in the window, as it does unless
 *            the sample misled, that gives the median, and if not, its workgroups count all magnitudes after all.
 *   small    k_robust_chunk_fused: one workgroup per chunk with a histogram of all 32768 magnitudes in its LDS.
 *   huge     (2^32 values or more) that histogram, 64 bits wide, in memory: k_clear_hist, k_magnitude_hist, k_robust_finish.
 */
constexpr uint32_t kMagBins = 32768;
constexpr uint32_t kHistThreads = 1024;
constexpr uint32_t kHistWaves = kHistThreads / 64;
constexpr uint32_t kFirstNonFinite = 0x7F80u;                /* magnitudes from here on are Inf / NaN */

/* Counts of a chunk: 32 bits unless the chunk holds 2^32 values or more (only a whole tensor can). */
template <typename CNT> __device__ __forceinline__ CNT scan_of(CNT x);

/* Inclusive prefix sum of 64-bit values over the 64 lanes of a wave, exact, without going through LDS: the four
 * 16-bit limbs are scanned separately with DPP (each limb sum stays below 2^22) and put together again. */
template <> __device__ __forceinline__ unsigned long long scan_of(unsigned long long x)
{
    unsigned long long r = 0;
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k)
        r += (unsigned long long)wave_incl_scan((uint32_t)(x >> (16 * k)) & 0xFFFFu) << (16 * k);
    return r;
}
template <> __device__ __forceinline__ uint32_t scan_of(uint32_t x) { return wave_incl_scan(x); }

/* zero of the bins that do not count: 0 (zero) and 0x7F80.. (Inf / NaN) */
__device__ __forceinline__ bool bin_counts(uint32_t b) { return b != 0u && b < kFirstNonFinite; }

/* The bin of a value's high word in a histogram in LDS that is filled after all.  Zeros, which do not count, go to the bins of Inf and
 * NaN, which do not either, one per lane: a wave's additions to a single word take their turns, and tensors of zeros mostly are
 * among those whose sample misleads (2^24 bf16 values, 99 % of the groups zero: 459 us, 43 now; the one-kernel form does
 * without, which would cost its 8.5 us 0.3). */
__device__ __forceinline__ uint32_t lds_bin(uint32_t word, uint32_t lane)
{
    const uint32_t m = word & 0x7FFFu;
    return m != 0u ? m : kFirstNonFinite + lane;
}

constexpr uint32_t kClearThreads = 1024;

/* One workgroup, 16 16-byte stores per thread. */
__global__ __launch_bounds__(kClearThreads) void k_clear_hist(unsigned long long* hist)
{
    /* the workspace is 8-byte aligned: the 16-byte stores are issued at that alignment */
    u32x4_a4* const p = reinterpret_cast<u32x4_a4*>(hist) + threadIdx.x;
    const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
    for (uint32_t k = 0; k < kHistBytes / (16u * kClearThreads); ++k) p[k * kClearThreads] = zero;
}

/* 16 bytes per thread and step: zeroes the workgroup's histogram (the caller's barrier follows) */
__device__ __forceinline__ void zero_lds_hist(uint32_t* s_hist)
{
    const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
    for (uint32_t k = 0; k < kMagBins / (4u * kHistThreads); ++k)
        reinterpret_cast<u32x4*>(s_hist)[k * kHistThreads + threadIdx.x] = zero;
}

/* Add what the workgroup counted to the chunk's histogram.  The workgroups start at different rows: their atomics
 * on one line come from eight XCDs and take their turns (256 workgroups: 4 us). */
template <typename CNT>
__device__ __forceinline__ void flush_lds_hist(const uint32_t* s_hist, CNT* hist, uint32_t wg)
{
    const uint32_t turn = wg * 128u;
    for (uint32_t i = threadIdx.x; i < kMagBins; i += kHistThreads) {
        const uint32_t b = (i + turn) & (kMagBins - 1u);
        const uint32_t cnt = s_hist[b];
        if (cnt) atomicAdd(&hist[b], (CNT)cnt);
    }
}

/* Workgroup `part` of `parts` counts its part of a tensor's magnitudes; zeroes s_hist first.  A tensor starts at some
 * element: the values in front of its first 16-byte boundary and behind its last one are taken one by one, the rest in 16-byte pieces. */
template <int DT>
__device__ __forceinline__ void tensor_into_lds(uint32_t* s_hist, const uint8_t* __restrict__ in, uint64_t n, uint32_t part, uint32_t parts)
{
    constexpr uint32_t ES = DT == ZIPCCL_BF16 ? 2u : 4u;
    constexpr uint32_t PER16 = 16u / ES;
    constexpr uint32_t NF = 4;                               /* loads in flight per thread */
    const uint64_t head = min(n, (uint64_t)(((16u - (uint32_t)(reinterpret_cast<uintptr_t>(in) & 15u)) & 15u) / ES));
    const uint64_t n16 = (n - head) / PER16;
    const uint8_t* __restrict__ mid = in + head * ES;
    const uint64_t stride = (uint64_t)parts * kHistThreads;
    const uint32_t lane = threadIdx.x & 63u;
    auto count = [&](const u32x4& v) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (DT == ZIPCCL_BF16) atomicAdd(&s_hist[lds_bin(w[k], lane)], 1u);
            atomicAdd(&s_hist[lds_bin(w[k] >> 16, lane)], 1u);
        }
    };
    auto count_one = [&](uint64_t e) {
        const uint32_t hi = DT == ZIPCCL_BF16 ? *reinterpret_cast<const uint16_t*>(in + e * 2)
                                              : *reinterpret_cast<const uint32_t*>(in + e * 4) >> 16;
        atomicAdd(&s_hist[lds_bin(hi, lane)], 1u);
    };
    uint64_t i = (uint64_t)part * kHistThreads + threadIdx.x;
    u32x4 v[NF];
    auto load = [&](uint64_t at) {
#pragma unroll
        for (uint32_t k = 0; k < NF; ++k) v[k] = ld_stream<u32x4>(mid + (at + k * stride) * 16);
    };
    /* the first loads travel while the histogram is zeroed */
    bool more = i + (NF - 1) * stride < n16;
    if (more) load(i);
    zero_lds_hist(s_hist);
    __syncthreads();
    while (more) {
#pragma unroll
        for (uint32_t k = 0; k < NF; ++k) count(v[k]);
        i += NF * stride;
        more = i + (NF - 1) * stride < n16;
        if (more) load(i);
    }
    for (; i < n16; i += stride) count(ld_stream<u32x4>(mid + i * 16));
    if (part == 0) {                                          /* head and tail: fewer than 16 bytes each */
        if (threadIdx.x < head) count_one(threadIdx.x);
        const uint64_t done = head + n16 * PER16;
        if (done + threadIdx.x < n) count_one(done + threadIdx.x);
    }
}

/* Arguments of the kernels below but for the split into chunks, which follows in the form that the launch allows. */
struct RobustIo {
    const uint8_t* in;
    unsigned long long* hist;         /* kHistBytes per chunk */
    uint8_t* table;                   /* 8 bytes per chunk */
    double* sigma;                    /* one per chunk; may be null */
    uint32_t stride;                  /* 1: every value counts; a power of two S: one group of 512 values per S groups */
    uint32_t shared;                  /* windowed form: see WindowPlan */
};

template <int DT>
__global__ __launch_bounds__(kHistThreads) void k_magnitude_hist(const RobustIo a, uint64_t n)
{
    __shared__ __attribute__((aligned(16))) uint32_t s_hist[kMagBins];     /* 128 KiB */
    tensor_into_lds<DT>(s_hist, a.in, n, blockIdx.x, gridDim.x);
    __syncthreads();
    flush_lds_hist(s_hist, a.hist, blockIdx.x);
}

/*
 * The same histogram over a sample of the chunk: its groups of 512 values are cut into blocks of S consecutive
 * groups (S = a.sample_stride, a power of two) and one group is taken from every block, at position
 * ((k * 2654435761 mod 2^32) >> 16) mod S inside block k (Knuth's multiplicative hash: the position varies from
 * block to block, so the sample does not alias with the periods of the tensor itself, rows of 8 or 16 groups
 * say).  A wave takes a group at a time, 8 values per lane, several groups in flight; a group that is cut short by
 * the chunk's end, and every group of a chunk that does not start on a 16-byte boundary, is read value by value.
 * Blocks k0, k0 + n_waves, ... below k_end are this wave's.  Zeroes s_hist first (all threads of the workgroup
 * call this), while the first loads travel.
 */
template <int DT, uint32_t NF, bool ZEROS>   /* NF groups in flight per wave; ZEROS: many of the values may be (lds_bin) */
__device__ __forceinline__ void sample_into_lds(uint32_t* s_hist, const uint8_t* __restrict__ in, uint64_t n, uint32_t S,
                                                uint32_t k0, uint32_t k_end, uint32_t n_waves)
{
    constexpr uint32_t ES = DT == ZIPCCL_BF16 ? 2u : 4u;
    constexpr uint32_t NV = DT == ZIPCCL_BF16 ? 1u : 2u;    /* 16-byte pieces per lane and group */
    const uint64_t ng = (n + kGroup - 1) / kGroup;           /* at most 2^23 */
    /* vector loads need a chunk that starts on a 16-byte boundary; then group 0, if whole, is an address that is
       always safe to load from */
    const bool vec = (reinterpret_cast<uintptr_t>(in) & 15u) == 0 && n >= kGroup;
    const uint32_t lane = threadIdx.x & 63u;
    auto bin = [&](uint32_t word) { return ZEROS ? lds_bin(word, lane) : word & 0x7FFFu; };
    auto one_by_one = [&](uint64_t first) {
        for (uint32_t j = 0; j < kLaneElems; ++j) {
            const uint64_t e = first + lane * kLaneElems + j;
            if (e < n) {
                const uint32_t hi = DT == ZIPCCL_BF16 ? *reinterpret_cast<const uint16_t*>(in + e * 2)
                                                      : *reinterpret_cast<const uint32_t*>(in + e * 4) >> 16;
                atomicAdd(&s_hist[bin(hi)], 1u);
            }
        }
    };
    u32x4 v[NF][NV];
    uint64_t first[NF];
    bool some[NF], whole[NF];
    /* the loads of all NF groups go out back to back: no branch between them (a group that is not there, or
       not whole, loads group 0 instead and is not counted from it) */
    auto load = [&](uint32_t from_block) {
#pragma unroll
        for (uint32_t u = 0; u < NF; ++u) {
            const uint32_t k = from_block + u * n_waves;
            const uint64_t g = (uint64_t)k * S + (((k * 2654435761u) >> 16) & (S - 1u));
            first[u] = g * kGroup;
            some[u] = k < k_end && g < ng;
            whole[u] = some[u] && vec && first[u] + kGroup <= n;
        }
        if (vec) {
#pragma unroll
            for (uint32_t u = 0; u < NF; ++u) {
                const uint64_t from = whole[u] ? first[u] : 0ull;
#pragma unroll
                for (uint32_t q = 0; q < NV; ++q)
                    v[u][q] = ld_stream<u32x4>(in + (from + lane * kLaneElems) * ES + 16u * q);
            }
        }
    };
    const bool any = k0 < k_end;
    if (any) load(k0);
    zero_lds_hist(s_hist);
    __syncthreads();
    if (!any) return;
    for (;;) {
#pragma unroll
        for (uint32_t u = 0; u < NF; ++u) {
            if (whole[u]) {
#pragma unroll
                for (uint32_t q = 0; q < NV; ++q) {
                    const uint32_t w[4] = {v[u][q].x, v[u][q].y, v[u][q].z, v[u][q].w};
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (DT == ZIPCCL_BF16) atomicAdd(&s_hist[bin(w[j])], 1u);
                        atomicAdd(&s_hist[bin(w[j] >> 16)], 1u);
                    }
                }
            }
        }
        /* a group cut short by the chunk's end, or any group of a chunk that is only element-aligned */
#pragma unroll
        for (uint32_t u = 0; u < NF; ++u)
            if (some[u] && !whole[u]) one_by_one(first[u]);
        k0 += NF * n_waves;
        if (k0 >= k_end) return;
        load(k0);
    }
}

/* blocks of S groups in a chunk of n values (at most 2^32 - 1): one group is sampled from each */
__device__ __forceinline__ uint32_t sample_blocks(uint64_t n, uint32_t S)
{
    return (uint32_t)(((n + kGroup - 1) / kGroup + S - 1) / S);
}

/*
 * Rank and table of one chunk by one workgroup of 1024 threads.  `bins` yields 16 bytes of counts at a time: in step k
 * thread t holds the PER bins from (k * 1024 + t) * PER on, so a wave's step is one row of 64 * PER consecutive
 * bins, read coalesced, and the counts never leave their registers: rows are summed by wave scans, every wave finds
 * the row of the rank among the row sums, and the wave that holds that row finds lane and bin.  One barrier.
 */
template <typename CNT, typename LOAD>
__device__ __forceinline__ void rank_and_table(LOAD bins, CNT* s_row, uint8_t* table, double* sigma)
{
    constexpr uint32_t PER = 16u / sizeof(CNT);
    constexpr uint32_t STEPS = kMagBins / (kHistThreads * PER);      /* 8 (32-bit counts) or 16 */
    constexpr uint32_t ROWS = STEPS * kHistWaves, RPL = ROWS / 64;   /* rows, and rows per lane when they are scanned */
    const uint32_t t = threadIdx.x, lane = t & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
    CNT v[STEPS][PER], inc[STEPS];
#pragma unroll
    for (uint32_t k = 0; k < STEPS; ++k) bins(k, v[k]);
#pragma unroll
    for (uint32_t k = 0; k < STEPS; ++k) {
        CNT sum = 0;
#pragma unroll
        for (uint32_t j = 0; j < PER; ++j) {
            if (!bin_counts((k * kHistThreads + t) * PER + j)) v[k][j] = 0;
            sum += v[k][j];
        }
        inc[k] = scan_of<CNT>(sum);
        if (lane == 63u) s_row[k * kHistWaves + wave] = inc[k];
    }
    __syncthreads();
    CNT row_sum[RPL], mine = 0;
#pragma unroll
    for (uint32_t r = 0; r < RPL; ++r) {
        row_sum[r] = s_row[lane * RPL + r];
        mine += row_sum[r];
    }
    const CNT upto = scan_of<CNT>(mine);
    const CNT total = __shfl(upto, 63, 64);
    if (total == 0) {
        if (wave == 0) table_from_sigma(__longlong_as_double(0x7FF8000000000000ll), table, sigma);
        return;
    }
    const CNT rank = (total - 1) / 2;
    /* exactly one lane's rows hold the rank */
    const uint32_t at = (uint32_t)__builtin_ctzll(__ballot(rank >= upto - mine && rank < upto));
    CNT before = upto - mine;
    uint32_t row = lane * RPL;
#pragma unroll
    for (uint32_t r = 0; r + 1 < RPL; ++r)
        if (row == lane * RPL + r && rank >= before + row_sum[r]) { before += row_sum[r]; ++row; }
    row = (uint32_t)__builtin_amdgcn_readfirstlane(__shfl(row, (int)at, 64));
    before = __shfl(before, (int)at, 64);
    if ((row & (kHistWaves - 1u)) != wave) return;
    const uint32_t step = row / kHistWaves;
    CNT w[PER] = {}, winc = 0;
#pragma unroll
    for (uint32_t k = 0; k < STEPS; ++k) {
        if (k == step) {
            winc = inc[k];
#pragma unroll
            for (uint32_t j = 0; j < PER; ++j) w[j] = v[k][j];
        }
    }
    CNT sum = 0;
#pragma unroll
    for (uint32_t j = 0; j < PER; ++j) sum += w[j];
    CNT run = before + winc - sum;
    const uint64_t owner = __ballot(rank >= run && rank < run + sum);
    uint32_t bin = (step * kHistThreads + t) * PER;
#pragma unroll
    for (uint32_t j = 0; j + 1 < PER; ++j) {
        run += w[j];
        if (rank >= run) bin = (step * kHistThreads + t) * PER + j + 1;
    }
    bin = (uint32_t)__shfl((int)bin, (int)__builtin_ctzll(owner), 64);
    const double med = (double)__uint_as_float(bin << 16);
    table_from_sigma(med / 0.6744897501960817, table, sigma);     /* Phi^-1(3/4) */
}

/* One workgroup, after the histogram of a huge tensor: 16 loads per thread, all in flight together. */
__global__ __launch_bounds__(kHistThreads) void k_robust_finish(const RobustIo a)
{
    typedef unsigned long long CNT;
    __shared__ CNT s_row[kMagBins / 128u];
    const u32x4_a4* const hist = reinterpret_cast<const u32x4_a4*>(a.hist) + threadIdx.x;
    rank_and_table<CNT>([&](uint32_t k, CNT* out) {
        const u32x4 q = hist[k * kHistThreads];
        __builtin_memcpy(out, &q, 16);
    }, s_row, a.table, a.sigma);
}

/*
 * A chunk whose sample is small enough for one workgroup: histogram, rank and table in one kernel, nothing outside LDS.
 * grid = chunks.
 */
template <int DT, class SPLIT>
__global__ __launch_bounds__(kHistThreads) void k_robust_chunk_fused(const RobustIo a, const SPLIT split)
{
    constexpr uint32_t ES = DT == ZIPCCL_BF16 ? 2u : 4u;
    __shared__ __attribute__((aligned(16))) uint32_t s_hist[kMagBins];     /* 128 KiB */
    __shared__ uint32_t s_row[kMagBins / 256u];
    const uint32_t c = blockIdx.x;
    const ChunkPlace place = place_of(split, c, DT);
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    /* one workgroup per chunk has the chunk's whole latency to hide: eight groups in flight per wave */
    sample_into_lds<DT, 8, false>(s_hist, a.in + place.elem_off * ES, place.n, a.stride, wave, sample_blocks(place.n, a.stride), kHistWaves);
    __syncthreads();
    rank_and_table<uint32_t>([&](uint32_t k, uint32_t* out) {
        const u32x4 q = reinterpret_cast<const u32x4*>(s_hist)[k * kHistThreads + threadIdx.x];
        __builtin_memcpy(out, &q, 16);
    }, s_row, a.table + 8u * c, a.sigma ? a.sigma + c : nullptr);
}

/*
 * What a workgroup of k_window_count leaves in its chunk's workspace, and behind the last of these, in the workspace's
 * second half, a histogram of 32-bit counts, zeroed, for the case that the window does not hold the rank.
 */
constexpr uint32_t kNarrow = 112, kWide = 496;        /* magnitudes in the window: 7/8 of an octave, or nearly 4 octaves */
template <uint32_t W>
struct Partial {
    uint32_t bins[W];                        /* counts of the magnitudes lo, lo + 1, ... */
    uint32_t below, valid, inside, lo;       /* neither zero nor Inf/NaN: those below lo, all, those in the window */
    uint32_t arrived;                        /* first one: workgroups that have added to the histogram */
    uint32_t unused[11];
};
constexpr uint32_t kPartialsBytes = kHistBytes / 2;
static_assert(sizeof(Partial<kNarrow>) * kHistBlocks <= kPartialsBytes && sizeof(Partial<kWide>) * kWideParts <= kPartialsBytes &&
              kMagBins * 4u <= kHistBytes - kPartialsBytes, "layout of a chunk's workspace");

/*
 * The median of a sample of the chunk, up to 8 magnitudes low: up to 1024 values, 64 strata of equal length, 16
 * consecutive values at a hashed position of each (256 positions of four cost 64 chunks 1 to 2 us more: pages).  By 16 waves that
 * hold all of it and look at one threshold each, four bits of the result per step.  request() issues the loads.
 *
 * Neighbours are often alike, and then such a sample weighs little more than its 64 positions, too little for the narrow window
 * where rows differ much: with rows of 4096 normal values whose scales are log-normal, spread by e^1 / e^1.5 / e^2 / e^3, the rank was outside for
 * 1 / 7 / 11 / 24 of 60 tensors of 512 rows, and everything was counted twice.  The sample shows it: the octave of its median and
 * the two beside it hold 0.74 of its values if they are normal, 0.54 / 0.43 / 0.36 / 0.26 with such rows.  Below a half, request_one()
 * takes 1024 values at 1024 places, after which none of the tensors at e^1.5 and more misses.  That costs 2 to 3 us, as much as the
 * second counts that it saves come to at about 0.45 (us per call, tensors in turn, without / with: 2^20 bf16 values, e^2, 16.6 / 13.2; 2^24 31.5 / 20.1; 2^26
 * 53.7 / 32.2; normal values 10.7 / 10.8, 16.9 / 17.0, 29.5 / 29.7).
 */
struct SampleMedian {
    uint32_t w[2];                           /* four magnitudes of a thread; those that do not count are 0x7FFF */

    template <int DT>
    __device__ __forceinline__ void request(const uint8_t* __restrict__ in, uint64_t n)
    {
        constexpr uint32_t ES = DT == ZIPCCL_BF16 ? 2u : 4u;
        const uint32_t t = threadIdx.x;
        w[0] = w[1] = 0u;
        if (t >= 256u) return;
        if (n >= 1024u) {
            const uint32_t stratum = t / 4u, len = (uint32_t)((n - 16u) / 64u);
            const uint8_t* const p = in + ((uint64_t)stratum * len + (((uint64_t)(stratum * 2654435761u) * len) >> 32) + 4u * (t & 3u)) * ES;
            if (DT == ZIPCCL_BF16) {
                const u32x2 v = *reinterpret_cast<const u32x2_a2*>(p);
                w[0] = v.x; w[1] = v.y;
            } else {
                const u32x4 v = *reinterpret_cast<const u32x4_a4*>(p);
                w[0] = perm(v.y, v.x, 0x07060302u); w[1] = perm(v.w, v.z, 0x07060302u);
            }
        } else {
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {
                const uint32_t e = t * 4u + j;
                if (e < n) {
                    const uint32_t hi = DT == ZIPCCL_BF16 ? *reinterpret_cast<const uint16_t*>(in + e * 2u) : *reinterpret_cast<const uint32_t*>(in + e * 4u) >> 16;
                    w[j >> 1] |= hi << (16u * (j & 1u));
                }
            }
        }
    }

    /* One value of each thread, from the groups of 512 that will be counted, `whole` (not 0) of them, group_of(k) whole in the
       chunk for every k < whole: a hashed one of each 1024th part of them, at a hashed place in it. */
    template <int DT, class GROUP_OF>
    __device__ __forceinline__ static uint32_t request_one(const uint8_t* __restrict__ in, uint32_t whole, GROUP_OF group_of)
    {
        const uint32_t t = threadIdx.x, hash = t * 2654435761u;
        const uint32_t k = (uint32_t)(((uint64_t)((t << 16) | (hash >> 16)) * whole) >> 26);
        const uint64_t e = (uint64_t)group_of(k) * kGroup + (hash & (kGroup - 1u));
        return DT == ZIPCCL_BF16 ? *reinterpret_cast<const uint16_t*>(in + e * 2u) : *reinterpret_cast<const uint32_t*>(in + e * 4u) >> 16;
    }

    __device__ __forceinline__ void put(uint32_t* s_sample)
    {
        if (threadIdx.x < 256u) {
            u32x2 m;
#pragma unroll
            for (uint32_t k = 0; k < 2; ++k) {
                const uint32_t x = w[k] & 0x7FFF7FFFu;
                const uint32_t lo = bin_counts(x & 0xFFFFu) ? x & 0xFFFFu : 0x7FFFu, hi = bin_counts(x >> 16) ? x >> 16 : 0x7FFFu;
                m[k] = lo | (hi << 16);
            }
            *reinterpret_cast<u32x2*>(s_sample + 2u * threadIdx.x) = m;
        }
    }

    __device__ __forceinline__ static void put_one(uint32_t* s_sample, uint32_t value)
    {
        const uint32_t x = value & 0x7FFFu;
        reinterpret_cast<uint16_t*>(s_sample)[threadIdx.x] = (uint16_t)(bin_counts(x) ? x : 0x7FFFu);
    }

    /* The median of what was put into s_sample (512 words); s_cnt: 2 x 16 words.  Called by all threads of the workgroup;
       doubtful is the same in all of them. */
    __device__ __forceinline__ static uint32_t find(const uint32_t* s_sample, uint32_t* s_cnt, uint32_t wave, uint32_t lane, bool& doubtful)
    {
        __syncthreads();
        uint32_t x[8];
#pragma unroll
        for (uint32_t q = 0; q < 2; ++q) {
            const u32x4 v = *reinterpret_cast<const u32x4*>(s_sample + 4u * (lane + 64u * q));
            x[4 * q] = v.x; x[4 * q + 1] = v.y; x[4 * q + 2] = v.z; x[4 * q + 3] = v.w;
        }
        auto below_limit = [&](uint32_t limit) {
            uint32_t cnt = 0;
#pragma unroll
            for (uint32_t k = 0; k < 8; ++k) cnt += __popc(pk_sub_u16(x[k], limit * 0x00010001u) & 0x80008000u);
            return cnt;
        };
        uint32_t base = 0, rank = 0, valid = 0;
#pragma unroll
        for (uint32_t step = 0; step < 3; ++step) {
            const uint32_t shift = 11u - 4u * step;
            /* the last wave counts all that count, once, and in the last step, which starts at the median's octave, those of the
               three octaves around it */
            const bool last = wave == 15u;
            uint32_t cnt = below_limit(!last ? base + ((wave + 1u) << shift) : (step < 2u ? kFirstNonFinite : min(base + 256u, kFirstNonFinite)));
            if (last && step == 2u) cnt -= below_limit(max(base, 128u) - 128u);
            cnt = wave_incl_scan(cnt);
            uint32_t* const s = s_cnt + 16u * (step & 1u);
            if (lane == 63u) s[wave] = cnt;
            __syncthreads();
            const uint32_t below = s[lane & 15u];
            const uint32_t lasts = __builtin_amdgcn_readlane(below, 15);
            if (step == 0) { valid = lasts; rank = (valid - 1u) / 2u; }
            if (step == 2) doubtful = lasts * 2u < valid;
            base += (uint32_t)__popcll(__ballot(below <= rank) & 0x7FFFu) << shift;
        }
        return base;
    }
};

/*
 * Reading bounds it in large tensors (2^29 bf16 values: 172 us, 6.2 TB/s); 2^24 values take 10.7 us, of which the launch is 2, the
 * sample 1.5, reading from HBM alone would be 5 and the additions in LDS alone 4 (with 4 us less to flush and nothing to zero,
 * estimate and table 18.1 -> 15.5 us; 2^20: 14.2 -> 9.3).  Every value still costs an addition in LDS, but to 112 or 496 counters
 * instead of 32768: nothing large is zeroed, and a workgroup's counts are 512 bytes (or 2 KiB) that it stores, where a histogram in
 * memory took a kernel that zeroes it and 4 us of atomic additions from 256 workgroups to the same lines.  Values
 * outside the window are added to a counter of the lane's own, so that they neither branch nor collide.
 * grid = (workgroups per chunk, chunks).  STREAM: the tensor is too large to stay in the caches for the compress
 * that usually follows.
 */
template <int DT, uint32_t W, bool STREAM, class SPLIT>
__global__ __launch_bounds__(kHistThreads) void k_window_count(const RobustIo a, const SPLIT split)
{
    constexpr uint32_t ES = DT == ZIPCCL_BF16 ? 2u : 4u;
    constexpr uint32_t NV = DT == ZIPCCL_BF16 ? 1u : 2u;     /* 16-byte pieces per lane and group */
    constexpr uint32_t NF = 2;                               /* groups in flight per wave (four: one chunk of 2^27 bf16 values 50 us instead of 48) */
    __shared__ __attribute__((aligned(16))) uint32_t s_sample[512];
    __shared__ uint32_t s_cnt[32];
    /* below, window, above (or not counted): outside the window a counter per lane and side, both on the lane's own bank */
    __shared__ uint32_t s_bins[64u + W + 64u];
    __shared__ uint32_t s_valid[kHistWaves];
    const uint32_t c = blockIdx.y;
    const ChunkPlace place = place_of(split, c, DT);
    const uint64_t n = place.n;
    const uint8_t* __restrict__ in = a.in + place.elem_off * ES;
    const uint32_t lane = lane_id();
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t S = a.stride, blocks = sample_blocks(n, S), n_waves = gridDim.x * kHistWaves;
    uint32_t k0 = blockIdx.x * kHistWaves + wave;

    SampleMedian median;
    median.request<DT>(in, n);
    /* the last block's group may be cut short by the chunk's end, or missing; the blocks before it hold whole ones */
    const uint32_t whole = blocks == 0u ? 0u : blocks - 1u;
    auto group_of = [&](uint32_t k) { return k * S + (((k * 2654435761u) >> 16) & (S - 1u)); };
    u32x4 v[NF][NV];
    auto load = [&](uint32_t u, uint32_t k) {
#pragma unroll
        for (uint32_t q = 0; q < NV; ++q) {
            const uint8_t* const p = (in + (uint64_t)group_of(k) * (kGroup * ES)) + q * 1024u + lane * 16u;
            v[u][q] = STREAM ? ld_stream_a2(p) : (u32x4)*reinterpret_cast<const u32x4_a2*>(p);
        }
    };
    /* a group that is not there loads the chunk's first and is not counted */
    if (k0 < whole) {
#pragma unroll
        for (uint32_t u = 0; u < NF; ++u) load(u, k0 + u * n_waves < whole ? k0 + u * n_waves : 0u);
    }
    for (uint32_t i = threadIdx.x; i < W + 128u; i += kHistThreads) s_bins[i] = 0u;
    bool doubtful;                                           /* (the wide window holds what such a sample can be off) */
    median.put(s_sample);
    uint32_t at = SampleMedian::find(s_sample, s_cnt, wave, lane, doubtful) + 4u;
    if (W == kNarrow && doubtful && whole >= 16u) {                          /* fewer groups are soon counted once more */
        SampleMedian::put_one(s_sample, SampleMedian::request_one<DT>(in, whole, group_of));
        at = SampleMedian::find(s_sample, s_cnt, wave, lane, doubtful) + 4u;
    }
    const uint32_t lo = min(max(at, W / 2u + 65u) - W / 2u, kFirstNonFinite - W);

    /* on magnitudes less one, so that zeros go to the top, behind Inf/NaN; d is signed, 64 for lo (which is 65 at least, so
       that the top stays positive) */
    const uint32_t from2 = (lo - 65u) * 0x00010001u, first2 = lane * 0x00010001u, last2 = (64u + W + ((lane - W) & 63u)) * 0x00010001u;
    uint32_t invalid = 0, calls = 0;
    auto count = [&](const uint32_t w[4]) {
        ++calls;
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t m = pk_sub_u16(w[k], 0x00010001u) & 0x7FFF7FFFu;
            invalid += __popc((m + 0x00810081u) & 0x80008000u);               /* from 0x7F7F on */
            const uint32_t b = pk_max_i16(pk_min_i16(pk_sub_u16(m, from2), last2), first2);
            atomicAdd(&s_bins[b & 0xFFFFu], 1u);
            atomicAdd(&s_bins[b >> 16], 1u);
        }
    };
    auto count_loaded = [&](uint32_t u) {
        const u32x4 x = v[u][0], y = v[u][NV - 1u];
        if (DT == ZIPCCL_BF16) {
            const uint32_t w[4] = {x.x, x.y, x.z, x.w};
            count(w);
        } else {
            const uint32_t w[4] = {perm(x.y, x.x, 0x07060302u), perm(x.w, x.z, 0x07060302u), perm(y.y, y.x, 0x07060302u), perm(y.w, y.z, 0x07060302u)};
            count(w);
        }
    };
    /* A group's successor is requested as soon as it is counted, not both once both are: one chunk of 2^27 fp32 values 86.3 -> 83.5 us,
       64 of 2^21 90.3 -> 87.3; bf16 64 of 2^19 20.4 -> 19.8, 64 of 2^21 55.7 -> 55.2, one of 2^27 the same (48.3, 48.2). */
    while (k0 < whole) {
#pragma unroll
        for (uint32_t u = 0; u < NF; ++u) {
            if (k0 + u * n_waves < whole) count_loaded(u);
            if (k0 + NF * n_waves < whole) load(u, k0 + (NF + u) * n_waves < whole ? k0 + (NF + u) * n_waves : 0u);
        }
        k0 += NF * n_waves;
    }
    if (blocks != 0u && whole % n_waves == blockIdx.x * kHistWaves + wave) {
        const uint64_t first = (uint64_t)group_of(whole) * kGroup;
        uint32_t w[4] = {0u, 0u, 0u, 0u};                    /* values that do not exist count as zeros */
#pragma unroll
        for (uint32_t j = 0; j < kLaneElems; ++j) {
            const uint64_t e = first + j * 64u + lane;
            if (e < n) w[j >> 1] |= (DT == ZIPCCL_BF16 ? *reinterpret_cast<const uint16_t*>(in + e * 2u)
                                                       : *reinterpret_cast<const uint32_t*>(in + e * 4u) >> 16) << (16u * (j & 1u));
        }
        count(w);
    }
    Partial<W>* const part = reinterpret_cast<Partial<W>*>(a.hist + (uint64_t)c * (kHistBytes / 8u));
    if (a.shared) {
        /* what the histogram of all magnitudes would be added to, if it comes to that; not earlier, where the wave's later
           loads would wait for these stores (64 chunks of 2^21 fp32 values 106 us at the start, 96 here) */
        u32x4_a4* const hist = reinterpret_cast<u32x4_a4*>(reinterpret_cast<uint8_t*>(part) + kPartialsBytes);
        for (uint32_t i = blockIdx.x * kHistThreads + threadIdx.x; i < kMagBins / 4u; i += gridDim.x * kHistThreads) hist[i] = u32x4{0u, 0u, 0u, 0u};
    }
    const uint32_t counted = wave_incl_scan(8u * calls - invalid);
    if (lane == 63u) s_valid[wave] = counted;
    __syncthreads();
    uint32_t* const mine = part[blockIdx.x].bins;
    if (threadIdx.x < W) mine[threadIdx.x] = s_bins[64u + threadIdx.x];
    if (wave != 1u) return;
    uint32_t inside = 0;
#pragma unroll
    for (uint32_t k = 0; k < W; k += 64u)
        if (k + lane < W) inside += s_bins[64u + k + lane];
    inside = wave_incl_scan(inside);
    const uint32_t below = wave_incl_scan(s_bins[lane]);
    const uint32_t valid = __builtin_amdgcn_readlane(row_incl_scan(s_valid[lane & 15u]), 15);
    if (lane == 63u) {
        *reinterpret_cast<u32x4_a4*>(&part[blockIdx.x].below) = u32x4{below, valid, inside, lo};
        part[blockIdx.x].arrived = 0u;
    }
}

/*
 * One workgroup per chunk adds up the `parts` Partials of it and looks for the rank among them: 1024 threads, a sixteen-byte
 * piece of a 32nd (wide window: an eighth) of the Partials each, all loads in flight together.  Where the sample misled, so that the rank
 * is not in the window, every magnitude is counted: by that workgroup alone in its LDS (`shared` not set),
 * or by all of the grid's, which add to the histogram that k_window_count zeroed; the last
 * to arrive looks for the rank there.  No workgroup waits for another.  grid = (workgroups per chunk for that, chunks).
 */
template <int DT, uint32_t W, class SPLIT>
__global__ __launch_bounds__(kHistThreads) void k_window_finish(const RobustIo a, uint32_t parts, const SPLIT split)
{
    constexpr uint32_t ES = DT == ZIPCCL_BF16 ? 2u : 4u, PIECES = W == kNarrow ? 32u : 128u, ROWS = kHistThreads / PIECES;
    constexpr uint32_t MOST = W == kNarrow ? kHistBlocks : kWideParts;
    __shared__ __attribute__((aligned(16))) uint32_t s_hist[kMagBins];     /* 128 KiB */
    __shared__ uint32_t s_head[3][4];
    __shared__ uint32_t s_row[kMagBins / 256u];
    const uint32_t c = blockIdx.y, t = threadIdx.x, lane = lane_id();
    const uint32_t wave = __builtin_amdgcn_readfirstlane(t >> 6);
    Partial<W>* const part = reinterpret_cast<Partial<W>*>(a.hist + (uint64_t)c * (kHistBytes / 8u));
    uint8_t* const table = a.table + 8u * c;
    double* const sigma = a.sigma ? a.sigma + c : nullptr;

    const u32x4 head = *reinterpret_cast<const u32x4_a4*>(&part[min(t, parts - 1u)].below);      /* below, valid, inside, lo */
    const uint32_t row = t / PIECES, q = min(t % PIECES, W / 4u - 1u);
    if (blockIdx.x == 0u) {
        u32x4 v[MOST / ROWS], sum = {0u, 0u, 0u, 0u};
#pragma unroll
        for (uint32_t k = 0; k < MOST / ROWS; ++k)
            if (W == kNarrow || ROWS * k < parts) v[k] = reinterpret_cast<const u32x4_a4*>(part[min(row + ROWS * k, parts - 1u)].bins)[q];
#pragma unroll
        for (uint32_t k = 0; k < MOST / ROWS; ++k)
            if (row + ROWS * k < parts) sum += v[k];
        reinterpret_cast<u32x4*>(s_hist)[t] = sum;
    }
    if (wave < 4u) {
#pragma unroll
        for (uint32_t k = 0; k < 3; ++k) {
            const uint32_t inc = wave_incl_scan(t < parts ? head[k] : 0u);
            if (lane == 63u) s_head[k][wave] = inc;
        }
    }
    __syncthreads();
    const uint32_t below = (s_head[0][0] + s_head[0][1]) + (s_head[0][2] + s_head[0][3]);
    const uint32_t valid = (s_head[1][0] + s_head[1][1]) + (s_head[1][2] + s_head[1][3]);
    const uint32_t inside = (s_head[2][0] + s_head[2][1]) + (s_head[2][2] + s_head[2][3]);
    const uint32_t rank = (valid - 1u) / 2u;
    if (valid == 0u) {
        if (blockIdx.x == 0u && wave == 0u) table_from_sigma(__longlong_as_double(0x7FF8000000000000ll), table, sigma);
        return;
    }
    if (rank >= below && rank - below < inside) {
        if (blockIdx.x != 0u) return;
        if (W <= 128u && wave != 0u) return;
        uint32_t even = 0, odd = 0;                          /* counts of magnitudes lo + 2 t and lo + 2 t + 1 */
        if (t < W / 2u) {
#pragma unroll
            for (uint32_t r = 0; r < ROWS; ++r) {
                const u32x2 w = *reinterpret_cast<const u32x2*>(s_hist + r * (4u * PIECES) + 2u * t);
                even += w.x;
                odd += w.y;
            }
        }
        uint32_t inc = wave_incl_scan(even + odd);
        if (W > 128u) {
            if (lane == 63u) s_row[wave] = inc;
            __syncthreads();
            for (uint32_t w = 0; w < wave; ++w) inc += s_row[w];
        }
        inc += below;
        const uint64_t owner = __ballot(rank >= inc - even - odd && rank < inc);
        if (W > 128u && owner == 0u) return;                 /* another wave's */
        uint32_t bin = head.w + 2u * t + (uint32_t)(rank >= inc - odd);
        bin = __builtin_amdgcn_readlane(bin, (uint32_t)__builtin_ctzll(owner));
        const double med = (double)__uint_as_float(bin << 16);
        table_from_sigma(med / 0.6744897501960817, table, sigma);     /* Phi^-1(3/4) */
        return;
    }
    const ChunkPlace place = place_of(split, c, DT);
    const uint8_t* __restrict__ in = a.in + place.elem_off * ES;
    __syncthreads();                                         /* s_hist is used anew */
    if (a.stride == 1u) tensor_into_lds<DT>(s_hist, in, place.n, blockIdx.x, gridDim.x);
    else sample_into_lds<DT, 4, true>(s_hist, in, place.n, a.stride, blockIdx.x * kHistWaves + wave, sample_blocks(place.n, a.stride), gridDim.x * kHistWaves);
    __syncthreads();
    if (!a.shared) {
        if (t == 0u) part[0].arrived = 1u;
        rank_and_table<uint32_t>([&](uint32_t k, uint32_t* out) {
            const u32x4 x = reinterpret_cast<const u32x4*>(s_hist)[k * kHistThreads + t];
            __builtin_memcpy(out, &x, 16);
        }, s_row, table, sigma);
        return;
    }
    uint32_t* const hist = reinterpret_cast<uint32_t*>(reinterpret_cast<uint8_t*>(part) + kPartialsBytes);
    flush_lds_hist(s_hist, hist, blockIdx.x);
    /* every thread's additions have been made when the workgroup arrives.  One fence per workgroup: each walks its XCD's
       L2, and one per wave took the fallback from 30 to 90 us */
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (t == 0u) {
        __threadfence();
        s_head[0][0] = atomicAdd(&part[0].arrived, 1u);
        __threadfence();
    }
    __syncthreads();
    if (s_head[0][0] + 1u != gridDim.x) return;
    rank_and_table<uint32_t>([&](uint32_t k, uint32_t* out) {
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j)                     /* other workgroups' additions: past this XCD's caches */
            out[j] = __hip_atomic_load(hist + (k * kHistThreads + t) * 4u + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }, s_row, table, sigma);
}

} // namespace

int launch_estimate(int dt, const MomentArgs& a, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    const bool stream_loads = a.n * (dt == ZIPCCL_BF16 ? 2u : 4u) > (64ull << 20);         /* see launch_window */
    if (dt == ZIPCCL_BF16 && stream_loads) hipLaunchKernelGGL((k_moments<ZIPCCL_BF16, true>), dim3(a.n_blocks), dim3(kThreads), 0, s, a);
    else if (dt == ZIPCCL_BF16) hipLaunchKernelGGL((k_moments<ZIPCCL_BF16, false>), dim3(a.n_blocks), dim3(kThreads), 0, s, a);
    else if (stream_loads) hipLaunchKernelGGL((k_moments<ZIPCCL_FP32, true>), dim3(a.n_blocks), dim3(kThreads), 0, s, a);
    else hipLaunchKernelGGL((k_moments<ZIPCCL_FP32, false>), dim3(a.n_blocks), dim3(kThreads), 0, s, a);
    if (hipGetLastError() != hipSuccess) return 1;
    hipLaunchKernelGGL(k_estimate_finish, dim3(1), dim3(kThreads), 0, s, a);
    return (int)hipGetLastError();
}


template <int DT, uint32_t W, class SPLIT>
static int launch_window(const HistArgs& a, const WindowPlan& plan, const SPLIT& split, hipStream_t s)
{
    const RobustIo io = {a.in, a.hist, a.table, a.sigma, a.sample_stride, plan.shared};
    const uint32_t chunks = a.tab.n_chunks;
    const dim3 grid(plan.parts, chunks), block(kHistThreads);
    if (plan.stream) hipLaunchKernelGGL((k_window_count<DT, W, true, SPLIT>), grid, block, 0, s, io, split);
    else hipLaunchKernelGGL((k_window_count<DT, W, false, SPLIT>), grid, block, 0, s, io, split);
    if (hipGetLastError() != hipSuccess) return 1;
    hipLaunchKernelGGL((k_window_finish<DT, W, SPLIT>), dim3(plan.finish, chunks), block, 0, s, io, plan.parts, split);
    return (int)hipGetLastError();
}

template <int DT>
static int launch_huge(const HistArgs& a, hipStream_t s)
{
    const RobustIo io = {a.in, a.hist, a.table, a.sigma, 1u, 1u};
    hipLaunchKernelGGL(k_clear_hist, dim3(1), dim3(kClearThreads), 0, s, a.hist);
    if (hipGetLastError() != hipSuccess) return 1;
    hipLaunchKernelGGL((k_magnitude_hist<DT>), dim3(kHistBlocks), dim3(kHistThreads), 0, s, io, a.tab.elem_off[1]);
    if (hipGetLastError() != hipSuccess) return 1;
    hipLaunchKernelGGL(k_robust_finish, dim3(1), dim3(kHistThreads), 0, s, io);
    return (int)hipGetLastError();
}

template <int DT>
static int launch_robust(const HistArgs& a, hipStream_t s)
{
    const uint32_t chunks = a.tab.n_chunks;
    if (robust_in_one_kernel(a.tab, a.sample_stride)) {
        const RobustIo io = {a.in, a.hist, a.table, a.sigma, a.sample_stride, 0u};
        if (is_equal_split(a.tab)) hipLaunchKernelGGL((k_robust_chunk_fused<DT, EqualSplit>), dim3(chunks), dim3(kHistThreads), 0, s, io, equal_split(a.tab));
        else hipLaunchKernelGGL((k_robust_chunk_fused<DT, ChunkTab>), dim3(chunks), dim3(kHistThreads), 0, s, io, a.tab);
        return (int)hipGetLastError();
    }
    /* 2^32 values or more: only a whole tensor, every value of which counts */
    if (chunks == 1u && a.tab.elem_off[1] > ZIPCCL_MAX_CHUNK_ELEMS) return launch_huge<DT>(a, s);
    const WindowPlan plan = window_plan(a.tab, DT, a.sample_stride);
    if (is_equal_split(a.tab)) return plan.wide ? launch_window<DT, kWide>(a, plan, equal_split(a.tab), s) : launch_window<DT, kNarrow>(a, plan, equal_split(a.tab), s);
    return plan.wide ? launch_window<DT, kWide>(a, plan, a.tab, s) : launch_window<DT, kNarrow>(a, plan, a.tab, s);
}

int launch_estimate_robust(int dt, const HistArgs& a, void* stream)
{
    return dt == ZIPCCL_BF16 ? launch_robust<ZIPCCL_BF16>(a, (hipStream_t)stream) : launch_robust<ZIPCCL_FP32>(a, (hipStream_t)stream);
}

} // namespace zipccl
