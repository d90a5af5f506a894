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
 */
template <int DT>
__global__ __launch_bounds__(kThreads) void k_moments(const MomentArgs a)
{
    constexpr uint32_t ES = DT == ZIPCCL_BF16 ? 2u : 4u;
    constexpr uint32_t PER16 = 16u / ES;               /* values per 16-byte load */
    __shared__ double s_sum[kWavesPerBlock], s_sq[kWavesPerBlock];
    double sum = 0.0, sq = 0.0;
    double pivot = a.n ? value_at<DT>(a.in, 0) : 0.0;
    if (!(fabs(pivot) < __longlong_as_double(0x7FF0000000000000ll))) pivot = 0.0;
    const bool aligned = (reinterpret_cast<uintptr_t>(a.in) & 15u) == 0;
    const uint64_t n16 = aligned ? a.n / PER16 : 0;    /* 16-byte pieces handled with vector loads */
    for (uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < n16; i += (uint64_t)gridDim.x * kThreads) {
        const u32x4 v = ld_stream<u32x4>(a.in + i * 16);
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
    }
    /* the tail (and everything, for a misaligned tensor) element by element */
    for (uint64_t i = n16 * PER16 + (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < a.n; i += (uint64_t)gridDim.x * kThreads) {
        const double x = value_at<DT>(a.in, i) - pivot;
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
    __shared__ double s_sum[kThreads], s_sq[kThreads];
    double sum = 0.0, sq = 0.0;
    for (uint32_t i = threadIdx.x; i < a.n_blocks; i += kThreads) { sum += a.partial[2 * i]; sq += a.partial[2 * i + 1]; }
    s_sum[threadIdx.x] = sum;
    s_sq[threadIdx.x] = sq;
    __syncthreads();
    for (uint32_t d = kThreads / 2; d >= 1; d >>= 1) {
        if (threadIdx.x < d) { s_sum[threadIdx.x] += s_sum[threadIdx.x + d]; s_sq[threadIdx.x] += s_sq[threadIdx.x + d]; }
        __syncthreads();
    }
    if (threadIdx.x >= 64) return;
    const double N = (double)a.n;
    double sigma = __longlong_as_double(0x7FF8000000000000ll);          /* NaN for fewer than two values */
    if (a.n >= 2) {
        const double var = (s_sq[0] - s_sum[0] * s_sum[0] / N) / (N - 1.0);      /* sums of x - pivot */
        sigma = sqrt(var > 0.0 ? var : (var == var ? 0.0 : var));
    }
    table_from_sigma(sigma, a.table, a.sigma);
}

/*
 * Robust sigma (for Eq.5 / Eq.2 when the tensor is not the zero-mean Gaussian of section 4.1: outlier
 * channels, LayerNorm gains among matrix weights): the median of |w| over Phi^-1(3/4).  The median is taken
 * over the 15-bit magnitudes of the values' high 16-bit words, so it is a count: a histogram of all 32768
 * magnitudes, in which the bin of rank (K - 1) / 2 among the K magnitudes that are neither zero nor Inf/NaN is
 * looked for.  Integer work until the final division: the result does not depend on any order.  Three forms,
 * each for one or more chunks at once (one histogram and one table per chunk; the whole tensor is one chunk):
 *   large    k_clear_hist zeroes one histogram per chunk in the workspace, k_magnitude_hist (or its sampled form)
 *            adds to it what about one workgroup per compute unit has counted in its LDS, k_robust_finish looks
 *            for the rank.  2^24 bf16 values, one chunk: 2.0 + 11.6 + 3.7 us, launches included (the
 *            histogram kernel without its flush: 4 us less).  With 64-bit counts zeroed, flushed and read twice over
 *            by the finish, whose one thread then took four erf in a row, the same three kernels were 3.0 + 13.8 +
 *            11.2 us.
 *   small    (at most kFusedGroups groups to count in every chunk) k_robust_partial: a few workgroups per chunk, each
 *            of which stores its own counts; k_robust_join adds them up and looks for the rank.  Nothing to clear, no
 *            atomics on memory.
 *   smaller  (or as many chunks as compute units) k_robust_chunk_fused: one workgroup per chunk, one kernel.
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

constexpr uint32_t kClearThreads = 1024;

/* One workgroup per histogram, 8 or 16 16-byte stores per thread (spread over 16 or 32 times as many workgroups the
 * kernel took 5 us longer for 64 histograms: the launch, not the memory, is its limit). */
template <typename CNT>
__global__ __launch_bounds__(kClearThreads) void k_clear_hist(unsigned long long* hist)
{
    /* grid = chunks (the workspace is 8-byte aligned: the 16-byte stores are issued at that alignment) */
    u32x4_a4* const p = reinterpret_cast<u32x4_a4*>(hist + (uint64_t)blockIdx.x * (kHistBytes / 8)) + threadIdx.x;
    const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
    for (uint32_t k = 0; k < kMagBins * sizeof(CNT) / (16u * kClearThreads); ++k) p[k * kClearThreads] = zero;
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
 * on one line come from eight XCDs and take their turns (the flush is 4 us of a call on 2^24 values). */
template <typename CNT>
__device__ __forceinline__ void flush_lds_hist(const uint32_t* s_hist, unsigned long long* hist_c, uint32_t wg)
{
    CNT* const hist = reinterpret_cast<CNT*>(hist_c);
    const uint32_t turn = wg * 128u;
    for (uint32_t i = threadIdx.x; i < kMagBins; i += kHistThreads) {
        const uint32_t b = (i + turn) & (kMagBins - 1u);
        const uint32_t cnt = s_hist[b];
        if (cnt) atomicAdd(&hist[b], (CNT)cnt);
    }
}

template <int DT, typename CNT>
__global__ __launch_bounds__(kHistThreads) void k_magnitude_hist(const HistArgs a)
{
    constexpr uint32_t ES = DT == ZIPCCL_BF16 ? 2u : 4u;
    constexpr uint32_t PER16 = 16u / ES;
    constexpr uint32_t NF = 4;                               /* loads in flight per thread */
    __shared__ __attribute__((aligned(16))) uint32_t s_hist[kMagBins];     /* 128 KiB */
    /* grid = (workgroups per chunk, chunks); a chunk starts at some element of the tensor: the values in front of
       its first 16-byte boundary and behind its last one are taken one by one, the rest in 16-byte pieces */
    const uint32_t c = blockIdx.y;
    const uint8_t* __restrict__ in = a.in + a.tab.elem_off[c] * ES;
    const uint64_t n = a.tab.elem_off[c + 1] - a.tab.elem_off[c];
    const uint64_t head = min(n, (uint64_t)(((16u - (uint32_t)(reinterpret_cast<uintptr_t>(in) & 15u)) & 15u) / ES));
    const uint64_t n16 = (n - head) / PER16;
    const uint8_t* __restrict__ mid = in + head * ES;
    const uint64_t stride = (uint64_t)gridDim.x * kHistThreads;
    auto count = [&](const u32x4& v) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (DT == ZIPCCL_BF16) atomicAdd(&s_hist[w[k] & 0x7FFFu], 1u);
            atomicAdd(&s_hist[(w[k] >> 16) & 0x7FFFu], 1u);
        }
    };
    auto count_one = [&](uint64_t e) {
        const uint32_t hi = DT == ZIPCCL_BF16 ? *reinterpret_cast<const uint16_t*>(in + e * 2)
                                              : *reinterpret_cast<const uint32_t*>(in + e * 4) >> 16;
        atomicAdd(&s_hist[hi & 0x7FFFu], 1u);
    };
    uint64_t i = (uint64_t)blockIdx.x * kHistThreads + threadIdx.x;
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
    if (blockIdx.x == 0) {                                    /* head and tail: fewer than 16 bytes each */
        if (threadIdx.x < head) count_one(threadIdx.x);
        const uint64_t done = head + n16 * PER16;
        if (done + threadIdx.x < n) count_one(done + threadIdx.x);
    }
    __syncthreads();
    flush_lds_hist<CNT>(s_hist, a.hist + (uint64_t)c * (kHistBytes / 8), blockIdx.x);
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
template <int DT, uint32_t NF>   /* NF groups in flight per wave */
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
    auto one_by_one = [&](uint64_t first) {
        for (uint32_t j = 0; j < kLaneElems; ++j) {
            const uint64_t e = first + lane * kLaneElems + j;
            if (e < n) {
                const uint32_t hi = DT == ZIPCCL_BF16 ? *reinterpret_cast<const uint16_t*>(in + e * 2)
                                                      : *reinterpret_cast<const uint32_t*>(in + e * 4) >> 16;
                atomicAdd(&s_hist[hi & 0x7FFFu], 1u);
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
                        if (DT == ZIPCCL_BF16) atomicAdd(&s_hist[w[j] & 0x7FFFu], 1u);
                        atomicAdd(&s_hist[(w[j] >> 16) & 0x7FFFu], 1u);
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

template <int DT>
__global__ __launch_bounds__(kHistThreads) void k_magnitude_hist_sampled(const HistArgs a)
{
    constexpr uint32_t ES = DT == ZIPCCL_BF16 ? 2u : 4u;
    __shared__ __attribute__((aligned(16))) uint32_t s_hist[kMagBins];     /* 128 KiB */
    /* grid = (workgroups per chunk, chunks) */
    const uint32_t c = blockIdx.y;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t n = a.tab.elem_off[c + 1] - a.tab.elem_off[c];
    sample_into_lds<DT, 4>(s_hist, a.in + a.tab.elem_off[c] * ES, n, a.sample_stride, blockIdx.x * kHistWaves + wave,
                           sample_blocks(n, a.sample_stride), gridDim.x * kHistWaves);
    __syncthreads();
    flush_lds_hist<uint32_t>(s_hist, a.hist + (uint64_t)c * (kHistBytes / 8), blockIdx.x);
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

/* One workgroup per chunk, after the histogram kernels: 8 (32-bit counts) or 16 loads per thread, all in flight together. */
template <typename CNT>
__global__ __launch_bounds__(kHistThreads) void k_robust_finish(const HistArgs a)
{
    constexpr uint32_t PER = 16u / sizeof(CNT);
    __shared__ CNT s_row[kMagBins / (64u * PER)];
    /* grid = chunks */
    const u32x4_a4* const hist = reinterpret_cast<const u32x4_a4*>(a.hist + (uint64_t)blockIdx.x * (kHistBytes / 8)) + threadIdx.x;
    rank_and_table<CNT>([&](uint32_t k, CNT* out) {
        const u32x4 q = hist[k * kHistThreads];
        __builtin_memcpy(out, &q, 16);
    }, s_row, a.table + 8u * blockIdx.x, a.sigma ? a.sigma + blockIdx.x : nullptr);
}

/*
 * A chunk whose sample is small enough for one workgroup: histogram, rank and table in one kernel, nothing outside LDS.
 * grid = chunks.
 */
template <int DT>
__global__ __launch_bounds__(kHistThreads) void k_robust_chunk_fused(const HistArgs a)
{
    constexpr uint32_t ES = DT == ZIPCCL_BF16 ? 2u : 4u;
    __shared__ __attribute__((aligned(16))) uint32_t s_hist[kMagBins];     /* 128 KiB */
    __shared__ uint32_t s_row[kMagBins / 256u];
    const uint32_t c = blockIdx.x;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t n = a.tab.elem_off[c + 1] - a.tab.elem_off[c];
    /* one workgroup per chunk has the chunk's whole latency to hide: eight groups in flight per wave */
    sample_into_lds<DT, 8>(s_hist, a.in + a.tab.elem_off[c] * ES, n, a.sample_stride, wave,
                           sample_blocks(n, a.sample_stride), kHistWaves);
    __syncthreads();
    rank_and_table<uint32_t>([&](uint32_t k, uint32_t* out) {
        const u32x4 q = reinterpret_cast<const u32x4*>(s_hist)[k * kHistThreads + threadIdx.x];
        __builtin_memcpy(out, &q, 16);
    }, s_row, a.table + 8u * c, a.sigma ? a.sigma + c : nullptr);
}

/*
 * Chunks that are too large for one workgroup to count quickly (a group of 512 values takes its compute unit's LDS
 * atomics 36 ns) and too few to fill the chip: G = gridDim.x <= 4 workgroups per chunk, each with at most 127 of
 * its blocks, i.e. fewer than 2^16 values, so that 16 bits hold every count.  A workgroup stores the rows of 256 bins in
 * which it counted anything, and the sum of every row, in its own 64 KiB of the chunk's workspace: the counts of the
 * bins that never count (Inf / NaN, 128 of them) leave room for the 128 row sums.
 */
constexpr uint32_t kPartials = 4;
constexpr uint32_t kPartialBytes = kMagBins * 2;
constexpr uint32_t kPartialGroups = 127;
static_assert(kPartials * kPartialBytes <= kHistBytes && kPartials * kPartialGroups == kFusedGroups &&
              kPartialGroups * kGroup < 65536u && kMagBins - kFirstNonFinite == kMagBins / 256u, "layout of the partial counts");

template <int DT>
__global__ __launch_bounds__(kHistThreads) void k_robust_partial(const HistArgs a)
{
    constexpr uint32_t ES = DT == ZIPCCL_BF16 ? 2u : 4u;
    __shared__ __attribute__((aligned(16))) uint32_t s_hist[kMagBins];     /* 128 KiB */
    /* grid = (workgroups per chunk, chunks) */
    const uint32_t c = blockIdx.y;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t n = a.tab.elem_off[c + 1] - a.tab.elem_off[c];
    const uint32_t blocks = sample_blocks(n, a.sample_stride);               /* at most kFusedGroups */
    sample_into_lds<DT, 8>(s_hist, a.in + a.tab.elem_off[c] * ES, n, a.sample_stride,
                           blockIdx.x * blocks / gridDim.x + wave, (blockIdx.x + 1u) * blocks / gridDim.x, kHistWaves);
    __syncthreads();
    uint16_t* const mine = reinterpret_cast<uint16_t*>(reinterpret_cast<uint8_t*>(a.hist + (uint64_t)c * (kHistBytes / 8)) +
                                                       blockIdx.x * kPartialBytes);
#pragma unroll
    for (uint32_t k = 0; k < kMagBins / (256u * kHistWaves); ++k) {
        const uint32_t row = k * kHistWaves + wave, b = row * 256u + lane * 4u;
        u32x4 q = *reinterpret_cast<const u32x4*>(s_hist + b);
        if (b == 0u) q.x = 0u;
        if (b >= kFirstNonFinite) q = u32x4{0u, 0u, 0u, 0u};
        const uint32_t sum = __builtin_amdgcn_readlane(wave_incl_scan((q.x + q.y) + (q.z + q.w)), 63);
        if (sum != 0u && b < kFirstNonFinite)
            *reinterpret_cast<u32x2*>(mine + b) = u32x2{q.x | (q.y << 16), q.z | (q.w << 16)};
        if (lane == 0) mine[kFirstNonFinite + row] = (uint16_t)sum;
    }
}

/* One wave per chunk: the row of the rank from the row sums, then the bin from that row of every partial. */
__global__ __launch_bounds__(64) void k_robust_join(const HistArgs a)
{
    /* grid = chunks; a.n_blocks partials each */
    const uint32_t c = blockIdx.x, lane = lane_id();
    const uint8_t* const part = reinterpret_cast<const uint8_t*>(a.hist + (uint64_t)c * (kHistBytes / 8));
    uint8_t* const table = a.table + 8u * c;
    double* const sigma = a.sigma ? a.sigma + c : nullptr;
    uint32_t sums[kPartials];                                  /* of rows 2 lane (low half) and 2 lane + 1 */
#pragma unroll
    for (uint32_t g = 0; g < kPartials; ++g)
        sums[g] = g < a.n_blocks ? *reinterpret_cast<const uint32_t*>(part + g * kPartialBytes + 2u * (kFirstNonFinite + 2u * lane)) : 0u;
    uint32_t even = 0, odd = 0;
#pragma unroll
    for (uint32_t g = 0; g < kPartials; ++g) { even += sums[g] & 0xFFFFu; odd += sums[g] >> 16; }
    const uint32_t upto = wave_incl_scan(even + odd);
    const uint32_t total = __builtin_amdgcn_readlane(upto, 63);
    if (total == 0u) {
        table_from_sigma(__longlong_as_double(0x7FF8000000000000ll), table, sigma);
        return;
    }
    const uint32_t rank = (total - 1u) / 2u;
    uint32_t before = upto - even - odd;
    const uint32_t at = (uint32_t)__builtin_ctzll(__ballot(rank >= before && rank < upto));
    uint32_t row = 2u * lane;
    if (rank >= before + even) { before += even; ++row; }
    row = __builtin_amdgcn_readlane(row, at);
    before = __builtin_amdgcn_readlane(before, at);
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (uint32_t g = 0; g < kPartials; ++g) {
        const uint32_t of_row = __builtin_amdgcn_readlane(sums[g], at) >> (16u * (row & 1u)) & 0xFFFFu;
        if (of_row != 0u && row * 256u + lane * 4u < kFirstNonFinite) {      /* rows without counts were not stored */
            const u32x2 q = *reinterpret_cast<const u32x2*>(part + g * kPartialBytes + 2u * (row * 256u + lane * 4u));
            w[0] += q.x & 0xFFFFu; w[1] += q.x >> 16; w[2] += q.y & 0xFFFFu; w[3] += q.y >> 16;
        }
    }
    const uint32_t sum = (w[0] + w[1]) + (w[2] + w[3]);
    uint32_t run = before + wave_incl_scan(sum) - sum;
    const uint64_t owner = __ballot(rank >= run && rank < run + sum);
    uint32_t bin = row * 256u + lane * 4u;
#pragma unroll
    for (uint32_t j = 0; j < 3; ++j) {
        run += w[j];
        if (rank >= run) bin = row * 256u + lane * 4u + j + 1u;
    }
    bin = __builtin_amdgcn_readlane(bin, (uint32_t)__builtin_ctzll(owner));
    const double med = (double)__uint_as_float(bin << 16);
    table_from_sigma(med / 0.6744897501960817, table, sigma);     /* Phi^-1(3/4) */
}

} // namespace

int launch_estimate(int dt, const MomentArgs& a, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    if (dt == ZIPCCL_BF16) hipLaunchKernelGGL((k_moments<ZIPCCL_BF16>), dim3(a.n_blocks), dim3(kThreads), 0, s, a);
    else hipLaunchKernelGGL((k_moments<ZIPCCL_FP32>), dim3(a.n_blocks), dim3(kThreads), 0, s, a);
    if (hipGetLastError() != hipSuccess) return 1;
    hipLaunchKernelGGL(k_estimate_finish, dim3(1), dim3(kThreads), 0, s, a);
    return (int)hipGetLastError();
}


/* Several workgroups per chunk and a second kernel from this many groups in the largest chunk on, as long as there are
 * no more of them than compute units (a compute unit's LDS holds one at a time).  Measured, us, bf16, one workgroup
 * against several: 64 chunks of 128 groups 10.2 / 11.2, of 192 13.1 / 11.9, of 448 21.9 / 14.0; one chunk of 128
 * groups 9.4 / 9.7, of 500 20.9 / 12.4; 128 chunks of 192 (two workgroups each) 13.4 / 12.5, and of 256, where two
 * workgroups per chunk cannot hold them, 15.5 / 15.9.  fp32: 64 chunks of 448 38.1 / 20.5. */
constexpr uint32_t kPartialFrom = 160;

int launch_estimate_robust_fused(int dt, const HistArgs& a, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    uint64_t largest = 0;
    for (uint32_t c = 0; c < a.tab.n_chunks; ++c) largest = std::max(largest, a.tab.elem_off[c + 1] - a.tab.elem_off[c]);
    const uint64_t groups = ((largest + kGroup - 1) / kGroup + a.sample_stride - 1) / a.sample_stride;
    const uint32_t chunks = a.tab.n_chunks;
    HistArgs b = a;
    b.n_blocks = (uint32_t)std::max<uint64_t>(std::min(kHistBlocks / chunks, kPartials), (groups + kPartialGroups - 1) / kPartialGroups);
    if (groups >= kPartialFrom && b.n_blocks * chunks <= kHistBlocks) {
        const dim3 grid(b.n_blocks, chunks);
        if (dt == ZIPCCL_BF16) hipLaunchKernelGGL((k_robust_partial<ZIPCCL_BF16>), grid, dim3(kHistThreads), 0, s, b);
        else hipLaunchKernelGGL((k_robust_partial<ZIPCCL_FP32>), grid, dim3(kHistThreads), 0, s, b);
        if (hipGetLastError() != hipSuccess) return 1;
        hipLaunchKernelGGL(k_robust_join, dim3(chunks), dim3(64), 0, s, b);
        return (int)hipGetLastError();
    }
    if (dt == ZIPCCL_BF16) hipLaunchKernelGGL((k_robust_chunk_fused<ZIPCCL_BF16>), dim3(chunks), dim3(kHistThreads), 0, s, a);
    else hipLaunchKernelGGL((k_robust_chunk_fused<ZIPCCL_FP32>), dim3(chunks), dim3(kHistThreads), 0, s, a);
    return (int)hipGetLastError();
}

template <int DT, typename CNT>
static int launch_large(const HistArgs& a, hipStream_t s)
{
    const dim3 grid(a.n_blocks, a.tab.n_chunks), chunks(a.tab.n_chunks);
    hipLaunchKernelGGL((k_clear_hist<CNT>), chunks, dim3(kClearThreads), 0, s, a.hist);
    if (hipGetLastError() != hipSuccess) return 1;
    if (a.sample_stride > 1u) hipLaunchKernelGGL((k_magnitude_hist_sampled<DT>), grid, dim3(kHistThreads), 0, s, a);
    else hipLaunchKernelGGL((k_magnitude_hist<DT, CNT>), grid, dim3(kHistThreads), 0, s, a);
    if (hipGetLastError() != hipSuccess) return 1;
    hipLaunchKernelGGL((k_robust_finish<CNT>), chunks, dim3(kHistThreads), 0, s, a);
    return (int)hipGetLastError();
}

int launch_estimate_robust(int dt, const HistArgs& a, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    /* 32-bit counts unless some chunk could overflow them; a sample is only taken of chunks below 2^32 values */
    bool wide = false;
    for (uint32_t c = 0; c < a.tab.n_chunks; ++c) wide |= a.tab.elem_off[c + 1] - a.tab.elem_off[c] > ZIPCCL_MAX_CHUNK_ELEMS;
    if (wide) return dt == ZIPCCL_BF16 ? launch_large<ZIPCCL_BF16, unsigned long long>(a, s) : launch_large<ZIPCCL_FP32, unsigned long long>(a, s);
    return dt == ZIPCCL_BF16 ? launch_large<ZIPCCL_BF16, uint32_t>(a, s) : launch_large<ZIPCCL_FP32, uint32_t>(a, s);
}

} // namespace zipccl
