/*
 * Compress side of libzipccl.so for gfx950 (CDNA4, wave64): k_compress, k_tile_scan, k_place.
 *
 * compress   : paper section 4 (split, 3-bit code, zero-points) with the kernel steps of
 *              section 4.2 re-designed for wave64: one wave handles a group of 512 values,
 *              8 values per lane (consecutive: one 16-byte load for bf16; whole fp32 groups: two
 *              quads, one from each half of the group, one 16-byte load each), a workgroup of
 *              8 or 16 waves handles a tile of 16 groups.  Per lane the work is SWAR on packed
 *              words: v_perm_b32 gathers the sign/mantissa and exponent bytes, packed 16-bit
 *              sub/min produce the codes, v_dot4_u32_u8 transposes code bits into plane bytes.
 *              Plane bytes and zero-point exponents are staged in LDS and leave as wide
 *              stores.  The zero-point offsets of section 4.2.3 are an exclusive prefix in
 *              element order (lane -> wave -> tile -> chunk), so the output is deterministic.
 *              The chunk-wide level, which the paper does with a block-level atomic add, has four forms.
 *              k_compress<kModeDirect>, chunks of a few tiles (two at most where the next form can be had): a workgroup counts
 *              the zero-points of its chunk's tiles before its own itself.
 *              k_compress<kModeChained>, a scan in one pass by tagged words: a workgroup tells its tile's count as soon as the values
 *              are there, writes everything whose place is known (SM, LO, planes) and then adds up what the tiles
 *              before have told (chain_prefix, which bounds that wait).  One launch, nothing moved twice.
 *              k_compress<kModeStash>, calls that may not chain (launch_compress_chained) or had better not (chained_pays):
 *              the zero-point exponents are parked in a stash; the per-tile counts become per-chunk prefixes inside
 *              k_place (chunks of up to kPlaceScanTiles tiles) or in k_tile_scan; k_place moves each
 *              tile's exponents to their final place and finishes index and header.
 *              k_compress<kModeCount> and <kModeEmit>, calls that may not chain, without room for a stash: counts,
 *              k_tile_scan, and everything else from a second read.
 * Everything here is integer work.
 */
#include <atomic>
#include <chrono>
#include <mutex>
#include <type_traits>

#include "zipccl_device.h"

namespace zipccl {
namespace {

/*
 * Workspace of zipccl_compress_static: device memory that belongs to the library, one copy per GPU, held until
 * the process ends.  Host code never uses this name as an address: static_scratch() asks the runtime for the
 * array's device address, once per device, and hands that out.
 */
static __device__ __align__(256) uint8_t scratch[ZIPCCL_STATIC_SCRATCH_BYTES];

/* How a tile's values are read: every group whole; cut short by the end of a chunk of at least 8 values; a chunk of
 * fewer than 8. */
enum LoadForm { kWhole, kRest, kTiny };

/* kRest: the 16 bytes that hold piece q of the lane's values. */
template <int DT>
__device__ __forceinline__ u32x4 request_rest(const uint8_t* __restrict__ cin, uint64_t gbase, uint32_t lane, uint64_t n, uint32_t q)
{
    constexpr uint32_t ES = DT == ZIPCCL_BF16 ? 2u : 4u, PER16 = 16u / ES;
    const uint32_t left = gbase >= n ? 0u : (uint32_t)min(n - gbase, (uint64_t)kGroup);
    const int64_t base = left != 0u ? (int64_t)gbase : 0;                    /* a group past the end: the chunk's first */
    const uint32_t e = lane * PER16 + q * (kGroup / 2);
    const uint32_t here = e >= left ? 0u : min(left - e, PER16);
    /* one with none loads from where the group has 16 bytes, or from the 16 bytes the chunk ends with */
    const int32_t none = left != 0u && left < PER16 ? (int32_t)left - (int32_t)PER16 : 0;
    const int32_t at = here != 0u ? (int32_t)e - (int32_t)(PER16 - here) : none;
    return ld_stream_a2(cin + (base + at) * (int64_t)ES);
}

/*
 * Load the lane's 8 values of the group at chunk-relative element gbase: bf16: 8 consecutive ones; fp32: two quads,
 * [4 lane, 4 lane + 4) of the group's first half and of its second, so that each load is 16 contiguous bytes per
 * lane (32 contiguous bytes per lane cost ~7 % of the bandwidth, measured).
 * hp[k] packs the high 16-bit words of values 2k (low half) and 2k+1 (high half); lp[k] the low words (fp32 only).
 * vmask bit j = value j exists; values that do not exist read as 0.  kRest: no load is under a condition, and the caller
 * requests every group's before it has the first moved into place (`rest`: request_rest): a lane (or quad) that the
 * chunk's end cuts short loads the 16 bytes that end there and moves them down, one without values loads 16 bytes that exist.
 * With eight loads under conditions per lane, each waited for, the tile behind the last whole one was what a call ended
 * with: 8191 bf16 values in two kernels 9.4 -> 7.7 us, 8 chunks of 2 097 147 22.8 -> 17.1 us, fp32 37.3 -> 27.6.
 */
template <int DT, int FORM>
__device__ __forceinline__ void load_lane(const uint8_t* __restrict__ cin, uint64_t gbase, uint32_t lane, uint64_t n,
                                          uint32_t hp[4], uint32_t lp[4], uint32_t& vmask, const u32x4* rest = nullptr)
{
    constexpr uint32_t ES = DT == ZIPCCL_BF16 ? 2u : 4u, PER16 = 16u / ES, NQ = DT == ZIPCCL_BF16 ? 1u : 2u;
    u32x4 v[NQ];
    /* gbase is wave-uniform: uniform 64-bit base + 32-bit lane offset */
    if (FORM == kWhole) {
        const uint8_t* __restrict__ p = cin + gbase * ES;
        vmask = 0xFFu;
#pragma unroll
        for (uint32_t q = 0; q < NQ; ++q) v[q] = ld_stream_a2(p + q * 1024u + lane * 16u);
    } else {
        const uint32_t left = gbase >= n ? 0u : (uint32_t)min(n - gbase, (uint64_t)kGroup);      /* values of the group */
        vmask = 0;
#pragma unroll
        for (uint32_t q = 0; q < NQ; ++q) {
            const uint32_t e = lane * PER16 + q * (kGroup / 2);
            const uint32_t here = e >= left ? 0u : min(left - e, PER16);         /* values of these 16 bytes */
            vmask |= ((1u << here) - 1u) << (4u * q);
            uint32_t w[4];
            if (FORM == kRest) {
                const u32x4 t = rest[q];
                w[0] = t.x; w[1] = t.y; w[2] = t.z; w[3] = t.w;
                const uint32_t down = here != 0u ? PER16 - here : 0u;            /* values that belong to the 16 bytes before */
                const uint32_t dw = ES * down / 4u;                              /* whole words of them, 0 .. 3 */
#pragma unroll
                for (uint32_t bit = 0; bit < 2u; ++bit) {
                    if ((dw >> bit) & 1u) {
#pragma unroll
                        for (uint32_t k = 0; k < 4u; ++k) w[k] = k + (1u << bit) < 4u ? w[(k + (1u << bit)) & 3u] : 0u;
                    }
                }
                if (DT == ZIPCCL_BF16 && (down & 1u)) {
#pragma unroll
                    for (uint32_t k = 0; k < 4u; ++k) w[k] = (w[k] >> 16) | (k < 3u ? w[(k + 1u) & 3u] << 16 : 0u);
                }
                if (here == 0u) w[0] = w[1] = w[2] = w[3] = 0u;
            } else {
                w[0] = w[1] = w[2] = w[3] = 0u;
#pragma unroll
                for (uint32_t j = 0; j < PER16; ++j) {
                    if (j < here) {
                        if (DT == ZIPCCL_BF16) w[j >> 1] |= (uint32_t)reinterpret_cast<const uint16_t*>(cin)[e + j] << (16u * (j & 1u));
                        else w[j & 3u] = reinterpret_cast<const uint32_t*>(cin)[e + j];
                    }
                }
            }
            v[q] = u32x4{w[0], w[1], w[2], w[3]};
        }
    }
    if (DT == ZIPCCL_BF16) {
        hp[0] = v[0].x; hp[1] = v[0].y; hp[2] = v[0].z; hp[3] = v[0].w;
        lp[0] = lp[1] = lp[2] = lp[3] = 0;
    } else {
        const u32x4 a = v[0], b = v[NQ - 1];
        const uint32_t x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            hp[k] = perm(x[2 * k + 1], x[2 * k], 0x07060302u);
            lp[k] = perm(x[2 * k + 1], x[2 * k], 0x05040100u);
        }
    }
}

/* What a lane derives from its 8 values (section 4: split, code, zero-point detection). */
struct LaneEnc {
    uint32_t sm0, sm1;      /* 8 sign+mantissa bytes */
    uint32_t ex0, ex1;      /* 8 raw exponent bytes */
    uint32_t b0, b1, b2;    /* plane bytes: bit j = bit k of the code of value j */
    uint32_t m;             /* bit j = value j is a zero-point (before masking non-existent values) */
};

/*
 * SWAR encode of 8 values held as four packed pairs of 16-bit words.
 * k7 = (dec[1] - 1) << 7 in both halves; a value of exponent E has
 * t = E - (dec[1] - 1): code = t for t in 1..7, zero-point otherwise.
 */
__device__ __forceinline__ LaneEnc encode8(const uint32_t w[4], uint32_t k7)
{
    LaneEnc r;
    uint32_t c4[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t wa = w[2 * h], wb = w[2 * h + 1];
        const uint32_t lo = perm(wb, wa, 0x06040200u);   /* low bytes: mantissa | E bit 0 << 7 */
        const uint32_t hi = perm(wb, wa, 0x07050301u);   /* high bytes: sign << 7 | E >> 1 */
        const uint32_t sm = bfi(0x7F7F7F7Fu, lo, hi);
        const uint32_t ex = bfi(0xFEFEFEFEu, hi << 1, lo >> 7);
        /* (E << 7) - k7 per half, clamped to 8 << 7: 1..7 << 7 inside the window */
        const uint32_t qa = pk_min_u16(pk_sub_u16(wa & 0x7F807F80u, k7), 0x04000400u) >> 7;
        const uint32_t qb = pk_min_u16(pk_sub_u16(wb & 0x7F807F80u, k7), 0x04000400u) >> 7;
        c4[h] = perm(qb, qa, 0x06040200u);               /* 4 code bytes, 8 = outside the window */
        if (h == 0) { r.sm0 = sm; r.ex0 = ex; } else { r.sm1 = sm; r.ex1 = ex; }
    }
    /* bit-matrix transpose with dot products: sum of bit * 2^j over the 8 code bytes */
    const uint32_t p0 = __builtin_amdgcn_udot4(c4[1] & 0x01010101u, 0x80402010u,
                        __builtin_amdgcn_udot4(c4[0] & 0x01010101u, 0x08040201u, 0u, false), false);
    const uint32_t p1 = __builtin_amdgcn_udot4(c4[1] & 0x02020202u, 0x80402010u,
                        __builtin_amdgcn_udot4(c4[0] & 0x02020202u, 0x08040201u, 0u, false), false);
    const uint32_t p2 = __builtin_amdgcn_udot4(c4[1] & 0x04040404u, 0x80402010u,
                        __builtin_amdgcn_udot4(c4[0] & 0x04040404u, 0x08040201u, 0u, false), false);
    r.b0 = p0;
    r.b1 = p1 >> 1;
    r.b2 = p2 >> 2;
    r.m = ~(r.b0 | r.b1 | r.b2) & 0xFFu;
    return r;
}

/* Zero-points among the lane's 8 values (the count of encode8's r.m), added to cnt.  first = dec[1] << 7 in both
 * halves: (E - dec[1]) << 7 is below 7 << 7 inside the window. */
__device__ __forceinline__ uint32_t count8(const uint32_t w[4], uint32_t first, uint32_t cnt)
{
#pragma unroll
    for (int k = 0; k < 4; ++k)
        cnt += __popc((pk_min_u16(pk_sub_u16(w[k] & 0x7F807F80u, first), 0x03800380u) + 0x00800080u) & 0x04000400u);
    return cnt;
}

/* The groups of a wave are WAVES apart in the tile, which shares a short tile evenly among the waves (neighbours instead:
 * 64 chunks of 65 531 bf16 values 12.0 against 10.6 us, whole tiles 1 % slower). */
template <uint32_t WAVES>
__device__ __forceinline__ uint32_t group_of(uint32_t wave, uint32_t u) { return u * WAVES + wave; }

template <uint32_t GROUPS>
struct CompressShared {
    uint8_t planes[3][GROUPS * kGroup / 8];   /* plane bytes of the tile, natural order */
    uint8_t esc[GROUPS][kGroup];           /* zero-point exponents, one region per group */
    uint32_t gcnt[GROUPS];                 /* zero-points per group */
    uint32_t before[kGroupsPerTile];       /* kModeDirect, kModeChained: zero-points a wave found in the tiles before */
    uint32_t counted;                      /* kModeChained: waves that have counted << 16 | their zero-points */
    uint32_t missing;                      /* and whether the count of a tile before did not come */
    uint64_t open;                         /* or of which of 64, */
    uint32_t total;                        /* and whether the count of all tiles before these is known */
};

/* One group of one wave, its values already loaded (load_lane): encode, store SM/LO, stage planes and
 * zero-points in LDS. */
template <int DT, bool FAST, bool STORE, class SHARED>
__device__ __forceinline__ void compress_group(uint8_t* __restrict__ slot, const SlotLayout& L, uint64_t n,
                                               uint64_t ts, uint32_t gi, uint32_t k7, uint32_t lane,
                                               SHARED& sh, const uint32_t hp[4], const uint32_t lp[4],
                                               uint32_t vmask)
{
    const uint64_t gbase = ts + (uint64_t)gi * kGroup;      /* wave-uniform */
    const uint64_t e = gbase + lane * kLaneElems;
    const LaneEnc r = encode8(hp, k7);
    const uint32_t m = r.m & vmask;
    if (DT == ZIPCCL_FP32) {
        /* two quads per lane (see load_lane): bits 0..3 of the plane bytes and of m belong to values
           [4 lane, 4 lane + 4) of the group, bits 4..7 to the same values of its second half */
        if (STORE) {
            /* the sections' padding is written along (as zeros: values that do not exist read as 0) */
            const uint64_t ea = gbase + lane * 4u, eb = ea + kGroup / 2;
            uint8_t* __restrict__ sm = slot + L.sm + gbase;
            if (FAST || ea < pad128(n)) st_stream<uint32_t>(sm + lane * 4u, r.sm0);
            if (FAST || eb < pad128(n)) st_stream<uint32_t>((sm + kGroup / 2) + lane * 4u, r.sm1);
            uint8_t* __restrict__ lo = slot + L.lo + 2 * gbase;
            if (FAST || 2 * ea < pad128(2 * n)) st_stream<u32x2>(lo + lane * 8u, u32x2{lp[0], lp[1]});
            if (FAST || 2 * eb < pad128(2 * n)) st_stream<u32x2>((lo + kGroup) + lane * 8u, u32x2{lp[2], lp[3]});
            /* a plane byte = the nibbles of two neighbouring lanes: even lanes assemble the byte of the
               first half, odd lanes that of the second (three planes at once, one byte each) */
            const uint32_t p3 = r.b0 | (r.b1 << 8) | (r.b2 << 16);
            const uint32_t q3 = __builtin_amdgcn_update_dpp(0u, p3, 0xB1, 0xF, 0xF, false);   /* quad_perm [1,0,3,2] */
            const uint32_t b3 = (lane & 1u) ? (((q3 >> 4) & 0x0F0F0Fu) | (p3 & 0xF0F0F0u))
                                            : ((p3 & 0x0F0F0Fu) | ((q3 & 0x0F0F0Fu) << 4));
            const uint32_t pi = gi * 64u + (lane >> 1) + 32u * (lane & 1u);
            sh.planes[0][pi] = (uint8_t)b3;
            sh.planes[1][pi] = (uint8_t)(b3 >> 8);
            sh.planes[2][pi] = (uint8_t)(b3 >> 16);
        }
        /* element order = all first quads by lane, then all second quads: one scan of both counts */
        const uint32_t mA = m & 15u, mB = m >> 4;
        const uint32_t cA = __popc(mA), cB = __popc(mB);
        const uint32_t inc = wave_incl_scan(cA | (cB << 16));
        const uint32_t totA = __builtin_amdgcn_readlane(inc, 63) & 0xFFFFu;
        if (lane == 63) sh.gcnt[gi] = (inc & 0xFFFFu) + (inc >> 16);
        if (STORE) {
            uint8_t* dst = &sh.esc[gi][(inc & 0xFFFFu) - cA];
            uint32_t mm = mA;
            while (mm) {
                const uint32_t j = __builtin_ctz(mm);
                mm &= mm - 1u;
                *dst++ = (uint8_t)perm(r.ex1, r.ex0, j | 0x0C0C0C00u);
            }
            dst = &sh.esc[gi][totA + (inc >> 16) - cB];
            mm = mB << 4;
            while (mm) {
                const uint32_t j = __builtin_ctz(mm);
                mm &= mm - 1u;
                *dst++ = (uint8_t)perm(r.ex1, r.ex0, j | 0x0C0C0C00u);
            }
        }
        return;
    }
    if (STORE) {
        if (FAST || e < pad128(n)) st_stream<u32x2>((slot + L.sm + gbase) + lane * 8u, u32x2{r.sm0, r.sm1});
        const uint32_t pi = gi * 64u + lane;
        sh.planes[0][pi] = (uint8_t)r.b0;
        sh.planes[1][pi] = (uint8_t)r.b1;
        sh.planes[2][pi] = (uint8_t)r.b2;
    }
    const uint32_t cnt = __popc(m);
    const uint32_t inc = wave_incl_scan(cnt);
    if (lane == 63) sh.gcnt[gi] = inc;
    if (STORE) {
        /* the lane's zero-point exponents, in element order, at its offset inside the group */
        uint8_t* dst = &sh.esc[gi][inc - cnt];
        uint32_t mm = m;
        while (mm) {
            const uint32_t j = __builtin_ctz(mm);
            mm &= mm - 1u;
            *dst++ = (uint8_t)perm(r.ex1, r.ex0, j | 0x0C0C0C00u);
        }
    }
}

/*
 * Chunk header, zeroed IDX / ESC padding and chunk_bytes, once the chunk's zero-point count is
 * known.  Called by NT cooperating threads numbered tid = 0..NT-1.
 */
template <int DT, uint32_t NT>
__device__ __forceinline__ void finish_chunk(uint8_t* __restrict__ slot, const SlotLayout& L, uint64_t n,
                                             uint64_t n_esc, uint32_t dec_lo, uint32_t dec_hi,
                                             uint64_t* chunk_bytes, uint32_t tid)
{
    const uint64_t ng = (n + kGroup - 1) / kGroup;
    const uint64_t cbytes = L.esc + pad128(n_esc);
    uint32_t* __restrict__ idx = reinterpret_cast<uint32_t*>(slot + L.idx);
    uint8_t* __restrict__ esc = slot + L.esc;
    for (uint32_t i = tid; i < 32u; i += NT) {
        uint32_t w = 0;
        switch (i) {
            case 0: w = kMagic; break;
            case 1: w = kVersion; break;
            case 2: w = (uint32_t)DT; break;
            case 3: w = kGroup; break;
            case 4: w = (uint32_t)n; break;
            case 5: w = (uint32_t)(n >> 32); break;
            case 6: w = n_esc; break;
            case 7: w = (uint32_t)(n_esc >> 32); break;
            case 8: w = (uint32_t)cbytes; break;
            case 9: w = (uint32_t)(cbytes >> 32); break;
            case 10: w = dec_lo; break;
            case 11: w = dec_hi; break;
            default: break;
        }
        reinterpret_cast<uint32_t*>(slot)[i] = w;
        const uint64_t ie = ng + i;                         /* zero the IDX padding */
        if (4 * ie < pad128(4 * ng)) idx[ie] = 0;
    }
    for (uint32_t i = tid; i < 128u; i += NT) {             /* zero the ESC padding */
        const uint64_t je = n_esc + i;
        if (je < pad128(n_esc)) esc[je] = 0;
    }
    if (tid == 0 && chunk_bytes) *chunk_bytes = cbytes;
}

/* Kernel arguments: CompressArgs without its table, which follows in the form that the launch allows; small ones, see
 * EqualSplit. */
struct CompressIo {
    const uint8_t* in;
    uint8_t* out;
    uint64_t* chunk_bytes;
    const uint32_t* d_table;
    uint32_t dec_lo, table_stride;
};
struct NoParking {};                                        /* kModeDirect */
struct Parking {
    uint32_t *tile_total, *tile_prefix;
    uint8_t* stash;
};
/* kModeChained: what the tiles of a launch tell one another, in words that hold a count and this launch's tag (chain_tag).  A word
 * with another tag has not been told yet, so the words need not be cleared.  A chunk's tiles have one each, and behind these the 64th, 128th, ... tile two more for the count of all
 * tiles up to it. */
struct Chain {
    uint64_t* words;
    uint64_t tag;
    uint32_t many;                                          /* rounds of workgroups: see chain_prefix */
};
constexpr uint32_t kChainStep = 64;
#ifndef ZIPCCL_CHAIN_PATIENCE
#define ZIPCCL_CHAIN_PATIENCE 128
#endif
constexpr uint32_t kChainPatience = ZIPCCL_CHAIN_PATIENCE;   /* how often a wave looks again for words that are not there */

/* dec[0..3] and dec[4..7]: from the kernel arguments (dec[1..7] are consecutive, the host has checked it) or, if the table
 * was estimated on the device, two words in its memory. */
__device__ __forceinline__ void table_words(const CompressIo& a, uint32_t c, uint32_t& dec_lo, uint32_t& dec_hi)
{
    if (a.d_table) {
        const uint32_t* __restrict__ tab_c = a.d_table + c * a.table_stride;      /* one table for all chunks, or one each */
        dec_lo = tab_c[0];
        dec_hi = tab_c[1];
    } else {
        dec_lo = a.dec_lo;
        dec_hi = ((a.dec_lo >> 8) & 0xFFu) * 0x01010101u + 0x06050403u;
    }
}

__device__ __forceinline__ uint64_t peek(const uint64_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void tell(uint64_t* p, uint64_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

/*
 * Zero-points in the chunk's tiles before tile t, as parts in sh.before (one per wave).  Words of tiles far back would be most of what is
 * read in long chunks: from `reach` tiles on, as many as run at a time, the counts start behind the last multiple of
 * kChainStep at least `reach` tiles back, whose total another round of workgroups has told: 2^29 bf16 values in one chunk 487 us without,
 * 292 now.  (Fewer words through totals of 16 and 256 tiles cost more than they save: whoever adds them up has stores under way,
 * which its loads wait for; 587 us.)
 *
 * Looks hold up one another and the words they look for, so between two of them a wave sleeps, some 1000 cycles in all but the
 * smallest launches; and in launches of many rounds a workgroup that has few words to read sleeps before the first look, which
 * would come too early (64 chunks of 2^23 bf16 values without / with 290 us for 314, of 3.7 million 131 for 141; at 2^24 it costs a microsecond; fp32
 * tiles, which take twice as long, lose by it: 64 of 2^21 160 us without, 162 with).
 *
 * Workgroups start in order, so those waited for run already or are next, unless other kernels hold part of the chip.  So the wait is bounded: a
 * workgroup one of whose waves has looked kChainPatience times, some 0.2 ms, goes back from its tile to the nearest total that has been told, and counts the
 * tiles that are missing on the way itself, from the input, and tells their counts on their behalf.  No workgroup depends on
 * another for its end.
 */
template <int DT, uint32_t WAVES, uint32_t GROUPS, class SHARED>
__device__ __forceinline__ void chain_prefix(const Chain& chain, uint64_t* words, uint32_t tiles, uint32_t t, const uint8_t* __restrict__ cin, uint64_t n,
                                             uint32_t e0, SHARED& sh, uint32_t lane, uint32_t wave)
{
    constexpr uint32_t NT = 64u * WAVES, GPW = GROUPS / WAVES;
    constexpr uint32_t reach = 8192u / WAVES;                /* eight waves per SIMD: 32 per compute unit, of 256 */
    constexpr int nap = GROUPS == 16u ? 1 : 16;              /* of 64 cycles */
    auto is_count = [&](uint64_t v) { return chain_told(v, chain.tag); };
    uint32_t from = 0;
    if (GROUPS > kGroupsPerTile && t >= reach + kChainStep) from = (t - reach) & ~(kChainStep - 1u);
    if (chain.many != 0u && from == 0u) __builtin_amdgcn_s_sleep(28);
    const uint64_t* const upto = words + tiles + 2u * (from / kChainStep) - 2u;   /* if from is not 0 */
    uint32_t sum = 0, left = kChainPatience;
    bool missing = false;
    for (uint32_t i = from + threadIdx.x; i < t + (from != 0u ? 2u : 0u); i += NT) {
        const uint64_t* const p = i < t ? words + i : upto + (i - t);
        uint64_t v = peek(p);
        while (left != 0u && __ballot(!is_count(v)) != 0u) {    /* the same in all lanes that have a word */
            --left;
            __builtin_amdgcn_s_sleep(nap);
            if (!is_count(v)) v = peek(p);
        }
        missing |= !is_count(v);
        sum += (uint32_t)(v & kChainCount) << (i == t + 1u ? 24u : 0u);
    }
    sum = wave_incl_scan(sum);
    if (lane == 63u) sh.before[wave] = sum;
    if (missing) sh.missing = 1u;
    __syncthreads();
    if (sh.missing == 0u) return;

    /* from the nearest tile back, 64 at a time, each with the total before them */
    sum = 0;
    bool total = false;
    for (uint32_t end = t; end != 0u && !total;) {
        const uint32_t base = (end - 1u) & ~(kChainStep - 1u);
        __syncthreads();
        if (wave == 0u) {
            const bool some = base + lane < end;
            const uint64_t v = some ? peek(words + base + lane) : 0u;
            const bool told = some && is_count(v);
            sum += told ? (uint32_t)(v & kChainCount) : 0u;
            const uint64_t open = __ballot(some && !told);
            if (lane == 0u) sh.open = open;
        } else if (wave == 1u) {
            bool known = false;
            if (GROUPS > kGroupsPerTile && base != 0u) {
                const uint64_t v = peek(words + tiles + 2u * (base / kChainStep) - 2u + (lane & 1u));
                known = __ballot(is_count(v)) == ~0ull;
                if (known && lane < 2u) sum += (uint32_t)(v & kChainCount) << (24u * lane);
            }
            if (lane == 0u) sh.total = known;
        }
        __syncthreads();
        total = sh.total != 0u;
        for (uint64_t open = sh.open; open != 0u;) {
            const uint32_t j = 63u - (uint32_t)__builtin_clzll(open);
            open ^= 1ull << j;
            __syncthreads();
            if (threadIdx.x == 0u) {
                const uint64_t v = peek(words + base + j);
                sh.missing = !is_count(v);
                sh.counted = is_count(v) ? (uint32_t)(v & kChainCount) : 0u;
            }
            __syncthreads();
            if (sh.missing != 0u) {
                uint32_t h[GPW][4], l[4], m, cnt = 0;
#pragma unroll
                for (uint32_t u = 0; u < GPW; ++u) load_lane<DT, kWhole>(cin, (uint64_t)(base + j) * (GROUPS * kGroup) + group_of<WAVES>(wave, u) * kGroup, lane, n, h[u], l, m);
#pragma unroll
                for (uint32_t u = 0; u < GPW; ++u) cnt = count8(h[u], e0 * 0x00800080u, cnt);
                cnt = __builtin_amdgcn_readlane(wave_incl_scan(cnt), 63);
                if (lane == 0u) atomicAdd(&sh.counted, cnt);
                __syncthreads();
                if (threadIdx.x == 0u) tell(words + base + j, chain.tag | sh.counted);
            }
            if (threadIdx.x == 0u) sum += sh.counted;
        }
        end = base;
    }
    sum = wave_incl_scan(sum);
    if (lane == 63u) sh.before[wave] = sum;                  /* 0 but for the first two */
    __syncthreads();
}

/* WAVES (8 or 16, see kWideTiles) share a tile: with four, of four groups each, 2^22 to 2^24 bf16 values took 3 to 6 % longer (from
 * 2^27 on the same), and in launches that leave most of the chip empty a wave's encodes came one after the other (32 x 4096
 * values 4.5 us, 3.8 with 16). */
template <int DT, int MODE, uint32_t WAVES, uint32_t GROUPS, class PARK, class SPLIT>
__global__ __launch_bounds__(64u * WAVES) void k_compress(const CompressIo a, const PARK park, const SPLIT split)
{
    constexpr uint32_t ES = DT == ZIPCCL_BF16 ? 2u : 4u;
    constexpr bool STORE = MODE != kModeCount;
    constexpr uint32_t GPW = GROUPS / WAVES, TILE = GROUPS * kGroup;
    __shared__ __attribute__((aligned(16))) CompressShared<GROUPS> sh;

    /* grid = (tiles of the largest chunk, chunks): no search, the chunk's geometry is three scalar loads at most */
    const uint32_t c = blockIdx.y, bx = blockIdx.x;
    const ChunkPlace place = place_of(split, c, DT);
    const uint32_t tiles = (place.tiles + GROUPS / kGroupsPerTile - 1u) / (GROUPS / kGroupsPerTile);
    if (bx >= tiles) return;
    const bool last_tile = bx + 1u == tiles;
    const uint64_t n = place.n;
    const uint64_t ts = (uint64_t)bx * TILE;
    const uint8_t* __restrict__ cin = a.in + place.elem_off * ES;
    uint8_t* __restrict__ slot = a.out + place.slot_off;
    const SlotLayout L = slot_layout(n, DT);
    const bool fast = ts + TILE <= n;                       /* a whole tile */
    const uint32_t lane = lane_id();
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   /* keep wave-derived math scalar */
    uint32_t dec_lo, dec_hi;
    table_words(a, c, dec_lo, dec_hi);
    const uint32_t e0 = (dec_lo >> 8) & 0xFFu;
    const uint32_t k7 = ((e0 - 1u) << 7) * 0x00010001u;

    /* all of the wave's loads go out before its first group is encoded: more bytes in flight, and no wait for a load ever
       includes the stores of the group before */
    uint32_t hp[GPW][4], lp[GPW][4], vm[GPW];
    /* kModeDirect: the zero-points of the chunk's tiles before this one, which are few, whole, and read by other
       workgroups too; two tiles' loads in flight together, while the tile's own travel */
    auto count_before = [&] {
        const uint32_t first = e0 * 0x00800080u;
        uint32_t cnt = 0;
        for (uint32_t b = 0; b < bx; b += 2) {
            uint32_t h[2][GPW][4], l[4], m;
#pragma unroll
            for (uint32_t k = 0; k < 2; ++k)
#pragma unroll
                for (uint32_t u = 0; u < GPW; ++u)
                    load_lane<DT, kWhole>(cin, (uint64_t)min(b + k, bx - 1u) * TILE + group_of<WAVES>(wave, u) * kGroup, lane, n, h[k][u], l, m);
            uint32_t second = 0;
#pragma unroll
            for (uint32_t u = 0; u < GPW; ++u) {
                cnt = count8(h[0][u], first, cnt);
                second = count8(h[1][u], first, second);
            }
            if (b + 1u < bx) cnt += second;
        }
        cnt = wave_incl_scan(cnt);
        if (lane == 63) sh.before[wave] = cnt;
    };
    /* kModeChained: the tile's own count, before anything else is done with its values; the wave that adds the last part of it
       tells the tiles behind */
    uint64_t* words = nullptr;
    if constexpr (MODE == kModeChained) {
        words = park.words + place.tile;
        if (threadIdx.x == 0) sh.counted = sh.missing = 0;
    }
    auto tell_own = [&] {
        if constexpr (MODE == kModeChained) {
            __syncthreads();                                /* sh.counted is 0 */
            uint32_t cnt = 0;
#pragma unroll
            for (uint32_t u = 0; u < GPW; ++u) cnt = count8(hp[u], e0 * 0x00800080u, cnt) - __popc(~vm[u] & 0xFFu);  /* values that do not exist are zeros */
            cnt = __builtin_amdgcn_readlane(wave_incl_scan(cnt), 63) | 0x10000u;
            if (lane == 0) {
                const uint32_t sum = atomicAdd(&sh.counted, cnt) + cnt;
                if (sum >> 16 == WAVES) tell(words + bx, park.tag | (sum & 0xFFFFu));
            }
        }
    };
    if (fast) {
#pragma unroll
        for (uint32_t u = 0; u < GPW; ++u)
            load_lane<DT, kWhole>(cin, ts + (uint64_t)group_of<WAVES>(wave, u) * kGroup, lane, n, hp[u], lp[u], vm[u]);
        if (MODE == kModeDirect) count_before();
        tell_own();
#pragma unroll
        for (uint32_t u = 0; u < GPW; ++u)
            compress_group<DT, true, STORE>(slot, L, n, ts, group_of<WAVES>(wave, u), k7, lane, sh, hp[u], lp[u], vm[u]);
    } else {
        if (n >= 8u) {
            /* every request before the first use of what one brings: left to itself the compiler waits for each of the
               four loads (fp32: for each four of eight) before the next (5000 bf16 values 4.9 -> 4.45 us, 8195 in two reads
               9.0 -> 8.2) */
            constexpr uint32_t NQ = DT == ZIPCCL_BF16 ? 1u : 2u;
            u32x4 rest[GPW][NQ];
#pragma unroll
            for (uint32_t u = 0; u < GPW; ++u)
#pragma unroll
                for (uint32_t q = 0; q < NQ; ++q) rest[u][q] = request_rest<DT>(cin, ts + (uint64_t)group_of<WAVES>(wave, u) * kGroup, lane, n, q);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (uint32_t u = 0; u < GPW; ++u)
                load_lane<DT, kRest>(cin, ts + (uint64_t)group_of<WAVES>(wave, u) * kGroup, lane, n, hp[u], lp[u], vm[u], rest[u]);
        } else {
#pragma unroll
            for (uint32_t u = 0; u < GPW; ++u)
                load_lane<DT, kTiny>(cin, ts + (uint64_t)group_of<WAVES>(wave, u) * kGroup, lane, n, hp[u], lp[u], vm[u]);
        }
        if (MODE == kModeDirect) count_before();
        tell_own();
#pragma unroll
        for (uint32_t u = 0; u < GPW; ++u)
            compress_group<DT, false, STORE>(slot, L, n, ts, group_of<WAVES>(wave, u), k7, lane, sh, hp[u], lp[u], vm[u]);
    }
    __syncthreads();

    /* every wave: tile-level exclusive prefix of the 16 group counts (lanes 0..15 hold them) */
    const uint32_t gc = lane < GROUPS ? sh.gcnt[lane] : 0u;
    const uint32_t ginc = GROUPS <= 16u ? row_incl_scan(gc) : wave_incl_scan(gc);
    const uint32_t gex = ginc - gc;
    const uint32_t tile_total = __builtin_amdgcn_readlane(ginc, GROUPS - 1);
    if constexpr (MODE == kModeCount || MODE == kModeStash) {
        if (threadIdx.x == 0) park.tile_total[place.tile + bx] = tile_total;
        if (MODE == kModeCount) return;
    }

    /* waves 1, 2, ...: 1 KiB of a plane each, 16 bytes per lane */
    auto store_planes = [&] {
#pragma unroll
        for (uint32_t u = 0; u < (3u * GROUPS / 16u + WAVES - 2u) / (WAVES - 1u); ++u) {
            const uint32_t piece = wave - 1u + u * (WAVES - 1u);
            if (wave != 0u && piece < 3u * GROUPS / 16u) {
                const uint32_t k = piece % 3u, at = piece / 3u * 1024u;
                const uint64_t pb = ts / 8 + at + lane * 16u;
                if (fast || pb < L.plane_bytes)
                    st_stream<u32x4>((slot + L.p0 + k * L.plane_bytes + ts / 8 + at) + lane * 16u,
                                     *reinterpret_cast<const u32x4*>(&sh.planes[k][at + lane * 16u]));
            }
        }
    };
    if (MODE == kModeChained) store_planes();

    if constexpr (MODE == kModeChained) chain_prefix<DT, WAVES, GROUPS>(park, words, tiles, bx, cin, n, e0, sh, lane, wave);

    /* kModeStash works tile-local, the other forms know the zero-points of the chunk before this tile */
    uint32_t P = 0;
    if constexpr (MODE == kModeEmit) P = park.tile_prefix[place.tile + bx];
    if (MODE == kModeDirect || MODE == kModeChained) P = __builtin_amdgcn_readlane(row_incl_scan(lane < WAVES ? sh.before[lane] : 0u), WAVES - 1u);
    if constexpr (MODE == kModeChained && GROUPS > kGroupsPerTile) {
        if (bx % kChainStep == kChainStep - 1u && threadIdx.x < 2u) {
            const uint32_t upto = P + tile_total;
            tell(words + tiles + bx / kChainStep * 2u + threadIdx.x, park.tag | (threadIdx.x == 0u ? upto & kChainCount : upto >> 24));
        }
    }
    const uint64_t ng = (n + kGroup - 1) / kGroup;
    uint32_t* __restrict__ idx = reinterpret_cast<uint32_t*>(slot + L.idx);
    uint8_t* __restrict__ esc = slot + L.esc + P;
    if constexpr (MODE == kModeStash) esc = park.stash + place.elem_off + ts;

    if (wave == 0) {
        /* group index (section 4.2.3); k_place adds the tile's prefix in stash mode */
        const uint64_t g = ts / kGroup + lane;
        if (lane < GROUPS && g < ng) idx[g] = P + gex;
    }
    if (MODE != kModeChained) store_planes();
    /* zero-point exponents: every wave copies the segments of its own groups, in element order; of most groups there are no
       more than 64, whose LDS reads go out together */
    uint8_t first64[GPW];
#pragma unroll
    for (uint32_t u = 0; u < GPW; ++u) first64[u] = sh.esc[group_of<WAVES>(wave, u)][lane];
#pragma unroll
    for (uint32_t u = 0; u < GPW; ++u) {
        const uint32_t gi = group_of<WAVES>(wave, u);
        const uint32_t cnt = __builtin_amdgcn_readlane(gc, gi);
        uint8_t* dst = esc + __builtin_amdgcn_readlane(gex, gi);
        if (lane < cnt) dst[lane] = first64[u];
#pragma unroll 1
        for (uint32_t i = lane + 64u; i < cnt; i += 64u) dst[i] = sh.esc[gi][i];
    }

    if ((MODE == kModeEmit || MODE == kModeDirect || MODE == kModeChained) && last_tile)
        finish_chunk<DT, 64u * WAVES>(slot, L, n, (uint64_t)P + tile_total, dec_lo, dec_hi,
                                   a.chunk_bytes ? a.chunk_bytes + c : nullptr, threadIdx.x);
}

/* Move nw aligned words: word i of dst = bytes [4i + sh8, 4i + sh8 + 4) of the aligned word array s32.
 * `width` lanes (this one is number `lane`) share the job, W words per lane and step, with all
 * loads of a step issued before its stores.  Reads reach at most 7 bytes past the last source byte. */
template <uint32_t W>
__device__ __forceinline__ void move_words(uint32_t* __restrict__ d32, const uint32_t* __restrict__ s32,
                                           uint32_t nw, uint32_t sh8, uint32_t lane, uint32_t width)
{
    for (uint32_t i0 = 0; i0 < nw; i0 += W * width) {
        uint32_t lo[W], hi[W];
#pragma unroll
        for (uint32_t k = 0; k < W; ++k) {
            const uint32_t i = i0 + k * width + lane;
            lo[k] = hi[k] = 0;
            if (i < nw) { lo[k] = s32[i]; hi[k] = s32[i + 1]; }
        }
#pragma unroll
        for (uint32_t k = 0; k < W; ++k) {
            const uint32_t i = i0 + k * width + lane;
            if (i < nw) d32[i] = __builtin_amdgcn_alignbyte(hi[k], lo[k], sh8);
        }
    }
}

/*
 * Stash mode, after k_tile_scan: 16 lanes per tile (16 tiles per workgroup, so that many tiles'
 * dependent loads are in flight per wave) move the tile's zero-point exponents from the stash
 * to ESC[P, P + count), add P to the tile's 16 index entries, and the last tile of a chunk
 * writes header, padding and chunk_bytes.  Tiles dense in zero-points (more than kPlaceBig
 * bytes) are moved afterwards, by one, two or four of the workgroup's waves each.
 */
/* SCAN: there was no k_tile_scan; the workgroup sums the chunk's tile counts before its own tiles itself
 * (chunks of at most kPlaceScanTiles tiles: the counts are few and cache-resident). */
template <int DT, bool SCAN, class SPLIT>
__global__ __launch_bounds__(kThreads) void k_place(const CompressIo a, const Parking park, const SPLIT split)
{
    constexpr uint32_t kSub = 16;                       /* lanes per tile */
    constexpr uint32_t kPlaceBig = 1024;                /* bytes a 16-lane group moves on its own */
    __shared__ uint32_t s_wave[kWavesPerBlock];
    __shared__ uint32_t s_ex[kThreads / kSub];
    __shared__ uint32_t s_nbig;
    __shared__ uint32_t s_big[kThreads / kSub];
    __shared__ uint64_t s_src[kThreads / kSub], s_dst[kThreads / kSub];
    __shared__ uint32_t s_nw[kThreads / kSub], s_sh[kThreads / kSub];
    constexpr uint32_t kAhead = 4;                      /* words per lane moved with what is requested ahead of the counts */
    if (threadIdx.x == 0) s_nbig = 0;

    /* grid = (16-tile groups of the largest chunk, chunks): the chunk's geometry is wave-uniform */
    const uint32_t c = blockIdx.y;
    const ChunkPlace place = place_of(split, c, DT);
    const uint32_t first = place.tile, ntc = place.tiles;
    if (blockIdx.x * (kThreads / kSub) >= ntc) return;  /* a shorter chunk than the largest of the launch */
    const uint64_t n = place.n;
    uint8_t* __restrict__ slot = a.out + place.slot_off;
    const SlotLayout L = slot_layout(n, DT);
    const uint32_t sub = threadIdx.x % kSub;
    const uint32_t tw = threadIdx.x / kSub;             /* tile inside the workgroup */
    const uint32_t ti = blockIdx.x * (kThreads / kSub) + tw;
    const uint32_t tl = min(ti, ntc - 1u);              /* past the last tile: the last one once more, not stored */

    /* Requested before anything is known: the tile's count, its 16 index entries, and the first bytes of its stash, 8 where
       a lane's 4 will be some of them, wherever the destination's words begin.  (The stash of a tile holds a byte for each of its
       values, and 64 readable ones follow the last.) */
    const uint8_t* __restrict__ src = park.stash + place.elem_off + (uint64_t)tl * kTile;
    const uint32_t room = (uint32_t)min(n - (uint64_t)tl * kTile, (uint64_t)kTile);       /* values of the tile */
    const uint64_t ng = (n + kGroup - 1) / kGroup;
    uint32_t* __restrict__ idx = reinterpret_cast<uint32_t*>(slot + L.idx);
    const uint64_t g = (uint64_t)tl * kGroupsPerTile + sub;
    const uint32_t cnt = park.tile_total[first + tl];
    const uint32_t idx_local = g < ng ? idx[g] : 0u;
    uint32_t w0[kAhead], w1[kAhead];
#pragma unroll
    for (uint32_t k = 0; k < kAhead; ++k) {
        const uint32_t at = 4u * (k * kSub + sub);
        typedef u32x2 u32x2_a1 __attribute__((aligned(1)));
        const u32x2 v = *reinterpret_cast<const u32x2_a1*>(src + (at < room ? at : 0u));
        w0[k] = v.x; w1[k] = v.y;
    }
    if (SCAN) {
        /* counts of the chunk's tiles before this workgroup's, and the exclusive prefix inside it */
        const uint32_t t0 = blockIdx.x * (kThreads / kSub);
        uint32_t part[4] = {0, 0, 0, 0};
        uint32_t i = threadIdx.x;
        for (; i + 3u * kThreads < t0; i += 4u * kThreads) {
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) part[k] += park.tile_total[first + i + k * kThreads];
        }
        for (; i < t0; i += kThreads) part[0] += park.tile_total[first + i];
        const uint32_t inc = wave_incl_scan((part[0] + part[1]) + (part[2] + part[3]));
        if ((threadIdx.x & 63u) == 63u) s_wave[threadIdx.x >> 6] = inc;
        if (threadIdx.x < kThreads / kSub) {            /* one row of 16 lanes */
            const uint32_t mine = t0 + threadIdx.x < ntc ? park.tile_total[first + t0 + threadIdx.x] : 0u;
            s_ex[threadIdx.x] = row_incl_scan(mine) - mine;
        }
    }
    __syncthreads();
    uint32_t dec_lo, dec_hi;
    table_words(a, c, dec_lo, dec_hi);

    if (ti < ntc) {
        uint32_t P;
        if (SCAN) P = ((s_wave[0] + s_wave[1]) + (s_wave[2] + s_wave[3])) + s_ex[tw];
        else P = park.tile_prefix[first + ti];
        if (P != 0u && g < ng) idx[g] = idx_local + P;

        /* byte-exact move to an arbitrarily aligned destination: head bytes, aligned words, tail bytes */
        uint8_t* __restrict__ dst = slot + L.esc + P;
        const uint32_t head = min((uint32_t)(-(int64_t)reinterpret_cast<uintptr_t>(dst)) & 3u, cnt);
        const uint32_t nw = (cnt - head) >> 2;
        const uint32_t done = head + 4u * nw, tail = cnt - done;
        uint32_t* __restrict__ d32 = reinterpret_cast<uint32_t*>(dst + head);
        if (sub == 0u) {
            for (uint32_t i = 0; i < head; ++i) dst[i] = (uint8_t)(w0[0] >> (8u * i));
        }
#pragma unroll
        for (uint32_t k = 0; k < kAhead; ++k) {
            const uint32_t i = k * kSub + sub;
            const uint32_t v = __builtin_amdgcn_alignbyte(w1[k], w0[k], head);
            if (i < nw) d32[i] = v;
            if (i == nw)
                for (uint32_t j = 0; j < tail; ++j) dst[done + j] = (uint8_t)(v >> (8u * j));
        }
        if (nw >= kAhead * kSub) {                      /* more than that */
            uint8_t tb = 0;
            if (sub < tail) tb = src[done + sub];
            const uint8_t* const from = src + head + 4u * kAhead * kSub;
            const uint32_t sh8 = reinterpret_cast<uintptr_t>(from) & 3u;
            const uint32_t* __restrict__ s32 = reinterpret_cast<const uint32_t*>(reinterpret_cast<uintptr_t>(from) & ~(uintptr_t)3);
            if (cnt <= kPlaceBig) {
                move_words<4>(d32 + kAhead * kSub, s32, nw - kAhead * kSub, sh8, sub, kSub);
            } else if (sub == 0) {
                const uint32_t k = atomicAdd(&s_nbig, 1u);
                s_big[k] = tw;
                s_src[tw] = reinterpret_cast<uint64_t>(s32);
                s_dst[tw] = reinterpret_cast<uint64_t>(d32 + kAhead * kSub);
                s_nw[tw] = nw - kAhead * kSub;
                s_sh[tw] = sh8;
            }
            if (sub < tail) dst[done + sub] = tb;
        }
        if (ti + 1u == ntc)
            finish_chunk<DT, kSub>(slot, L, n, (uint64_t)P + cnt, dec_lo, dec_hi,
                                   a.chunk_bytes ? a.chunk_bytes + c : nullptr, sub);
    }
    __syncthreads();
    const uint32_t nbig = s_nbig;
    /* all four waves on a single tile, two on each of two or three, one on each of more; 8 words per lane and step (16 tiles
       of nothing but zero-points one after the other: 2^20 values 49.8 us, 36.4 a wave each) */
    const uint32_t wave = threadIdx.x >> 6;
    auto move = [&](auto waves) {
        constexpr uint32_t per = decltype(waves)::value;
        for (uint32_t b = wave / per; b < nbig; b += kWavesPerBlock / per) {
            const uint32_t k = s_big[b];
            move_words<8>(reinterpret_cast<uint32_t*>(s_dst[k]), reinterpret_cast<const uint32_t*>(s_src[k]), s_nw[k],
                          s_sh[k], (wave % per) * 64u + lane_id(), per * 64u);
        }
    };
    if (nbig == 1u) move(std::integral_constant<uint32_t, 4>{});
    else if (nbig <= 3u) move(std::integral_constant<uint32_t, 2>{});
    else move(std::integral_constant<uint32_t, 1>{});
}

/*
 * Exclusive prefix of every chunk's per-tile zero-point counts.  Workgroup (x, y) owns segment x
 * (kScanSeg tiles) of chunk y: it sums the chunk's counts before its segment itself (the count
 * array is small and cache-resident, and this keeps workgroups independent of each other), then
 * scans its segment.
 */
constexpr uint32_t kScanSeg = 4 * kThreads;

__global__ __launch_bounds__(kThreads) void k_tile_scan(const CompressArgs a)
{
    __shared__ uint32_t s_wave[kWavesPerBlock];
    const uint32_t c = blockIdx.y;
    const uint32_t first = a.tab.tile_start[c], end = a.tab.tile_start[c + 1];
    const uint32_t seg0 = first + blockIdx.x * kScanSeg;
    if (seg0 >= end) return;
    const uint32_t lane = lane_id(), wave = threadIdx.x >> 6;

    /* counts of the chunk before this segment */
    uint32_t part[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    uint32_t i = first + threadIdx.x;
    for (; i + 7u * kThreads < seg0; i += 8u * kThreads) {     /* eight independent loads in flight per thread */
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k) part[k] += a.tile_total[i + k * kThreads];
    }
    for (; i < seg0; i += kThreads) part[0] += a.tile_total[i];
    uint32_t before = ((part[0] + part[1]) + (part[2] + part[3])) + ((part[4] + part[5]) + (part[6] + part[7]));
    before = wave_incl_scan(before);
    if (lane == 63) s_wave[wave] = before;
    __syncthreads();
    uint32_t base = 0;
#pragma unroll
    for (uint32_t w = 0; w < kWavesPerBlock; ++w) base += s_wave[w];
    __syncthreads();

    /* scan of the segment: four consecutive tiles per thread */
    const uint32_t i0 = seg0 + 4u * threadIdx.x;
    uint32_t v[4], mine = 0;
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
        v[k] = i0 + k < end ? a.tile_total[i0 + k] : 0u;
        mine += v[k];
    }
    const uint32_t inc = wave_incl_scan(mine);
    if (lane == 63) s_wave[wave] = inc;
    __syncthreads();
    uint32_t run = base + inc - mine;
    for (uint32_t w = 0; w < wave; ++w) run += s_wave[w];
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
        if (i0 + k < end) a.tile_prefix[i0 + k] = run;
        run += v[k];
    }
}

} // namespace

int static_scratch(void** ptr, size_t* bytes)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* addr[kMaxDevices];            /* device address of `scratch` on each GPU, once resolved */
    int dev = -1;
    const hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return (int)e;
    if (dev < 0 || dev >= kMaxDevices) return (int)hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        const hipError_t es = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));   /* for the current device */
        if (es != hipSuccess) return (int)es;
        if (!p) return (int)hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    *bytes = sizeof scratch;
    return 0;
}

static CompressIo io_of(const CompressArgs& a) { return CompressIo{a.in, a.out, a.chunk_bytes, a.d_table, a.dec_lo, a.table_stride}; }
static Parking parking_of(const CompressArgs& a) { return Parking{a.tile_total, a.tile_prefix, a.stash}; }

/*
 * Waves per tile: 16, one group each, for fp32, whose groups are two loads each, and in bf16 launches of up to this many
 * tiles, where every wave beyond the first few has a SIMD of its own; 8 in larger bf16 launches, where 16 hold too
 * few bytes in flight.  us, 4 / 8 / 16 waves, bf16: 2^17 values in 8 chunks 4.5 / 4.0 / 3.8, 2^21 7.9 / 7.55 / 7.5, 9 * 2^18 7.9 / 7.7 / 7.8, 2^22
 * in 8 8.4 / 8.1 / 8.9, 2^23 11.3 / 10.6 / 12.4, 2^24 15.8 / 15.4 / 18.5, 2^27 in 64 82.0 / 81.7 / 100.6, 2^29 302.4 / 302.4 / 390, with rows of gains
 * 327.6 / 323.4 / 413; fp32: 2^17 5.5 / 4.65 / 4.2, 2^23 17.1 / 16.5 / 16.4, 2^27 in 64 175 / 171 / 168.
 */
constexpr uint32_t kWideTiles = 256;

/* The smallest arguments that hold the split; the two-read kernels, whose calls are none of the small ones, take the table. */
template <int DT>
static void launch_compress_dt(int mode, const CompressArgs& a, hipStream_t s)
{
    const dim3 grid(max_chunk_tiles(a.tab), a.tab.n_chunks);
    const CompressIo io = io_of(a);
    const Parking park = parking_of(a);
    const bool equal = is_equal_split(a.tab);
#define ZIPCCL_LAUNCH(MODE, PARK, P, SPLIT, S)                                                                         \
    do {                                                                                                               \
        if constexpr (DT == ZIPCCL_BF16) {                                                                             \
            if (a.tab.tile_start[a.tab.n_chunks] > kWideTiles) {                                                       \
                hipLaunchKernelGGL((k_compress<DT, MODE, 8u, 16u, PARK, SPLIT>), grid, dim3(512u), 0, s, io, P, S);         \
                break;                                                                                                 \
            }                                                                                                          \
        }                                                                                                              \
        hipLaunchKernelGGL((k_compress<DT, MODE, 16u, 16u, PARK, SPLIT>), grid, dim3(1024u), 0, s, io, P, S);               \
    } while (0)
    if (mode == kModeDirect) {
        if (equal) ZIPCCL_LAUNCH(kModeDirect, NoParking, NoParking{}, EqualSplit, equal_split(a.tab));
        else if (is_few_split(a.tab)) ZIPCCL_LAUNCH(kModeDirect, NoParking, NoParking{}, FewSplit, few_split(a.tab));
        else ZIPCCL_LAUNCH(kModeDirect, NoParking, NoParking{}, ChunkTab, a.tab);
    } else if (mode == kModeStash) {
        if (equal) ZIPCCL_LAUNCH(kModeStash, Parking, park, EqualSplit, equal_split(a.tab));
        else ZIPCCL_LAUNCH(kModeStash, Parking, park, ChunkTab, a.tab);
    } else if (mode == kModeCount) {
        ZIPCCL_LAUNCH(kModeCount, Parking, park, ChunkTab, a.tab);
    } else {
        ZIPCCL_LAUNCH(kModeEmit, Parking, park, ChunkTab, a.tab);
    }
#undef ZIPCCL_LAUNCH
}

/* of 8192 values: launch_chained_dt */
constexpr uint32_t kSmallTiles = 640;
template <int DT>
constexpr uint32_t kSmallTilesEstimated = DT == ZIPCCL_BF16 ? 2304u : 2048u;

/* The tag of a launch (Chain), whose number is counted up from one that differs from process to process.  What a workspace holds of
 * earlier launches of this process has other tags; what else it holds would have to be this very one of 2^40 in a word of a tile
 * that is late. */
static uint64_t launch_tag()
{
    static std::atomic<uint64_t> next{[] {
        uint64_t x = (uint64_t)std::chrono::system_clock::now().time_since_epoch().count() ^ (reinterpret_cast<uintptr_t>(&x) << 20);
        x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;         /* splitmix64 */
        x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
        return (x ^ (x >> 31)) % kChainTags;
    }()};
    return chain_tag(next.fetch_add(1, std::memory_order_relaxed));
}

/* Whether the table is one for the whole tensor in device memory. */
static bool is_estimated(const CompressArgs& a) { return a.d_table != nullptr && a.table_stride == 0u; }

/*
 * Groups of a tile and waves that share it in the chained form.  Small launches take small tiles, which fill more of the chip; in larger ones
 * every round of workgroups ends with a wait, which larger tiles make fewer of.  us, 16 groups and 16 waves / 16 and 8 / 32 and 8 / 32 and
 * 16, equal chunks: bf16 2^20 4.3 / 4.3 / 5.2 / 5.0, 2^22 6.1 / 5.6 / 6.0 / 5.6, 2^23 10.6 / 8.1 / 7.5 / 7.3, 2^24 19.8 / 14.6 / 13.0 / 14.1, 2^26 80 / 57 /
 * 43 / 50; fp32 2^20 4.8 / 5.0 / 6.6 / 6.1, 2^22 8.6 / 7.4 / 8.1 / 7.4, 2^23 15.3 / 13.5 / 12.9 / 13.5, 2^24 26.8 / 24.7 / 26.4 / 24.7, 2^27 219 /
 * 193 / 170 / 161.  (64 groups and 16 waves: bf16 2^23 7.5, 2^24 12.9, 2^26 43.5, 64 chunks of 2^23 286, one of 2^29 297; fp32 2^24 25.4, 2^27 167.)
 *
 * A table for the whole tensor in device memory is most often the robust estimate's, which has read the tensor just now, and what the
 * caches hold of it comes so quickly that small tiles last longer: up to the sizes at which they stop doing so.  us, 8 equal chunks (one and
 * 64 much the same), estimate and compress, with a stash / 16 groups and 8 waves / 32 groups.  Behind the robust one, three tensors in turn: bf16 2^23 22.1 /
 * 19.9 / 20.8, 2^24 27.0 / 26.1 / 26.8, 18 * 2^20 28.5 / 27.2 / 28.8, 18.5 * 2^20 30.2 / 30.7 / 30.1, 20 * 2^20 30.3 / 34.0 / 30.0, 2^25 40.1 / 47.3 / 41.0,
 * 2^26 71.6 / 79.8 / 72.5 (one chunk 75.8 / 87.4 / 71.9); fp32 2^23 24.8 / 21.8 / 25.4, 2^24 39.9 / 38.5 / 39.7, 17 * 2^20 46.0 / 45.9 / 45.2.  The same with more
 * tensors than the caches hold: bf16 2^23 24.3 / 21.7 / 20.6, 2^24 29.7 / 28.4 / 27.0, 2^25 40.3 / 47.6 / 40.7; fp32 2^23 26.3 / 23.4 / 25.7.  Others pay for the
 * rule between 10 * 2^20 and its limit.  Standard deviation and compress: bf16 10 * 2^20 22.2 / 20.4 / 19.8, 2^24 27.0 / 26.1 / 24.1; fp32 2^24 41.5 / 39.5 /
 * 38.4.  A table kept from earlier, and the tensor in the caches: bf16 10 * 2^20 13.0 / 9.9 / 9.9, 2^24 16.4 / 14.6 / 13.4; not there, 14.2 / 12.1 / 10.5 and
 * 17.5 / 16.9 / 14.0; fp32 2^24 27.3 / 26.2 / 24.8.
 */
template <int DT>
static void launch_chained_dt(const CompressArgs& a, hipStream_t s)
{
    const CompressIo io = io_of(a);
    const uint32_t tiles = a.tab.tile_start[a.tab.n_chunks];
    const Chain chain = {a.words, launch_tag(), DT == ZIPCCL_BF16 && tiles > kManyTiles};
    auto launch = [&](auto waves, auto groups, const auto& split) {
        constexpr uint32_t W = decltype(waves)::value, G = decltype(groups)::value, per = G / kGroupsPerTile;
        using SPLIT = std::decay_t<decltype(split)>;
        const dim3 grid((max_chunk_tiles(a.tab) + per - 1u) / per, a.tab.n_chunks);
        hipLaunchKernelGGL((k_compress<DT, kModeChained, W, G, Chain, SPLIT>), grid, dim3(64u * W), 0, s, io, chain, split);
    };
    auto by_size = [&](const auto& split) {
        constexpr std::integral_constant<uint32_t, 8> c8;
        constexpr std::integral_constant<uint32_t, 16> c16;
        constexpr std::integral_constant<uint32_t, 32> c32;
        if (tiles <= kWideTiles) launch(c16, c16, split);
        else if (tiles <= (is_estimated(a) ? kSmallTilesEstimated<DT> : kSmallTiles)) launch(c8, c16, split);
        else if constexpr (DT == ZIPCCL_FP32) launch(c16, c32, split);
        else launch(c8, c32, split);
    };
    if (is_equal_split(a.tab)) by_size(equal_split(a.tab));
    else if (is_few_split(a.tab)) by_size(few_split(a.tab));
    else by_size(a.tab);
}

/* Not taken where it does not pay, nor for a stream that is being captured: a launch that a graph replays has the same tag every time. */
int launch_compress_chained(int dt, const CompressArgs& a, void* stream)
{
    if (!chained_pays(a, dt)) return kNotTaken;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing((hipStream_t)stream, &capture) != hipSuccess) {
        (void)hipGetLastError();                             /* of this question; the launches in its stead report their own */
        return kNotTaken;
    }
    if (capture != hipStreamCaptureStatusNone) return kNotTaken;
    if (dt == ZIPCCL_BF16) launch_chained_dt<ZIPCCL_BF16>(a, (hipStream_t)stream);
    else launch_chained_dt<ZIPCCL_FP32>(a, (hipStream_t)stream);
    return (int)hipGetLastError();
}

int launch_compress(int dt, int mode, const CompressArgs& a, void* stream)
{
    if (dt == ZIPCCL_BF16) launch_compress_dt<ZIPCCL_BF16>(mode, a, (hipStream_t)stream);
    else launch_compress_dt<ZIPCCL_FP32>(mode, a, (hipStream_t)stream);
    return (int)hipGetLastError();
}

int launch_tile_scan(const CompressArgs& a, void* stream)
{
    const dim3 grid((max_chunk_tiles(a.tab) + kScanSeg - 1) / kScanSeg, a.tab.n_chunks);
    hipLaunchKernelGGL(k_tile_scan, grid, dim3(kThreads), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

template <int DT>
static void launch_place_dt(bool scan, const CompressArgs& a, hipStream_t s)
{
    const dim3 grid((max_chunk_tiles(a.tab) + 15) / 16, a.tab.n_chunks), block(kThreads);   /* 16 tiles per workgroup */
    const CompressIo io = io_of(a);
    const Parking park = parking_of(a);
    if (!scan) hipLaunchKernelGGL((k_place<DT, false, ChunkTab>), grid, block, 0, s, io, park, a.tab);
    else if (is_equal_split(a.tab)) hipLaunchKernelGGL((k_place<DT, true, EqualSplit>), grid, block, 0, s, io, park, equal_split(a.tab));
    else hipLaunchKernelGGL((k_place<DT, true, ChunkTab>), grid, block, 0, s, io, park, a.tab);
}

int launch_place(int dt, bool scan, const CompressArgs& a, void* stream)
{
    if (dt == ZIPCCL_BF16) launch_place_dt<ZIPCCL_BF16>(scan, a, (hipStream_t)stream);
    else launch_place_dt<ZIPCCL_FP32>(scan, a, (hipStream_t)stream);
    return (int)hipGetLastError();
}

} // namespace zipccl
