/*
 * Decompress side of libzipccl.so for gfx950 (CDNA4, wave64): k_decompress (paper section 4, third
 * paragraph) and k_decompress_reduce (decode + local FP32 reduction of the zipped Reduce-Scatter,
 * sections 3.3 and 5.2).  No workgroup depends on another.  Work decomposition as on the compress side:
 * a wave owns a group of 512 values at a time, 8 values per lane (consecutive ones; k_decompress, fp32:
 * two quads, one from each half of the group, so that every tensor access is 16 contiguous bytes per
 * lane; the bf16 reduction of large shards: two groups, 16 values per lane); decoding is SWAR on packed bytes (table-driven bit spread, v_perm_b32 / v_bfi_b32
 * recombination) with a DPP wave scan to locate each lane's zero-point exponents.
 */
#include <type_traits>

#include "zipccl_device.h"

namespace zipccl {
namespace {

/*
 * Entry of the 4-bit stage of the expand table, for a zero-point mask q of four values:
 * .x = v_perm selector putting the r-th byte of a compacted list at the position of the r-th
 * set bit of q (0x0c = constant 0 elsewhere), .y = 0xff in the bytes of set bits.
 */
__device__ __forceinline__ uint2 expand_entry(uint32_t q)
{
    uint32_t sel = 0, msk = 0, r = 0;
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
        if ((q >> i) & 1u) { sel |= r << (8 * i); msk |= 0xFFu << (8 * i); ++r; }
        else sel |= 0x0Cu << (8 * i);
    }
    return make_uint2(sel, msk);
}

/* bits 0..3 of x -> bit 0 of bytes 0..3 */
__device__ __forceinline__ uint32_t spread4(uint32_t x)
{
    return __umul24(x, 0x204081u) & 0x01010101u;
}

/*
 * Decoder tables in LDS, built once per workgroup (one entry of each per thread):
 * spread[k][b]  = the 8 bits of plane byte b at bit k of 8 bytes (.x = values 0..3, .y = values 4..7),
 *                 so that the three planes of a lane combine with one OR;
 * expand[m]     = for the lane's 8-bit zero-point mask m: v_perm selectors (.x for values 0..3, .y for
 *                 values 4..7) that put the r-th byte of the lane's 8-byte list window at the position
 *                 of the r-th set bit of m, and the byte masks of the set bits (.z, .w).
 */
struct DecTables {
    uint2 spread[3][256];
    u32x4 expand[256];
    uint2 expand4[16];   /* building block of expand[] */
};

/* Contains a workgroup barrier; the caller's next barrier makes the tables visible.  The first 256 threads of the
 * workgroup's build them. */
template <uint32_t THREADS = kThreads>
__device__ __forceinline__ void build_tables(DecTables& t)
{
    const uint32_t b = threadIdx.x;
    const bool mine = THREADS == 256u || b < 256u;
    if (b < 16) t.expand4[b] = expand_entry(b);
    if (mine) {
        const uint32_t lo = spread4(b & 15u), hi = spread4(b >> 4);
        t.spread[0][b] = make_uint2(lo, hi);
        t.spread[1][b] = make_uint2(lo << 1, hi << 1);
        t.spread[2][b] = make_uint2(lo << 2, hi << 2);
    }
    __syncthreads();
    if (mine) {
        /* values 4..7 continue in the window where values 0..3 stopped */
        const uint2 a = t.expand4[b & 15u], c = t.expand4[b >> 4];
        const uint32_t skip = __popc(b & 15u) * 0x01010101u;
        t.expand[b] = u32x4{a.x, c.x + (skip & c.y), a.y, c.y};
    }
}

/* Bytes of LDS per group for its zero-point exponents: 512 + up to 15 of misalignment, rounded up to
 * whole 16-byte words (33 of them) + 16 so that a lane's three aligned words never leave the region. */
constexpr uint32_t kEscRegion = 544;
constexpr uint32_t kListLanes = 33;     /* lanes that fetch 16 bytes of the list each */

/* What a lane reads for its 8 values of one group. */
struct DecIn {
    uint32_t sm0, sm1;       /* 8 sign+mantissa bytes */
    uint32_t b0, b1, b2;     /* plane bytes */
    uint32_t lo[4];          /* fp32: 8 low 16-bit words */
    uint32_t base;           /* IDX entry of the group = list position of its first zero-point */
    uint32_t count;          /* zero-points of the group according to IDX (next entry - this one) */
    uint32_t vmask;          /* bit j = value j exists */
    uint32_t idx_bad;        /* slice_bad of the group's entry and the next */
};

/* The lane's zero-point bytes (up to 8, in element order) and where its mask says they go. */
struct DecEsc {
    uint32_t m;              /* bit j = value j is a zero-point */
    uint32_t l8, h8;         /* the 8 list bytes from the lane's first zero-point on */
    uint32_t wA, wB;         /* two-quad lanes (fp32): the list bytes of the first and of the second quad */
    uint32_t bad;            /* nonzero: planes and IDX disagree about the group */
};

/* r.base and next bound the group's slice of the zero-point list: check them, set r.count.  That the first two entries
 * of a chunk ascend is checked elsewhere, once. */
__device__ __forceinline__ void check_index(DecIn& r, uint32_t next, uint32_t n_esc)
{
    r.idx_bad = slice_bad(r.base, next, n_esc, false);
    r.count = r.idx_bad ? 0u : next - r.base;
}

/* Phase 1a: fetch the slice [base, base + count): 16 aligned bytes per lane by the first 33 lanes, which
 * covers 512 bytes at any alignment.  Aligned reads stay inside pad128(n_esc); lanes past the slice read
 * the 16 bytes in front of the list instead (the end of the static part), so the load needs no predicate
 * and every group issues the same number of loads. */
__device__ __forceinline__ void decode_fetch_list(const uint8_t* __restrict__ slot, const SlotLayout& L,
                                                  const DecIn& r, uint32_t next, uint32_t lane, u32x4& v)
{
    const uint32_t end = r.count != 0u ? next : 0u;              /* nothing to fetch for an empty slice */
    const uint32_t a = (r.base & ~15u) + 16u * lane;
    const uint8_t* __restrict__ esc = slot + L.esc;
    v = *reinterpret_cast<const u32x4*>(esc + (a < end ? (int64_t)a : (int64_t)-16));
}

/* Which of the lane's 8 values of the group at gs exist (bit j = value j): bf16: 8 consecutive ones; fp32: two quads,
 * [4 lane, 4 lane + 4) of the group's first half and of its second. */
template <int DT>
__device__ __forceinline__ uint32_t value_mask(uint64_t n, uint64_t gs, uint32_t lane)
{
    const uint32_t left = gs >= n ? 0u : (uint32_t)min(n - gs, (uint64_t)kGroup);      /* values of the group */
    if (DT == ZIPCCL_BF16) {
        const uint32_t e = lane * kLaneElems;
        return e >= left ? 0u : (1u << min(left - e, 8u)) - 1u;
    }
    const uint32_t a = lane * 4u, b = a + kGroup / 2;
    return (a >= left ? 0u : (1u << min(left - a, 4u)) - 1u) | ((b >= left ? 0u : (1u << min(left - b, 4u)) - 1u) << 4);
}

/*
 * Phase 1b: the lane's SM bytes, plane bytes and (fp32) low words.  Every output row of 1 KiB is 16 contiguous bytes per
 * lane, so fp32 lanes hold two quads (value_mask).  FAST: a whole group.  Otherwise lanes without values read the
 * first bytes of the group's part of the section instead, and a group past the end reads group 0's (the chunk is not
 * empty): no load is under a condition, so all groups' loads are in flight together.  The planes of a group that has
 * any value are there as a whole.
 */
template <int DT, bool FAST, bool STREAM = true>
__device__ __forceinline__ void decode_load(const uint8_t* __restrict__ slot, const SlotLayout& L, uint64_t n,
                                            uint64_t gstart, uint32_t lane, DecIn& r)
{
    r.vmask = FAST ? 0xFFu : value_mask<DT>(n, gstart, lane);
    const uint64_t gs = FAST || gstart < n ? gstart : 0u;
    /* wave-uniform 64-bit bases + 32-bit lane offsets */
    const uint8_t* __restrict__ sm = slot + L.sm + gs;
    const uint8_t* __restrict__ pl = slot + L.p0 + (gs >> 3);     /* 64-byte aligned: a group's 64 plane bytes */
    /* fp32: the lane fetches one plane byte per plane, the one it shares with its neighbour: even lanes that of the
       first half, odd lanes that of the second (quad_plane_bytes sorts the nibbles out) */
    const uint32_t pi = DT == ZIPCCL_BF16 ? lane : (lane >> 1) + 32u * (lane & 1u);
    const uint32_t ia = FAST || (r.vmask & 15u) ? lane * 4u : 0u, ib = FAST || (r.vmask >> 4) ? kGroup / 2 + lane * 4u : 0u;
    if (DT == ZIPCCL_BF16) {
        const u32x2 v = ld_as<STREAM, u32x2>(sm + (FAST || r.vmask ? lane * 8u : 0u));
        r.sm0 = v.x; r.sm1 = v.y;
    } else {
        r.sm0 = ld_as<STREAM, uint32_t>(sm + ia);
        r.sm1 = ld_as<STREAM, uint32_t>(sm + ib);
    }
    /* the planes before the low words: they are wanted first, and loads are waited for in order */
    r.b0 = ld_as<STREAM, uint8_t>(pl + pi);
    r.b1 = ld_as<STREAM, uint8_t>((pl + L.plane_bytes) + pi);
    r.b2 = ld_as<STREAM, uint8_t>((pl + 2 * L.plane_bytes) + pi);
    r.lo[0] = r.lo[1] = r.lo[2] = r.lo[3] = 0;
    if (DT == ZIPCCL_FP32) {
        const uint8_t* __restrict__ lo = slot + L.lo + 2 * gs;
        const u32x2 la = ld_as<STREAM, u32x2>(lo + 2u * ia);
        const u32x2 lb = ld_as<STREAM, u32x2>(lo + 2u * ib);
        r.lo[0] = la.x; r.lo[1] = la.y; r.lo[2] = lb.x; r.lo[3] = lb.y;
    }
}

/* After decode_load of fp32: from the plane bytes shared by a pair of lanes to each lane's own
 * byte (bits 0..3 = its first quad, bits 4..7 = its second), the three planes at once. */
__device__ __forceinline__ void quad_plane_bytes(DecIn& r, uint32_t lane)
{
    const uint32_t p3 = (r.b0 & 0xFFu) | ((r.b1 & 0xFFu) << 8) | ((r.b2 & 0xFFu) << 16);
    const uint32_t q3 = __builtin_amdgcn_update_dpp(0u, p3, 0xB1, 0xF, 0xF, false);   /* quad_perm [1,0,3,2] */
    const uint32_t b3 = (lane & 1u) ? (((q3 >> 4) & 0x0F0F0Fu) | (p3 & 0xF0F0F0u))
                                    : ((p3 & 0x0F0F0Fu) | ((q3 & 0x0F0F0Fu) << 4));
    r.b0 = b3 & 0xFFu;
    r.b1 = (b3 >> 8) & 0xFFu;
    r.b2 = b3 >> 16;
}

/* Phase 1c: park the slice in the wave's LDS region so that lanes can pick their bytes by position. */
__device__ __forceinline__ void decode_park_list(uint8_t* lds, uint32_t lane, const u32x4& v)
{
    if (lane < kListLanes) *reinterpret_cast<u32x4*>(lds + 16u * lane) = v;
}

/* Phase 2: wave scan of the per-lane zero-point counts, then the lane's bytes from the LDS region.
 * Straight-line code (no branch on whether the group has zero-points) so that the four groups a
 * wave works on can be interleaved by the scheduler. */
__device__ __forceinline__ DecEsc decode_locate(const DecIn& in, const uint8_t* lds)
{
    DecEsc r;
    r.m = ((in.b0 | in.b1 | in.b2) ^ 0xFFu) & in.vmask;     /* code 0 = zero-point; tail bits are not */
    const uint32_t cnt = __popc(r.m);
    const uint32_t inc = wave_incl_scan(cnt);
    const uint32_t gtot = __builtin_amdgcn_readlane(inc, 63);
    r.bad = in.idx_bad | (gtot ^ in.count);   /* planes and IDX must agree */
    /* the lane's zero-point exponents are the bytes [p, p + cnt) of the region, p <= 15 + 512 - cnt
       (clamped, so that a corrupt stream still reads inside the region) */
    const uint32_t p = min((in.base & 15u) + (inc - cnt), kGroup + 15u);
    /* three aligned words and two byte alignments: a single 8-byte read at the byte address p is accepted by the
       hardware but made the fused reduce, whose LDS pipe is two thirds busy, 35 % slower (measured) */
    const uint32_t* w = reinterpret_cast<const uint32_t*>(lds + (p & ~3u));
    r.l8 = __builtin_amdgcn_alignbyte(w[1], w[0], p & 3u);
    r.h8 = __builtin_amdgcn_alignbyte(w[2], w[1], p & 3u);
    return r;
}

/* Phase 2 for two-quad lanes: element order is all first quads by lane, then all second quads, so the
 * lane's zero-points sit in two places of the slice; one scan carries both counts. */
__device__ __forceinline__ DecEsc decode_locate_quad(const DecIn& in, const uint8_t* lds)
{
    DecEsc r;
    r.m = ((in.b0 | in.b1 | in.b2) ^ 0xFFu) & in.vmask;
    const uint32_t cA = __popc(r.m & 15u), cB = __popc(r.m >> 4);
    const uint32_t inc = wave_incl_scan(cA | (cB << 16));
    const uint32_t tot = __builtin_amdgcn_readlane(inc, 63);
    const uint32_t totA = tot & 0xFFFFu;
    r.bad = in.idx_bad | ((totA + (tot >> 16)) ^ in.count);
    const uint32_t pA = min((in.base & 15u) + (inc & 0xFFFFu) - cA, kGroup + 15u);
    const uint32_t pB = min((in.base & 15u) + totA + (inc >> 16) - cB, kGroup + 15u);
    const uint32_t* wa = reinterpret_cast<const uint32_t*>(lds + (pA & ~3u));
    const uint32_t* wb = reinterpret_cast<const uint32_t*>(lds + (pB & ~3u));
    r.wA = __builtin_amdgcn_alignbyte(wa[1], wa[0], pA & 3u);
    r.wB = __builtin_amdgcn_alignbyte(wb[1], wb[0], pB & 3u);
    r.l8 = r.h8 = 0;
    return r;
}

/* Rebuild the bytes of the high 16-bit words of the lane's 8 values (section 4, third paragraph):
 * lA / hA = low / high bytes of values 0..3, lB / hB of values 4..7. */
template <bool QUAD = false>
__device__ __forceinline__ void decode_bytes(const DecIn& in, const DecEsc& es, uint32_t e0, const DecTables& tab,
                                             uint32_t& lA, uint32_t& hA, uint32_t& lB, uint32_t& hB)
{
    /* code bytes of values 0..3 and 4..7 (plane bits spread by table), then exponent = dec[1] - 1 + code */
    const uint32_t k4 = (e0 - 1u) * 0x01010101u;
    const uint2 t0 = tab.spread[0][in.b0], t1 = tab.spread[1][in.b1], t2 = tab.spread[2][in.b2];
    uint32_t eA = (t0.x | t1.x | t2.x) + k4;
    uint32_t eB = (t0.y | t1.y | t2.y) + k4;
    if (QUAD) {   /* each quad's zero-point exponents from its own window */
        const uint2 xa = tab.expand4[es.m & 15u], xb = tab.expand4[es.m >> 4];
        eA = bfi(xa.y, perm(0u, es.wA, xa.x), eA);
        eB = bfi(xb.y, perm(0u, es.wB, xb.x), eB);
    } else {   /* zero-point exponents dropped in place: the lane's list bytes are the 8-byte window l8:h8 */
        const u32x4 x = tab.expand[es.m];
        eA = bfi(x.z, perm(es.h8, es.l8, x.x), eA);
        eB = bfi(x.w, perm(es.h8, es.l8, x.y), eB);
    }
    /* recombine with sign and mantissa: low byte = mantissa | E bit 0 << 7, high = sign | E >> 1 */
    lA = bfi(0x7F7F7F7Fu, in.sm0, eA << 7); hA = bfi(0x80808080u, in.sm0, eA >> 1);
    lB = bfi(0x7F7F7F7Fu, in.sm1, eB << 7); hB = bfi(0x80808080u, in.sm1, eB >> 1);
}

/* The same as four words holding the 8 high 16-bit words in element order. */
template <bool QUAD = false>
__device__ __forceinline__ void decode_values(const DecIn& in, const DecEsc& es, uint32_t e0,
                                              const DecTables& tab, uint32_t hp[4])
{
    uint32_t lA, hA, lB, hB;
    decode_bytes<QUAD>(in, es, e0, tab, lA, hA, lB, hB);
    hp[0] = perm(hA, lA, 0x05010400u);
    hp[1] = perm(hA, lA, 0x07030602u);
    hp[2] = perm(hB, lB, 0x05010400u);
    hp[3] = perm(hB, lB, 0x07030602u);
}

/* Rebuild the lane's 8 values as they are stored, 16 bytes per row of 1 KiB: bf16: one row; fp32: one of the group's
 * first half and one of its second. */
template <int DT>
__device__ __forceinline__ void decode_rows(const DecIn& in, const DecEsc& es, uint32_t e0, const DecTables& tab,
                                            u32x4 row[DT == ZIPCCL_BF16 ? 1 : 2])
{
    uint32_t hp[4];
    decode_values<DT == ZIPCCL_FP32>(in, es, e0, tab, hp);
    if (DT == ZIPCCL_BF16) {
        row[0] = u32x4{hp[0], hp[1], hp[2], hp[3]};
    } else {
        uint32_t x[8];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            x[2 * k] = perm(hp[k], in.lo[k], 0x05040100u);
            x[2 * k + 1] = perm(hp[k], in.lo[k], 0x07060302u);
        }
        row[0] = u32x4{x[0], x[1], x[2], x[3]};
        row[DT == ZIPCCL_BF16 ? 0 : 1] = u32x4{x[4], x[5], x[6], x[7]};
    }
}

/* The first `count` values of a lane's 16 bytes, at most three pieces of 8, 4 and 2 bytes if not all (value by value, the
 * code alone was a good part of a small launch).  A chunk of a single tile is not streamed: it shares its cache lines with
 * the chunks next to it, which other workgroups write, and streamed, each piece of a line goes to memory by itself (128
 * chunks of 8 bf16 values 3.4 us, 2.9 with plain stores; of 100 fp32 values 3.5 and 3.3).  Behind other tiles a rest is
 * streamed like them: what plain stores leave in the caches is written out when the kernel ends (128 chunks of 65 531 fp32
 * values 13.4 us, 14.7 with plain stores). */
template <int DT>
__device__ __forceinline__ void store_first(uint8_t* p, const u32x4& v, uint32_t count, bool stream)
{
    constexpr uint32_t N = DT == ZIPCCL_BF16 ? 8u : 4u;
    if (count == N) {
        if (stream) {
            /* the two empty statements keep the compiler from making one store, a plain one, of the two */
            asm volatile("");
            st_stream_a2(p, v);
            asm volatile("");
        } else {
            *reinterpret_cast<u32x4_a2*>(p) = v;
        }
    } else {
        uint32_t w0 = v.x, w1 = v.y;
        if (count & (N / 2u)) {
            *reinterpret_cast<u32x2_a2*>(p) = u32x2{w0, w1};
            p += 8; w0 = v.z; w1 = v.w;
        }
        if (count & (N / 4u)) {
            *reinterpret_cast<u32_a2*>(p) = w0;
            p += 4; w0 = w1;
        }
        if (DT == ZIPCCL_BF16 && (count & 1u)) *reinterpret_cast<uint16_t*>(p) = (uint16_t)w0;
    }
}

/*
 * Chunk header check (all wave-uniform): the static part is readable (the host checked it), magic,
 * version, dtype, G and n must match the call, the table must be a window (dec[0] = 0, dec[1..7]
 * consecutive), and the zero-point list the header promises must fit into the readable bytes.  The
 * reserved bytes 48..127 are not looked at.
 */
struct HeaderWords { uint32_t h[12]; };

/* All twelve words are fetched before any is looked at (one round of scalar loads, no chain of
 * dependent ones); a kernel can request them early and look at them later. */
__device__ __forceinline__ HeaderWords load_header(const uint8_t* __restrict__ slot)
{
    const uint32_t* hw = reinterpret_cast<const uint32_t*>(slot);
    HeaderWords r;
#pragma unroll
    for (int i = 0; i < 12; ++i) r.h[i] = hw[i];
    return r;
}

template <int DT>
__device__ __forceinline__ bool check_header(const HeaderWords& hdr, const SlotLayout& L, uint64_t n,
                                             uint64_t slot_off, uint64_t comp_capacity, uint32_t& e0, uint32_t& n_esc)
{
    const uint32_t* h = hdr.h;
    const uint64_t n_hdr = (uint64_t)h[4] | ((uint64_t)h[5] << 32);
    const uint64_t ne = (uint64_t)h[6] | ((uint64_t)h[7] << 32);
    const uint64_t cbytes = (uint64_t)h[8] | ((uint64_t)h[9] << 32);
    const uint32_t dec_lo = h[10], dec_hi = h[11];
    e0 = (dec_lo >> 8) & 0xFFu;
    n_esc = (uint32_t)ne;
    uint32_t wrong = (h[0] ^ kMagic) | (h[1] ^ kVersion) | (h[2] ^ (uint32_t)DT) | (h[3] ^ kGroup);
    wrong |= (uint32_t)(n_hdr != n) | (uint32_t)(ne > n) | (uint32_t)(cbytes != L.esc + pad128(ne));
    wrong |= (uint32_t)(slot_off + cbytes > comp_capacity);
    wrong |= (uint32_t)(e0 < 1u) | (uint32_t)(e0 > 249u);
    wrong |= dec_lo & 0xFFu;                                   /* dec[0] is written as 0 */
    wrong |= (dec_lo >> 8) ^ (e0 | ((e0 + 1u) << 8) | ((e0 + 2u) << 16));
    wrong |= dec_hi ^ ((e0 + 3u) | ((e0 + 4u) << 8) | ((e0 + 5u) << 16) | ((e0 + 6u) << 24));
    const bool ok = wrong == 0u;
    return ok;
}

/* Kernel arguments: DecompressArgs without its table, which follows in the form that the launch allows (see EqualSplit). */
struct DecompressIo {
    const uint8_t* comp;
    uint64_t comp_capacity;
    uint8_t* out;
    uint32_t* status;
};

/* GPW (1, 2 or 4) groups per wave: a workgroup decodes a tile of 4 * GPW groups.  The compressed format does not know
 * tiles (groups are located through IDX alone), so this is free to differ from the compress side's tile. */
template <int DT, uint32_t GPW, bool STREAM, class SPLIT>
/* waves per SIMD: 8 (<= 64 VGPRs); launches with four fp32 groups per wave hold no more than 4 */
__global__ __launch_bounds__(kThreads, DT == ZIPCCL_FP32 && GPW == 4u ? 4 : 8)
void k_decompress(const DecompressIo a, const SPLIT split)
{
    constexpr uint32_t ES = DT == ZIPCCL_BF16 ? 2u : 4u;
    constexpr uint32_t TILE = kGroup * kWavesPerBlock * GPW;
    __shared__ DecTables s_tab;
    __shared__ __attribute__((aligned(16))) uint8_t s_esc[kWavesPerBlock][GPW][kEscRegion];

    /* grid = (tiles of the largest chunk, chunks) */
    const uint32_t c = blockIdx.y;
    const ChunkPlace place = place_of(split, c, DT);
    const uint64_t n = place.n;
    const uint32_t tiles = n == 0 ? 1u : (uint32_t)((n + TILE - 1) / TILE);    /* an empty chunk still has its header checked */
    if (blockIdx.x >= tiles) return;
    const uint64_t ts = (uint64_t)blockIdx.x * TILE;
    const uint8_t* __restrict__ slot = a.comp + place.slot_off;
    uint8_t* __restrict__ cout = a.out + place.elem_off * ES;
    const SlotLayout L = slot_layout(n, DT);
    /* whole tiles need no masks */
    const bool fast = ts + TILE <= n;
    const uint32_t lane = lane_id();
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   /* scalar: group addresses and index entries stay out of the vector registers */
    const uint32_t ng = (uint32_t)((n + kGroup - 1) / kGroup);                /* at most 2^23 */
    /* A chunk of the tensor starts at some element of it, so that rows of 1 KiB may share cache lines with their
       neighbours.  One or two groups per wave are neighbours: the pieces of a shared line come from one wave, one after
       the other (from two waves of a tile, each half a line at its own time, they took twice as long: 64 chunks of
       262 139 values, bf16 29.1 -> 12.4 us, fp32 49.1 -> 23.5; 11.5 and 22.9 on line boundaries).  Four groups per
       wave, for chunks on line boundaries only, are four apart, which shares a short tile evenly among the waves
       (2^24 bf16 values: 11.7 us, 12.1 with neighbours). */
    constexpr bool NEIGHBOURS = GPW <= 2u;
    constexpr uint32_t step = NEIGHBOURS ? 1u : kWavesPerBlock;
    const uint32_t g0 = (uint32_t)(ts / kGroup) + (NEIGHBOURS ? wave * GPW : wave);
    const uint64_t gs0 = (uint64_t)g0 * kGroup;

    /* What does not depend on the header or on IDX goes out first (the static part is readable: the host
       checked it): SM, planes and low words of the wave's groups, and the groups' index entries.
       The table build and the header check run while these loads are in flight. */
    const HeaderWords hdr = load_header(slot);
    DecIn in[GPW];
    uint32_t next[GPW];
    if (n != 0) {
        const uint32_t* __restrict__ idx = reinterpret_cast<const uint32_t*>(slot + L.idx);
        if (fast) {
#pragma unroll
            for (uint32_t u = 0; u < GPW; ++u) decode_load<DT, true, STREAM>(slot, L, n, gs0 + (uint64_t)(u * step) * kGroup, lane, in[u]);
        } else {
#pragma unroll
            for (uint32_t u = 0; u < GPW; ++u) decode_load<DT, false, STREAM>(slot, L, n, gs0 + (uint64_t)(u * step) * kGroup, lane, in[u]);
        }
#pragma unroll
        for (uint32_t u = 0; u < GPW; ++u) {
            const uint32_t g = g0 + u * step;
            in[u].base = idx[min(g, ng - 1)];
            next[u] = idx[min(g + 1, ng - 1)];
        }
    }
    build_tables(s_tab);

    uint32_t e0, n_esc;
    const bool ok = check_header<DT>(hdr, L, n, place.slot_off, a.comp_capacity, e0, n_esc);
    __syncthreads();
    if (!ok) {
        if (threadIdx.x == 0 && a.status) atomicOr(a.status, (uint32_t)ZIPCCL_ERR_CORRUPT);
        return;
    }
    if (n == 0) return;

    uint32_t bad = 0;
    constexpr uint32_t ROWS = DT == ZIPCCL_BF16 ? 1u : 2u;
    uint8_t* __restrict__ dst = cout + gs0 * ES;
    DecEsc es[GPW];
    /* phases over the wave's groups, so that each phase's loads are all in flight together; a group past the end
       has an empty slice */
    auto locate = [&](auto whole_tile) {
        constexpr bool FAST = decltype(whole_tile)::value;
        u32x4 lv[GPW];
#pragma unroll
        for (uint32_t u = 0; u < GPW; ++u) {
            const uint32_t g = g0 + u * step;
            if (FAST) in[u].vmask = 0xFFu;
            else if (g >= ng) in[u].base = n_esc;
            if (g + 1 >= ng) next[u] = n_esc;
            check_index(in[u], next[u], n_esc);
        }
#pragma unroll
        for (uint32_t u = 0; u < GPW; ++u) decode_fetch_list(slot, L, in[u], next[u], lane, lv[u]);
#pragma unroll
        for (uint32_t u = 0; u < GPW; ++u) decode_park_list(s_esc[wave][u], lane, lv[u]);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (uint32_t u = 0; u < GPW; ++u) {
            if (DT == ZIPCCL_FP32) {
                quad_plane_bytes(in[u], lane);
                es[u] = decode_locate_quad(in[u], s_esc[wave][u]);
            } else {
                es[u] = decode_locate(in[u], s_esc[wave][u]);
            }
            bad |= es[u].bad;
        }
    };
    if (fast) {
        locate(std::true_type{});
#pragma unroll
        for (uint32_t u = 0; u < GPW; ++u) {
            u32x4 row[ROWS];
            decode_rows<DT>(in[u], es[u], e0, s_tab, row);
#pragma unroll
            for (uint32_t q = 0; q < ROWS; ++q) st_stream_a2((dst + (u * step * ROWS + q) * 1024u) + lane * 16u, row[q]);
        }
    } else {
        locate(std::false_type{});
        /* every row is finished before the first store: what is left of a row behind one waits for its low words, and
           such a wait includes the store */
        u32x4 row[GPW][ROWS];
#pragma unroll
        for (uint32_t u = 0; u < GPW; ++u) {
            if (gs0 + (uint64_t)u * step * kGroup >= n) break;
            decode_rows<DT>(in[u], es[u], e0, s_tab, row[u]);
#pragma unroll
            for (uint32_t q = 0; q < ROWS; ++q) asm volatile("" : "+v"(row[u][q]));
        }
#pragma unroll
        for (uint32_t u = 0; u < GPW; ++u) {
            if (gs0 + (uint64_t)u * step * kGroup >= n) break;
#pragma unroll
            for (uint32_t q = 0; q < ROWS; ++q)
                store_first<DT>((dst + (u * step * ROWS + q) * 1024u) + lane * 16u, row[u][q],
                                __popc(DT == ZIPCCL_BF16 ? in[u].vmask : (in[u].vmask >> (4u * q)) & 15u), tiles > 1u);
        }
    }
    /* here and not with the other checks, whose schedule it disturbs (235 * 10^6 bf16 values 127.4 -> 127.9 us) */
    if (g0 == 0u) bad |= slice_bad(in[0].base, next[0], n_esc, true);
    if (bad && a.status) atomicOr(a.status, (uint32_t)ZIPCCL_ERR_CORRUPT);
}

/* The bits a sum is stored as: a NaN sum becomes the one quiet NaN 0x7FC00000 (which payload and sign a NaN
 * result carries is left to the implementation by IEEE 754; this makes the output the same bits everywhere). */
__device__ __forceinline__ uint32_t sum_bits(float f)
{
    return f != f ? 0x7FC00000u : __float_as_uint(f);
}

/* fp32 bits (from sum_bits: no NaN other than 0x7FC00000, which this maps to 0x7FC0) -> bf16 bits, round to nearest even */
__device__ __forceinline__ uint32_t f32_bits_to_bf16_bits(uint32_t u)
{
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

/* A 32-bit load through the constant address space: for a wave-uniform address the compiler issues it
 * as a scalar load whatever stores the kernel contains.  Only for memory no kernel writes while this one
 * runs (the compressed input). */
__device__ __forceinline__ uint32_t load_const_u32(const uint8_t* p)
{
    typedef const uint32_t __attribute__((address_space(4))) * cptr;
    return *reinterpret_cast<cptr>(reinterpret_cast<uintptr_t>(p));
}

/*
 * A stage of the reduce pipeline = one peer's copy of one group.  The buffer holds the stage's loads in
 * flight and what describes it (cur_*), and, fetched ahead with scalar loads, the description and index
 * entries of the stage that uses the buffer next (pre_*).  Everything but the loaded words is wave-uniform.
 */
struct StageBuf {
    DecIn in;
    u32x4 lv;
    uint64_t pre_off;                 /* next stage: slot offset, */
    uint32_t pre_g;                   /* group, */
    uint32_t pre_base, pre_next;      /* the group's index entry and the following one, */
    uint32_t pre_nesc, pre_dec;       /* the slot's zero-point count and header word holding dec[0..3] */
    bool pre_last;                    /* and whether it is the last peer of its group */
    uint32_t cur_g, cur_e0;
    bool cur_last;
};

/*
 * Local reduction of the zipped Reduce-Scatter (paper sections 3.3 and 5.2): decode the slices
 * received from the peers (slots back to back, n values each) and sum them in FP32, peers in slot
 * order.  One pass: every compressed byte is read once and only the sum is written.
 *
 * A wave owns n_groups groups (gs0, gs0 + 2048, ...) and walks the stages (group, peer), peers
 * innermost, as one software pipeline that does not drain between groups: while stage k is decoded,
 * the loads of stage k + 1 are in flight and the index entries of stage k + 2 have been requested.
 * Every stage issues the same number of loads, so that a wait for the older ones never has to drain
 * the younger ones; past the last stage the look-ahead repeats the last stage's requests.
 * The sum starts at -0.0f, the identity of FP32 addition for everything that is not a NaN, and one
 * addition per accepted slot follows; a NaN sum is stored as 0x7FC00000 (sum_bits).
 */
template <int DT, int ODT, bool FAST>
__device__ __forceinline__ void reduce_stages(const ReduceArgs& a, const SlotLayout& L, uint64_t gs0, uint32_t n_groups,
                                              uint32_t n_acc, uint32_t lane, uint8_t* lds, const DecTables& tab,
                                              const uint32_t* s_peer, bool all_ok, uint32_t& bad)
{
    constexpr uint32_t OES = ODT == ZIPCCL_BF16 ? 2u : 4u;
    const uint64_t n = a.n;
    const uint32_t ng = (uint32_t)((n + kGroup - 1) / kGroup);     /* n < 2^32: group numbers fit 32 bits */
    const uint32_t T = n_acc * n_groups;
    float acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = -0.0f;

    /* the look-ahead front: describe its stage into r.pre_* (the slot's header was checked by the
       workgroup; zero-point count, table and index entries come by scalar loads), then advance.
       The index position moves along with the stage instead of being recomputed. */
    uint32_t jf = 0, adv_left = T - 1u;
    uint32_t gf = (uint32_t)(gs0 / kGroup);
    uint64_t idx_f = L.idx + 4u * (uint64_t)gf;                /* of IDX[gf] in a slot */
    uint32_t next_f = gf + 1u < ng ? 4u : 0u;                  /* from there to the following entry, if any */
    uint64_t off_f = 0;                                        /* all slots accepted: offset of slot jf */
    auto front = [&](StageBuf& r) {
        /* some slot rejected: the j-th accepted one is not slot j */
        r.pre_off = all_ok ? off_f : (uint64_t)__builtin_amdgcn_readfirstlane(s_peer[jf]) * a.slot_cap;
        const uint8_t* __restrict__ slot = a.comp + r.pre_off;
        r.pre_nesc = load_const_u32(slot + 24);
        r.pre_dec = load_const_u32(slot + 40);
        r.pre_g = gf;
        r.pre_last = jf + 1u == n_acc;
        r.pre_base = load_const_u32(slot + idx_f);
        r.pre_next = load_const_u32(slot + idx_f + next_f);
        if (adv_left != 0u) {
            --adv_left;
            ++jf;
            off_f += a.slot_cap;
            if (jf == n_acc) {
                jf = 0;
                off_f = 0;
                gf += kWavesPerBlock;
                idx_f += 4u * kWavesPerBlock;
                next_f = gf + 1u < ng ? 4u : 0u;
            }
        }
    };
    /* issue every vector load of the stage r.pre_* describes.  The lanes' offsets inside a slot
       (section + group + lane) are kept in vector registers and renewed when the group changes, so that
       a stage adds nothing but the slot's address.  FAST = false differs in them, in the mask of the lane's
       values that exist and in the stores: loads under a condition would be waited for one by one (a shard of
       1 000 003 values took 10.8 us with them, one of 2^20 without any 7.8). */
    uint32_t g_iss = 0xFFFFFFFFu;
    uint64_t v_sm = 0, v_pl = 0, v_lo = 0;
    auto issue = [&](StageBuf& r) {
        r.cur_g = r.pre_g; r.cur_e0 = (r.pre_dec >> 8) & 0xFFu; r.cur_last = r.pre_last;
        const uint8_t* __restrict__ slot = a.comp + r.pre_off;
        const uint32_t next = r.pre_g + 1u < ng ? r.pre_next : r.pre_nesc;
        r.in.base = r.pre_base;
        check_index(r.in, next, r.pre_nesc);
        if (!FAST || r.pre_g != g_iss) {
            g_iss = r.pre_g;
            const uint64_t gs = (uint64_t)g_iss * kGroup, e = gs + lane * kLaneElems;
            /* lanes past the end of the shard read the sections' first bytes instead; the planes of a group that
               has any value are there as a whole */
            const bool some = FAST || e < n;
            v_sm = L.sm + (some ? e : 0u);
            /* the group's 3 x 64 plane bytes in one load: lanes 0..15 fetch the words of plane 0,
               16..31 those of plane 1, 32..47 (and again 48..63) those of plane 2 */
            v_pl = L.p0 + (gs >> 3) + (lane & 15u) * 4u + (uint64_t)min(lane >> 4, 2u) * L.plane_bytes;
            v_lo = L.lo + (some ? 2 * e : 0u);
        }
        /* the list as in decode_fetch_list, relative to 16 bytes before it */
        const uint32_t end = r.in.count != 0u ? next : 0u;
        const uint32_t a16 = (r.in.base & ~15u) + 16u * lane;
        r.lv = *reinterpret_cast<const u32x4*>((slot + (L.esc - 16)) + (a16 < end ? a16 + 16u : 0u));
        const u32x2 sm = ld_stream<u32x2>(slot + v_sm);
        r.in.sm0 = sm.x; r.in.sm1 = sm.y;
        /* a plain load, not a streaming one: a group's 64 bytes of a plane are half a cache line, and the
           other half is the neighbouring group's, which another wave decodes at another time (streamed,
           such lines came from memory twice: 13 % more bytes fetched and 204 instead of 179 us for
           8 x 2^26 values) */
        r.in.b0 = *reinterpret_cast<const uint32_t*>(slot + v_pl);
        if (DT == ZIPCCL_FP32) {
            const u32x4 lo = ld_stream<u32x4>(slot + v_lo);
            r.in.lo[0] = lo.x; r.in.lo[1] = lo.y; r.in.lo[2] = lo.z; r.in.lo[3] = lo.w;
        }
    };
    /* decode the stage in r and add it; after a group's last peer the sums are stored */
    auto consume = [&](StageBuf& r) {
        /* nothing that uses the stage's loaded words may be scheduled before this point (among the loads
           of the next stage, where it would wait for them to land as well) */
        __builtin_amdgcn_sched_barrier(0);
        /* the word holding the lane's byte of plane k sits in lane 16 k + lane / 4 */
        r.in.vmask = 0xFFu;
        if (!FAST) {
            const uint64_t e = (uint64_t)r.cur_g * kGroup + lane * kLaneElems;
            r.in.vmask = e >= n ? 0u : (n - e >= kLaneElems ? 0xFFu : (1u << (uint32_t)(n - e)) - 1u);
        }
        const uint32_t w = r.in.b0, from = (lane >> 2) * 4u, sh = 8u * (lane & 3u);
        r.in.b0 = __builtin_amdgcn_ubfe(__builtin_amdgcn_ds_bpermute(from, w), sh, 8u);
        r.in.b1 = __builtin_amdgcn_ubfe(__builtin_amdgcn_ds_bpermute(from + 64u, w), sh, 8u);
        r.in.b2 = __builtin_amdgcn_ubfe(__builtin_amdgcn_ds_bpermute(from + 128u, w), sh, 8u);
        /* park the slice; the wave's region holds 64 x 16 bytes, so every lane writes what it fetched and the
           store needs no predicate (lanes past the slice hold bytes that no lane picks) */
        *reinterpret_cast<u32x4*>(lds + 16u * lane) = r.lv;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const DecEsc es = decode_locate(r.in, lds);
        __builtin_amdgcn_wave_barrier();
        bad |= es.bad;
        float x[8];
        if (DT == ZIPCCL_BF16) {
            uint32_t lA, hA, lB, hB;
            decode_bytes(r.in, es, r.cur_e0, tab, lA, hA, lB, hB);
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {    /* value j as FP32 bits: high byte, low byte, 16 zero bits */
                const uint32_t sel = ((4u + j) << 24) | (j << 16) | 0x0C0Cu;
                x[j] = __uint_as_float(perm(hA, lA, sel));
                x[4 + j] = __uint_as_float(perm(hB, lB, sel));
            }
        } else {
            uint32_t hp[4];
            decode_values(r.in, es, r.cur_e0, tab, hp);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                x[2 * k] = __uint_as_float(perm(hp[k], r.in.lo[k], 0x05040100u));
                x[2 * k + 1] = __uint_as_float(perm(hp[k], r.in.lo[k], 0x07060302u));
            }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] += x[j];
        if (r.cur_last) {
            uint8_t* __restrict__ og = a.out + (uint64_t)r.cur_g * kGroup * OES;
            if (FAST) {
                /* a NaN among the lane's sums is rare: one unordered compare per pair of sums finds out, and
                   only then are the eight looked at one by one (sum_bits) */
                const bool any_nan = (acc[0] != acc[0] || acc[1] != acc[1]) | (acc[2] != acc[2] || acc[3] != acc[3]) |
                                     (acc[4] != acc[4] || acc[5] != acc[5]) | (acc[6] != acc[6] || acc[7] != acc[7]);
                if (__builtin_expect(__ballot(any_nan) != 0ull, 0)) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) acc[j] = __uint_as_float(sum_bits(acc[j]));
                }
                if (ODT == ZIPCCL_FP32) {
                    /* The lane's 8 sums are 32 contiguous bytes, a pattern that stores slowly.  Once per
                       group they go through the wave's LDS region (free between decodes), half a group at
                       a time, and come back as 16 contiguous bytes per lane: two streaming stores of 1 KiB. */
                    const u32x4 lo4 = u32x4{__float_as_uint(acc[0]), __float_as_uint(acc[1]),
                                            __float_as_uint(acc[2]), __float_as_uint(acc[3])};
                    const u32x4 hi4 = u32x4{__float_as_uint(acc[4]), __float_as_uint(acc[5]),
                                            __float_as_uint(acc[6]), __float_as_uint(acc[7])};
                    u32x4 row[2];
#pragma unroll
                    for (uint32_t h = 0; h < 2; ++h) {
                        if ((lane >> 5) == h) {
                            *reinterpret_cast<u32x4*>(lds + (lane & 31u) * 32u) = lo4;
                            *reinterpret_cast<u32x4*>(lds + (lane & 31u) * 32u + 16u) = hi4;
                        }
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                        row[h] = *reinterpret_cast<const u32x4*>(lds + lane * 16u);
                        __builtin_amdgcn_wave_barrier();
                    }
                    st_stream_a4(og + lane * 16u, row[0]);
                    st_stream_a4((og + 2 * kGroup) + lane * 16u, row[1]);
                } else {
                    uint32_t o[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        o[k] = f32_bits_to_bf16_bits(__float_as_uint(acc[2 * k])) | (f32_bits_to_bf16_bits(__float_as_uint(acc[2 * k + 1])) << 16);
                    st_stream_a4(og + lane * 16u, u32x4{o[0], o[1], o[2], o[3]});
                }
            } else {
                /* the sums are finished here: sunk into the branches below, what is left of them waits for the stage's
                   low words there, and such a wait includes the store of the branch before (eight stores one after
                   the other: 200 003 fp32 values of two peers 4.7 -> 4.1 us) */
                asm volatile("" : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "+v"(acc[4]), "+v"(acc[5]), "+v"(acc[6]), "+v"(acc[7]));
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if ((r.in.vmask >> j) & 1u) {
                        const uint64_t i = lane * kLaneElems + j;
                        if (ODT == ZIPCCL_FP32) *reinterpret_cast<uint32_t*>(og + i * 4) = sum_bits(acc[j]);
                        else *reinterpret_cast<uint16_t*>(og + i * 2) = (uint16_t)f32_bits_to_bf16_bits(sum_bits(acc[j]));
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] = -0.0f;
        }
    };

    /* two buffers used in turn (a copy from one to the other would have to wait for the loads).
       front()'s scalar loads return out of order, so any wait for one of them (or for an LDS access)
       waits for all: a stage requests them first, then issues its vector loads with what the previous
       stage's requests brought (long complete: the LDS waits of its decode saw to that), then decodes. */
    StageBuf bufA, bufB;
    front(bufA);
    front(bufB);
    __builtin_amdgcn_s_waitcnt(0xC07F);  /* lgkmcnt(0): nothing pending when the loop is entered */
    issue(bufA);
    uint32_t k = 0;                      /* stage whose loads bufA holds */
    while (k + 2u < T) {                 /* two stages, each with a real stage to look ahead to */
        front(bufA);
        asm volatile("" ::: "memory");
        issue(bufB);
        consume(bufA);
        front(bufB);
        asm volatile("" ::: "memory");
        issue(bufA);
        consume(bufB);
        k += 2u;
    }
    if (k + 2u == T) {                   /* two stages left */
        issue(bufB);
        consume(bufA);
        consume(bufB);
    } else {
        consume(bufA);
    }
}

/* What a wave has in flight of one peer's copy of a pair of groups; everything but the loaded words is wave-uniform. */
struct PairBuf {
    u32x4 sm;                         /* 16 sign+mantissa bytes */
    uint32_t p0, p1, p2;              /* 16 code bits of each plane */
    u32x4 lv;
    const uint8_t* pre_slot;          /* next stage: its slot, */
    uint32_t pre_base, pre_mid, pre_next;    /* the index entries of the two groups and the following one, */
    uint32_t pre_nesc, pre_dec;       /* the slot's zero-point count and header word holding dec[0..3] */
    const uint8_t* list;              /* 16 bytes in front of the aligned start of the pair's slice of the list */
    PairSlices sl;
    uint32_t e0;
};

/* Bytes of LDS per wave: the slice of two groups at any alignment (1024 + 15) and the words a lane may read past
 * the last position it can be sent to; 2 KiB of sums on their way out. */
constexpr uint32_t kPairRegion = 2048;
static_assert(kPairRegion >= 2 * kGroup + 15 + 8 + 12, "a lane's words stay inside the region");

/*
 * The same for bf16 and whole tiles, two neighbouring groups (1024 values, 16 consecutive ones per lane) at a time and
 * one such pair per wave: a stage is a peer.  The kernel is bound by instruction issue, and much of a stage does not
 * depend on how many values a lane holds: one scan locates the zero-points of both groups (group a is lanes 0..31), one
 * fetch brings their slices, which are adjacent, and the walk over slots and index entries is paid once.  A lane's
 * plane bits are two bytes of a whole cache line per plane, loaded directly.  Addresses are scalar bases with the
 * lane's constant offset: the scalar unit has the room now that a stage is twice as large.
 * 8 x 2^25 bf16 -> FP32: 96.4 -> 84.6 us (6.1 TB/s of the 520 MB it cannot do without), 8 x 2^26: 187.6 -> 165.3.  More
 * than one pair per wave is slower (2^25: 89.0 with two, 102.7 with four; 2 peers: 40.0, 41.1, 45.5).
 */
template <int ODT>
__device__ __forceinline__ void reduce_pair(const ReduceArgs& a, const SlotLayout& L, uint64_t gs, uint32_t n_acc, uint32_t lane,
                                            uint8_t* lds, const DecTables& tab, const uint32_t* s_peer, bool all_ok, uint32_t& bad)
{
    constexpr uint32_t OES = ODT == ZIPCCL_BF16 ? 2u : 4u;
    const uint32_t ng = (uint32_t)((a.n + kGroup - 1) / kGroup), g = (uint32_t)(gs / kGroup);
    const bool last_pair = g + 2u >= ng;
    const uint64_t o_idx = L.idx + 4u * (uint64_t)g, o_sm = L.sm + gs, o_pl = L.p0 + (gs >> 3);      /* in a slot */
    const uint32_t lane16 = lane * 16u;
    float acc[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[j] = -0.0f;

    uint32_t jf = 0;
    const uint8_t* slot_f = a.comp;                            /* all slots accepted: slot jf */
    auto front = [&](PairBuf& r) {
        /* some slot rejected: the j-th accepted one is not slot j */
        r.pre_slot = all_ok ? slot_f : a.comp + (uint64_t)__builtin_amdgcn_readfirstlane(s_peer[jf]) * a.slot_cap;
        r.pre_nesc = load_const_u32(r.pre_slot + 24);
        r.pre_dec = load_const_u32(r.pre_slot + 40);
        r.pre_base = load_const_u32(r.pre_slot + o_idx);
        r.pre_mid = load_const_u32(r.pre_slot + o_idx + 4);
        r.pre_next = load_const_u32(r.pre_slot + o_idx + (last_pair ? 4u : 8u));
        if (jf + 1u < n_acc) {
            ++jf;
            slot_f += a.slot_cap;
        }
    };
    auto issue = [&](PairBuf& r) {
        r.e0 = (r.pre_dec >> 8) & 0xFFu;
        const uint32_t next = last_pair ? r.pre_nesc : r.pre_next;
        r.sl = pair_slices(r.pre_base, r.pre_mid, next, r.pre_nesc);
        r.list = r.pre_slot + (L.esc - 16u) + r.sl.from;
        r.lv = *reinterpret_cast<const u32x4*>(r.list + pair_list_offset(r.sl, lane));
        r.sm = ld_stream<u32x4>((r.pre_slot + o_sm) + lane16);
        const uint8_t* const pl = r.pre_slot + o_pl;
        r.p0 = ld_stream<uint16_t>(pl + 2u * lane);
        r.p1 = ld_stream<uint16_t>((pl + L.plane_bytes) + 2u * lane);
        r.p2 = ld_stream<uint16_t>((pl + 2u * L.plane_bytes) + 2u * lane);
    };
    auto consume = [&](PairBuf& r) {
        /* nothing that uses the stage's loaded words may be scheduled before this point */
        __builtin_amdgcn_sched_barrier(0);
        *reinterpret_cast<u32x4*>(lds + lane16) = r.lv;
        if (__builtin_expect(pair_has_last_piece(r.sl), 0)) {
            if (lane == 0) *reinterpret_cast<u32x4*>(lds + kPairLastPiece) = *reinterpret_cast<const u32x4*>(r.list + 16u + kPairLastPiece);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const uint32_t m = ((r.p0 | r.p1 | r.p2) ^ 0xFFFFu) & 0xFFFFu;
        const uint32_t cnt = __popc(m);
        const uint32_t inc = wave_incl_scan(cnt);
        const uint32_t tot_a = __builtin_amdgcn_readlane(inc, 31), tot = __builtin_amdgcn_readlane(inc, 63);
        bad |= r.sl.bad | (tot_a ^ r.sl.count_a) | ((tot - tot_a) ^ r.sl.count_b);      /* planes and IDX must agree */
        /* the lane's zero-point exponents, those of its first eight values in front (clamped, so that a corrupt stream
           still reads inside the region) */
        const uint32_t first = min(r.sl.mis + (inc - cnt), 2u * kGroup + 15u);
        const uint32_t at[2] = {first, first + (uint32_t)__popc(m & 0xFFu)};
        float x[16];
#pragma unroll
        for (uint32_t h = 0; h < 2; ++h) {
            const uint32_t* w = reinterpret_cast<const uint32_t*>(lds + (at[h] & ~3u));
            DecEsc es;
            es.m = h ? m >> 8 : m & 0xFFu;
            es.l8 = __builtin_amdgcn_alignbyte(w[1], w[0], at[h] & 3u);
            es.h8 = __builtin_amdgcn_alignbyte(w[2], w[1], at[h] & 3u);
            DecIn in;
            in.sm0 = h ? r.sm.z : r.sm.x; in.sm1 = h ? r.sm.w : r.sm.y;
            in.b0 = h ? r.p0 >> 8 : r.p0 & 0xFFu;
            in.b1 = h ? r.p1 >> 8 : r.p1 & 0xFFu;
            in.b2 = h ? r.p2 >> 8 : r.p2 & 0xFFu;
            uint32_t lA, hA, lB, hB;
            decode_bytes(in, es, r.e0, tab, lA, hA, lB, hB);
#pragma unroll
            for (uint32_t j = 0; j < 4; ++j) {    /* value j as FP32 bits: high byte, low byte, 16 zero bits */
                const uint32_t sel = ((4u + j) << 24) | (j << 16) | 0x0C0Cu;
                x[8 * h + j] = __uint_as_float(perm(hA, lA, sel));
                x[8 * h + 4 + j] = __uint_as_float(perm(hB, lB, sel));
            }
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[j] += x[j];
        /* the additions happen here: put off past the next stage's loads, the decoded values cost more registers
           than there are */
        asm volatile("" : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "+v"(acc[4]), "+v"(acc[5]), "+v"(acc[6]), "+v"(acc[7]),
                          "+v"(acc[8]), "+v"(acc[9]), "+v"(acc[10]), "+v"(acc[11]), "+v"(acc[12]), "+v"(acc[13]), "+v"(acc[14]), "+v"(acc[15]));
    };

    /* the pipeline of reduce_stages, stage k = accepted slot k */
    PairBuf bufA, bufB;
    front(bufA);
    front(bufB);
    __builtin_amdgcn_s_waitcnt(0xC07F);  /* lgkmcnt(0): nothing pending when the loop is entered */
    issue(bufA);
    uint32_t k = 0;                      /* stage whose loads bufA holds */
    while (k + 2u < n_acc) {             /* two stages, each with a real stage to look ahead to */
        front(bufA);
        asm volatile("" ::: "memory");
        issue(bufB);
        consume(bufA);
        front(bufB);
        asm volatile("" ::: "memory");
        issue(bufA);
        consume(bufB);
        k += 2u;
    }
    if (k + 2u == n_acc) {               /* two stages left */
        issue(bufB);
        consume(bufA);
        consume(bufB);
    } else {
        consume(bufA);
    }

    uint8_t* __restrict__ og = a.out + gs * OES;
    bool any_nan = false;
#pragma unroll
    for (int j = 0; j < 16; j += 2) any_nan |= acc[j] != acc[j] || acc[j + 1] != acc[j + 1];
    if (__builtin_expect(__ballot(any_nan) != 0ull, 0)) {
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[j] = __uint_as_float(sum_bits(acc[j]));
    }
    /* The lane's 16 sums are 64 (bf16: 32) contiguous bytes; they leave through the wave's LDS region as 16
       contiguous bytes per lane, 2 KiB at a time. */
    constexpr uint32_t PIECES = 16u * OES / 16u, ROUNDS = PIECES / 2u;       /* 16-byte pieces per lane */
    u32x4 piece[PIECES];
    if (ODT == ZIPCCL_FP32) {
#pragma unroll
        for (uint32_t q = 0; q < PIECES; ++q)
            piece[q] = u32x4{__float_as_uint(acc[4 * q]), __float_as_uint(acc[4 * q + 1]),
                             __float_as_uint(acc[4 * q + 2]), __float_as_uint(acc[4 * q + 3])};
    } else {
#pragma unroll
        for (uint32_t q = 0; q < PIECES; ++q) {
            uint32_t o[4];
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k)
                o[k] = f32_bits_to_bf16_bits(__float_as_uint(acc[8 * q + 2 * k])) |
                       (f32_bits_to_bf16_bits(__float_as_uint(acc[8 * q + 2 * k + 1])) << 16);
            piece[q] = u32x4{o[0], o[1], o[2], o[3]};
        }
    }
    constexpr uint32_t LANES = 64u / ROUNDS;                                 /* lanes that hand over per round */
#pragma unroll
    for (uint32_t h = 0; h < ROUNDS; ++h) {
        if (lane / LANES == h) {
#pragma unroll
            for (uint32_t q = 0; q < PIECES; ++q)
                *reinterpret_cast<u32x4*>(lds + ((lane % LANES) * PIECES + q) * 16u) = piece[q];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const u32x4 r0 = *reinterpret_cast<const u32x4*>(lds + lane16);
        const u32x4 r1 = *reinterpret_cast<const u32x4*>(lds + 1024u + lane16);
        __builtin_amdgcn_wave_barrier();
        st_stream_a4((og + h * 2048u) + lane16, r0);
        st_stream_a4((og + h * 2048u + 1024u) + lane16, r1);
    }
}

/*
 * One launch covers a call: workgroups 0 .. a.n_full - 1 take whole tiles of a.gpw groups per wave (every group
 * complete, the output dword-aligned: the form without bounds checks), the workgroups after them the rest of the
 * shard in tiles of a.gpw_rest groups per wave through the general form.  Groups per wave: the larger, the fewer
 * workgroups pay for the header checks and the table build; 1 for small shards, and for the rest behind whole
 * tiles, so that there are enough workgroups to fill the chip.  PAIR: whole tiles are taken by reduce_pair
 * (a.gpw = 2).  REST = false: the launch holds whole tiles only (the general form is compiled out: it costs the
 * whole-tile workgroups registers to share a kernel with it).  Workgroup a.n_work, if there is one, only looks at the slots'
 * first index entries.  Dynamic LDS: one 32-bit word per peer.
 */
template <int DT, int ODT, bool REST, bool PAIR>
__global__ __launch_bounds__(kThreads, DT == ZIPCCL_BF16 ? (REST ? 7 : 8) : 6) void k_decompress_reduce(const ReduceArgs a)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t s_dyn[];
    uint32_t* s_peer = reinterpret_cast<uint32_t*>(s_dyn);     /* the accepted slots, in slot order */
    __shared__ DecTables s_tab;
    /* per wave: the zero-point slice of the group or pair being decoded, or sums on their way out */
    constexpr uint32_t kRegion = PAIR ? kPairRegion : (kEscRegion > 1024u ? kEscRegion : 1024u);
    __shared__ __attribute__((aligned(16))) uint8_t s_esc[kWavesPerBlock][kRegion];
    __shared__ uint32_t s_wcnt[kWavesPerBlock];
    build_tables(s_tab);

    const uint64_t n = a.n;
    const bool whole = !REST || blockIdx.x < a.n_full;        /* workgroup-uniform */
    const uint32_t gpw = whole ? a.gpw : a.gpw_rest;
    constexpr uint64_t kGroupStride = (uint64_t)kGroup * kWavesPerBlock;
    const uint64_t ts = whole ? (uint64_t)blockIdx.x * (kGroupStride * a.gpw)
                              : (uint64_t)a.n_full * (kGroupStride * a.gpw) + (uint64_t)(blockIdx.x - a.n_full) * (kGroupStride * a.gpw_rest);
    const SlotLayout L = slot_layout(n, DT);
    const uint32_t lane = lane_id();
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   /* scalar: group addresses are wave-uniform */

    /* every slot's header is checked once per workgroup, one peer per thread; the accepted ones are
       listed in slot order (ballot + per-wave counts), the others are left out of the sum */
    uint32_t n_acc = 0;
    for (uint32_t r = 0; r < a.n_peers; r += kThreads) {
        const uint32_t p = r + threadIdx.x;
        const uint64_t slot_off = (uint64_t)p * a.slot_cap;
        uint32_t e0 = 0, n_esc = 0;
        const bool ok = p < a.n_peers && check_header<DT>(load_header(a.comp + slot_off), L, n, slot_off, a.comp_capacity, e0, n_esc);
        const uint64_t votes = __ballot(ok);
        if (lane == 0) s_wcnt[wave] = (uint32_t)__popcll(votes);
        __syncthreads();
        uint32_t before = 0, total = 0;
#pragma unroll
        for (uint32_t w = 0; w < kWavesPerBlock; ++w) {
            const uint32_t c = s_wcnt[w];
            before += w < wave ? c : 0u;
            total += c;
        }
        if (ok) {
            const uint32_t pos = n_acc + before + (uint32_t)__popcll(votes & ((1ull << lane) - 1ull));
            s_peer[pos] = p;
        }
        n_acc += total;
        __syncthreads();
    }
    n_acc = __builtin_amdgcn_readfirstlane(n_acc);
    uint32_t bad = n_acc != a.n_peers;

    if (!PAIR && blockIdx.x == a.n_work) {
        /* a workgroup behind the others looks whether the first two index entries of every slot ascend, for shards whose
           first group is not in a pair, which asks for itself.  (Asked at every stage, this costs 16 peers' slots of a few
           tiles 3 %; by the waves of the first workgroup, in the header check or at their end, 1 to 2 %.) */
        for (uint32_t j = threadIdx.x; j < n_acc; j += kThreads) {
            const uint8_t* const slot = a.comp + (uint64_t)s_peer[j] * a.slot_cap;
            const uint32_t* const idx = reinterpret_cast<const uint32_t*>(slot + L.idx);
            const uint32_t n_esc = *reinterpret_cast<const uint32_t*>(slot + 24);
            bad |= slice_bad(idx[0], n > kGroup ? idx[1] : n_esc, n_esc, true);
        }
        if (bad && a.status) atomicOr(a.status, (uint32_t)ZIPCCL_ERR_CORRUPT);
        return;
    }
    if (PAIR && whole) {                /* whole tiles of 8 groups: two neighbouring ones per wave */
        if (n_acc != 0u) {
            reduce_pair<ODT>(a, L, ts + (uint64_t)wave * (2 * kGroup), n_acc, lane, s_esc[wave], s_tab, s_peer, n_acc == a.n_peers, bad);
            if (bad && a.status) atomicOr(a.status, (uint32_t)ZIPCCL_ERR_CORRUPT);
            return;
        }
    }
    /* this wave's groups start at gs0, gs0 + 2048, ...; those that begin inside n count */
    const uint64_t gs0 = ts + (uint64_t)wave * kGroup;
    uint32_t n_groups = gpw;
    if (!whole) n_groups = gs0 >= n ? 0u : (uint32_t)min((uint64_t)gpw, (n - gs0 + kGroupStride - 1) / kGroupStride);
    if (n_groups != 0u) {
        if (n_acc != 0u) {
            if (!PAIR && whole) reduce_stages<DT, ODT, true>(a, L, gs0, n_groups, n_acc, lane, s_esc[wave], s_tab, s_peer, n_acc == a.n_peers, bad);
            else if (REST) reduce_stages<DT, ODT, false>(a, L, gs0, n_groups, n_acc, lane, s_esc[wave], s_tab, s_peer, n_acc == a.n_peers, bad);
        } else {
            /* no slot accepted: the sum of nothing */
            constexpr uint32_t OES = ODT == ZIPCCL_BF16 ? 2u : 4u;
            for (uint32_t u = 0; u < n_groups; ++u) {
                const uint64_t e = gs0 + u * kGroupStride + lane * kLaneElems;
                for (uint32_t j = 0; j < kLaneElems; ++j) {
                    if (e + j < n) {
                        if (ODT == ZIPCCL_FP32) *reinterpret_cast<uint32_t*>(a.out + (e + j) * OES) = 0u;
                        else *reinterpret_cast<uint16_t*>(a.out + (e + j) * OES) = 0u;
                    }
                }
            }
        }
    }
    if (bad && a.status) atomicOr(a.status, (uint32_t)ZIPCCL_ERR_CORRUPT);
}

/* Arguments of k_reduce_split, with the slot's layout from the host: a shard that is small enough for it has offsets of 32 bits. */
struct SplitArgs {
    const uint8_t* comp;
    uint64_t comp_capacity, slot_cap;
    uint8_t* out;
    uint32_t* status;
    uint32_t n, n_peers;
    uint32_t lo, p0, plane_bytes, idx, esc;       /* SlotLayout; sm is 128 */
};

/*
 * The same sums for small shards, which have too few groups to fill the chip: S waves share a group's peers, Q consecutive
 * ones each per round of S * Q, decode them into LDS, and every wave then adds an S-th of the group's values over all
 * peers of the round, in slot order.  A wave per group walks its peers one after the other, and that chain of decodes is
 * what a small call lasts; here it is Q long.  Nothing of a slot but its zero-point list depends on its header, so the
 * rest is requested before the headers are checked, and a round's before the sums of the one before it.  G groups per
 * workgroup share its tables (8 x 1 000 003 bf16 values: 8.2 us with a wave per group, 7.1 with G = 1, 6.9 with 2).  At
 * that size vector and scalar issue are what bounds it, some 290 instructions of each per wave, half of them the two
 * decodes; below 2^18 values it is latency: launch, headers, index, list (8 x 2^15: 6.3 -> 3.8 us, 2.1 of them the launch).
 * Dynamic LDS: one 32-bit word per peer.
 */
template <int DT, int ODT, uint32_t S, uint32_t G, uint32_t Q>
__global__ __launch_bounds__(64u * S * G) void k_reduce_split(const SplitArgs a)
{
    constexpr uint32_t OES = ODT == ZIPCCL_BF16 ? 2u : 4u, THREADS = 64u * S * G, R = S * Q;
    constexpr uint32_t PIECES = DT == ZIPCCL_BF16 ? 1u : 2u;          /* 16-byte pieces of a lane's 8 decoded values */
    constexpr uint32_t NV = kLaneElems / S;                           /* values per lane in the sums */
    extern __shared__ __attribute__((aligned(16))) uint8_t s_dyn[];
    uint32_t* const s_ok = reinterpret_cast<uint32_t*>(s_dyn);        /* per slot: accepted? */
    __shared__ DecTables s_tab;
    __shared__ __attribute__((aligned(16))) uint8_t s_esc[S * G][1024];
    __shared__ __attribute__((aligned(16))) uint8_t s_val[G][R][PIECES * 1024u];
    __shared__ uint32_t s_rejected;

    const uint32_t n = a.n, ng = (n + kGroup - 1u) / kGroup;
    const uint32_t lane = lane_id();
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t sub = wave % S, gw = wave / S;
    const bool here = blockIdx.x * G + gw < ng;                       /* the last workgroup may have fewer groups */
    const uint32_t g = min(blockIdx.x * G + gw, ng - 1u), gs = g * kGroup;
    const bool last_group = g + 1u == ng;
    const uint32_t left = n - gs, e = lane * kLaneElems;              /* values from the group's first on; the lane's first */
    /* lanes past the end of the shard read the group's first bytes instead */
    const uint32_t lane8 = e < left ? e : 0u;
    const uint32_t vmask = e >= left ? 0u : (1u << min(left - e, 8u)) - 1u;

    struct Stage { DecIn in; uint32_t next, nesc, dec; const uint8_t* slot; } st[Q];
    auto request = [&](uint32_t first) {
        const uint32_t p = first + sub * Q, last = a.n_peers - 1u;
        const uint8_t* slot = a.comp + min(p, last) * a.slot_cap;
#pragma unroll
        for (uint32_t q = 0; q < Q; ++q) {
            Stage& r = st[q];
            r.slot = slot;
            r.nesc = load_const_u32(slot + 24);
            r.dec = load_const_u32(slot + 40);
            const uint8_t* const idx = slot + (a.idx + 4u * g);
            r.in.base = load_const_u32(idx);
            r.next = load_const_u32(idx + (last_group ? 0u : 4u));
            const u32x2 sm = ld_stream<u32x2>((slot + (128u + gs)) + lane8);
            r.in.sm0 = sm.x; r.in.sm1 = sm.y;
            /* half a cache line each, whose other half another wave wants: not streamed */
            const uint8_t* const pl = slot + (a.p0 + gs / 8u);
            r.in.b0 = *(pl + lane);
            r.in.b1 = *((pl + a.plane_bytes) + lane);
            r.in.b2 = *((pl + 2u * a.plane_bytes) + lane);
            if (DT == ZIPCCL_FP32) {
                const u32x4 lo = ld_stream<u32x4>((slot + (a.lo + 2u * gs)) + 2u * lane8);
                r.in.lo[0] = lo.x; r.in.lo[1] = lo.y; r.in.lo[2] = lo.z; r.in.lo[3] = lo.w;
            }
            if (p + q < last) slot += a.slot_cap;                     /* behind the last peer: the last once more */
        }
    };
    request(0);

    if (threadIdx.x == 0) s_rejected = 0;
    build_tables<THREADS>(s_tab);                                     /* contains a barrier */
    SlotLayout L;                                                     /* what check_header wants of it */
    L.esc = a.esc;
    for (uint32_t p = threadIdx.x; p < a.n_peers; p += THREADS) {
        const uint64_t slot_off = (uint64_t)p * a.slot_cap;
        uint32_t e0 = 0, n_esc = 0;
        const bool ok = check_header<DT>(load_header(a.comp + slot_off), L, n, slot_off, a.comp_capacity, e0, n_esc);
        s_ok[p] = ok;
        if (!ok) atomicAdd(&s_rejected, 1u);
    }
    __syncthreads();
    const uint32_t rejected = __builtin_amdgcn_readfirstlane(s_rejected);
    uint32_t bad = rejected;

    float acc[NV];
#pragma unroll
    for (uint32_t j = 0; j < NV; ++j) acc[j] = -0.0f;
    const uint32_t i0 = (sub * 64u + lane) * NV;                      /* the lane's values of the group in the sums */
    uint8_t* const lds = s_esc[wave];
    for (uint32_t first = 0;;) {
        const uint32_t p0 = first + sub * Q;
        u32x4 lv[Q];
        bool go[Q];
#pragma unroll
        for (uint32_t q = 0; q < Q; ++q) {
            Stage& r = st[q];
            go[q] = p0 + q < a.n_peers;
            /* of a rejected slot nothing but the static part may be read */
            if (rejected != 0u && go[q]) go[q] = __builtin_amdgcn_readfirstlane(s_ok[p0 + q]) != 0u;
            if (last_group) r.next = r.nesc;
            r.in.idx_bad = slice_bad(r.in.base, r.next, r.nesc, true);
            r.in.count = r.in.idx_bad | (uint32_t)!go[q] ? 0u : r.next - r.in.base;
            r.in.vmask = vmask;
            /* the list as in decode_fetch_list, relative to 16 bytes before it */
            const uint32_t end = r.in.count != 0u ? r.next : 0u, a16 = (r.in.base & ~15u) + 16u * lane;
            lv[q] = *reinterpret_cast<const u32x4*>((r.slot + (a.esc - 16u)) + (a16 < end ? a16 + 16u : 0u));
        }
#pragma unroll
        for (uint32_t q = 0; q < Q; ++q) {
            if (!go[q]) continue;                                     /* wave-uniform */
            *reinterpret_cast<u32x4*>(lds + 16u * lane) = lv[q];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const DecEsc es = decode_locate(st[q].in, lds);
            __builtin_amdgcn_wave_barrier();
            bad |= es.bad;
            uint32_t hp[4];
            decode_values(st[q].in, es, (st[q].dec >> 8) & 0xFFu, s_tab, hp);
            u32x4* const to = reinterpret_cast<u32x4*>(s_val[gw][sub * Q + q] + lane * (16u * PIECES));
            if (DT == ZIPCCL_BF16) {
                to[0] = u32x4{hp[0], hp[1], hp[2], hp[3]};
            } else {
                uint32_t x[8];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    x[2 * k] = perm(hp[k], st[q].in.lo[k], 0x05040100u);
                    x[2 * k + 1] = perm(hp[k], st[q].in.lo[k], 0x07060302u);
                }
                to[0] = u32x4{x[0], x[1], x[2], x[3]};
                to[PIECES - 1u] = u32x4{x[4], x[5], x[6], x[7]};
            }
        }
        const uint32_t count = min(R, a.n_peers - first), done = first;
        first += R;
        const bool more = first < a.n_peers;
        if (more) request(first);
        __syncthreads();
        auto add = [&](uint32_t j) {
            typedef float values __attribute__((ext_vector_type(NV)));
            typedef uint16_t halves __attribute__((ext_vector_type(NV)));
            const uint8_t* const v = s_val[gw][j] + i0 * (DT == ZIPCCL_BF16 ? 2u : 4u);
            if (DT == ZIPCCL_BF16) {
                const halves x = *reinterpret_cast<const halves*>(v);
#pragma unroll
                for (uint32_t k = 0; k < NV; ++k) acc[k] += __uint_as_float((uint32_t)x[k] << 16);
            } else {
                const values x = *reinterpret_cast<const values*>(v);
#pragma unroll
                for (uint32_t k = 0; k < NV; ++k) acc[k] += x[k];
            }
        };
        if (rejected == 0u && count == R) {
#pragma unroll
            for (uint32_t j = 0; j < R; ++j) add(j);
        } else {
            for (uint32_t j = 0; j < count; ++j)
                if (s_ok[done + j] != 0u) add(j);
        }
        if (!more) break;
        __syncthreads();
    }
    if (!here) return;
    if (rejected == a.n_peers) {                                      /* the sum of nothing */
#pragma unroll
        for (uint32_t j = 0; j < NV; ++j) acc[j] = 0.0f;
    }
    uint32_t u[NV];
#pragma unroll
    for (uint32_t j = 0; j < NV; ++j) {
        u[j] = sum_bits(acc[j]);
        if (ODT == ZIPCCL_BF16) u[j] = f32_bits_to_bf16_bits(u[j]);
    }
    uint8_t* __restrict__ o = (a.out + (uint64_t)gs * OES) + i0 * OES;
    if (left >= kGroup) {                                             /* a whole group, at any element */
        typedef uint32_t words __attribute__((ext_vector_type(NV), aligned(4)));
        typedef uint16_t halves __attribute__((ext_vector_type(NV), aligned(2)));
        words w;
        halves h;
#pragma unroll
        for (uint32_t j = 0; j < NV; ++j) { w[j] = u[j]; h[j] = (uint16_t)u[j]; }
        if (ODT == ZIPCCL_FP32) *reinterpret_cast<words*>(o) = w;
        else *reinterpret_cast<halves*>(o) = h;
    } else {
#pragma unroll
        for (uint32_t j = 0; j < NV; ++j) {
            if (i0 + j < left) {
                if (ODT == ZIPCCL_FP32) *reinterpret_cast<uint32_t*>(o + j * 4u) = u[j];
                else *reinterpret_cast<uint16_t*>(o + j * 2u) = (uint16_t)u[j];
            }
        }
    }
    if (bad && a.status) atomicOr(a.status, (uint32_t)ZIPCCL_ERR_CORRUPT);
}

} // namespace

/*
 * Large fp32 launches ask for LDS that they do not use, so that five workgroups share a compute unit and not eight, which get in one
 * another's way at the memory.  us with 8 / 6 / 5 / 4: 64 chunks of 2^21 values with rows of gains 163.4 / 164.0 / 161.2 / 163.9, normal
 * ones 160.2 / 160.6 / 158.8 / -, one chunk of 2^27 162.5 / 162.8 / 159.5 / -, 2^26 82.4 / 82.5 / 81.5 / -; 64 odd chunks of 120 million values in
 * all 149.5 / 151.2 / 149.5 / -, 2^25 43.0 / 42.9 / 42.9 / 43.8.  bf16 launches, with half the bytes in flight, lose by it (2^29 294 /
 * 299 with 6).
 */
constexpr uint64_t kFiveFrom = 1ull << 25;
constexpr uint32_t kFiveLds = 14u << 10;                     /* on top of 14.4 KiB; a compute unit has 160 */
static_assert(5u * (sizeof(DecTables) + kWavesPerBlock * 2u * kEscRegion + kFiveLds) <= (160u << 10) &&
              6u * (sizeof(DecTables) + kWavesPerBlock * 2u * kEscRegion + kFiveLds) > (160u << 10), "five, not six");

template <int DT, uint32_t GPW, bool STREAM = true>
static int launch_decompress_gpw(const DecompressArgs& a, hipStream_t s)
{
    constexpr uint64_t TILE = (uint64_t)kGroup * kWavesPerBlock * GPW;
    uint64_t tiles = 1;
    for (uint32_t c = 0; c < a.tab.n_chunks; ++c) {
        const uint64_t t = (a.tab.elem_off[c + 1] - a.tab.elem_off[c] + TILE - 1) / TILE;
        tiles = t > tiles ? t : tiles;
    }
    const dim3 grid((uint32_t)tiles, a.tab.n_chunks), block(kThreads);
    const DecompressIo io = {a.comp, a.comp_capacity, a.out, a.status};
    const uint32_t lds = DT == ZIPCCL_FP32 && GPW == 2u && a.tab.elem_off[a.tab.n_chunks] > kFiveFrom ? kFiveLds : 0u;
    if (is_equal_split(a.tab)) hipLaunchKernelGGL((k_decompress<DT, GPW, STREAM, EqualSplit>), grid, block, lds, s, io, equal_split(a.tab));
    else if (GPW < 4u && is_few_split(a.tab)) hipLaunchKernelGGL((k_decompress<DT, GPW, STREAM, FewSplit>), grid, block, lds, s, io, few_split(a.tab));
    else hipLaunchKernelGGL((k_decompress<DT, GPW, STREAM, ChunkTab>), grid, block, lds, s, io, a.tab);
    return (int)hipGetLastError();
}

/*
 * Groups per wave by the values of the launch, from timings on MI355X (us in a graph, 1 / 2 / 4 groups).  bf16: 2^18
 * values 2.9 / 3.2 / 3.9, 2^20 3.4 / 3.4 / 4.1, 2^21 4.2 / 3.7 / 4.2, 2^22 - / 4.5 / 4.6, 4.5 * 2^20 - / 5.6 / 5.3, 5.25 *
 * 2^20 - / 6.0 / 5.3, 2^23 9.4 / 7.4 / 6.0, 2^24 15.2 / 11.9 / 11.8, 24 * 2^20 21.0 / 16.3 / 17.1; 2^28 72.6 with two, 74.4
 * with four.  fp32: 2^18 3.3 / 3.7 / 4.6, 2^20 4.2 / 4.4 / 5.4, 2^21 5.0 / 5.0 / 5.9, 2^22 7.3 / 6.5 / 7.6, 5 * 2^20 - / 8.0
 * / 8.9, 5.25 * 2^20 - / 9.9 / 8.7, 6 * 2^20 - / 9.9 / 8.7, 6.25 * 2^20 - / 11.1 / 12.5, 7.25 * 2^20 - / 12.9 / 12.9, 2^23 - /
 * 13.5 / 12.6, 8.1 * 2^20 - / 13.9 / 15.1.  In small launches fewer groups per wave mean more waves that share one chain
 * of latencies.  Launches of a few workgroups per compute unit take the time of the fullest unit: in steps of 2^21
 * values (256 workgroups of 8192) with four, of 2^20 with two, so that four win towards the upper end of their steps; for
 * fp32 these are the ones that end at 6 and at 8 * 2^20.  Four only where the chunks start on line boundaries (64 chunks of
 * 131 073 bf16 values 7.9 us with two neighbouring groups, 8.3 with four), and below 5 * 2^20 bf16 values not for many
 * chunks with rests (128 chunks of 37 824 values 6 % slower with four).
 *
 * Launches of four groups on more than kPlainFrom bf16 values (21 to 40 MiB of them), and all of fp32 values (20 to 24 and 29 to 32 MiB), do not
 * stream their loads: of the compressed buffer, which something has written shortly before, a part is then still read from the last-level
 * cache.  us, streamed / plain, with 1, 3, 5 and 12 sets of buffers in turn, 2^24 bf16 values: every buffer copied into before its call
 * 13.7 / 10.8, 12.9 / 10.0, 10.2 / 9.2, 11.2 / 9.7; all copied into, then all decompressed 13.6 / 10.7, 13.9 / 10.1, 12.1 / 11.2, 13.1 / 13.5; not
 * written between the calls 11.5 / 8.9, 11.6 / 10.1, 12.6 / 10.2, 12.9 / 12.9; compressed into before its call 12.0 / 10.4, 13.2 / 13.4, 12.8 /
 * 12.8, 12.8 / 12.9.  6 * 2^20 fp32, copied into before the call: 11.8 / 9.7, 9.8 / 8.5, 8.3 / 8.2, 8.3 / 8.1.  With more sets than the cache holds
 * between write and read it loses up to 6 %.  On either side of these sizes, buffers copied into before the call: 2^23 bf16 8.4 / 8.5, 7.1 / 6.9,
 * 7.0 / 6.7, 5.6 / 6.6; 24 * 2^20, two groups per wave, 15.2 / 14.8, 11.1 / 12.1, 11.9 / 13.4, 11.9 / 13.3.
 */
constexpr uint64_t kPlainFrom = 21ull << 19;
int launch_decompress(int dt, const DecompressArgs& a, void* stream)
{
    const uint64_t n = a.tab.elem_off[a.tab.n_chunks] - a.tab.elem_off[0];
    hipStream_t s = (hipStream_t)stream;
    uint64_t starts = reinterpret_cast<uintptr_t>(a.out), ends = 0;
    for (uint32_t c = 0; c < a.tab.n_chunks; ++c) {
        starts |= elem_size(dt) * a.tab.elem_off[c];
        ends |= a.tab.elem_off[c + 1];
    }
    const bool lines = starts % 128u == 0;
    if (dt == ZIPCCL_FP32) {
        if (n < (2ull << 20)) return launch_decompress_gpw<ZIPCCL_FP32, 1>(a, s);
        const bool four = (n > (5ull << 20) && n <= (6ull << 20)) || (n > (29ull << 18) && n <= (8ull << 20));
        return lines && four ? launch_decompress_gpw<ZIPCCL_FP32, 4, false>(a, s) : launch_decompress_gpw<ZIPCCL_FP32, 2>(a, s);
    }
    if (n < (1ull << 20)) return launch_decompress_gpw<ZIPCCL_BF16, 1>(a, s);
    const bool few_rests = a.tab.n_chunks <= 64u || ends % kTile == 0;
    const bool four = n < (20ull << 20) && (n > (5ull << 20) || (n > (4ull << 20) && few_rests));
    if (!lines || !four) return launch_decompress_gpw<ZIPCCL_BF16, 2>(a, s);
    return n > kPlainFrom ? launch_decompress_gpw<ZIPCCL_BF16, 4, false>(a, s) : launch_decompress_gpw<ZIPCCL_BF16, 4>(a, s);
}


/*
 * Groups per wave of the fused reduce, from timings on MI355X over shards of 2^18 to 2^27 values, 2 to 64 peers.  One
 * group per wave while the shard gives the chip's resident workgroups too little to do for a second group to pay, two
 * from there on: for bf16 as a pair of neighbours (reduce_pair), where more peers make a longer chain per wave and want
 * more waves.  us, one group against a pair, 128 / 256 / 384 / 512 tiles of 8192 values: 8 peers 7.8 / 9.1, 10.3 / 10.5,
 * 13.2 / 13.6, 15.6 / 15.4, then 18.8 / 17.1 at 640; 2 peers 7.1 / 6.1 at 384; 16 peers 20.8 / 21.3 at 384, 22.6 / 23.5 at
 * 448 (the last whole number of one-group workgroups per compute unit), 25.0 / 24.0 at 456; 64 peers 69.9 / 78.5 at 384, 88.8
 * / 89.2 at 512.  bf16 sums, and shards with a rest, whose kernel leaves room for fewer waves, are no worse off as
 * pairs from 384 tiles on (16 peers, 448 tiles and 1000 values: one group 11 % slower).
 */
static uint32_t reduce_groups_per_wave(uint64_t n, int dt, int out_dt, uint32_t n_peers)
{
    const uint64_t tiles = n / kTile;
    if (dt == ZIPCCL_FP32) return tiles < 2560u ? 1u : 2u;
    const uint32_t from = n_peers > 16u ? 512u : (n_peers > 6u && out_dt == ZIPCCL_FP32 && n % kTile == 0 ? 449u : 384u);
    return tiles < from ? 1u : 2u;
}

/*
 * Which shards take k_reduce_split, with how many waves per group x peers per wave and round: those whose groups, one per
 * wave, leave most of the chip's waves empty, while the split's own work per wave (tables, headers, handing over) still
 * costs less than the chain it cuts.  us, wave per group / split, bf16, 2^18 values: 2 peers 3.8 / 3.3 (2 x 1), 4 4.7 / 3.3 (4 x 1),
 * 8 6.6 / 4.0 (4 x 2), 16 10.6 / 5.2 (8 x 2; 5.9 with 4 x 2), 64 34.3 / 13.0.  They meet at about 1.6 * 10^6 values for 2 peers,
 * 1.2 * 10^6 where the peers fill the rounds (8 peers 9.5 / 8.5 there, 9.3 / 9.4 at 1.35 * 10^6), 0.8 * 10^6 otherwise (5 peers
 * 6.5 / 5.7 at 0.7, 6.5 / 6.5 at 1.05); fp32, which moves more per value, at 1.4 and 0.8 * 10^6 (8 peers 8.6 / 7.3 at 0.7, 8.9 / 8.8
 * at 1.05), and 4 x 1 is no worse than 4 x 2 there.
 */
enum SplitForm { kNoSplit, kSplit2x1, kSplit4x1, kSplit4x2, kSplit8x2 };

static SplitForm split_form(uint64_t n, int dt, uint32_t n_peers)
{
    const bool bf16 = dt == ZIPCCL_BF16;
    if (n == 0 || n_peers < 2u) return kNoSplit;
    if (n_peers == 2u) return n <= (bf16 ? 192u : 160u) * (uint64_t)kTile ? kSplit2x1 : kNoSplit;
    if (n > (bf16 ? (n_peers % 4u == 0u ? 146u : 96u) : 86u) * (uint64_t)kTile) return kNoSplit;
    if ((n_peers > 8u && n <= 16u * kTile) || (n_peers > 12u && n <= 32u * kTile)) return kSplit8x2;
    return bf16 && (n_peers - 1u) % 8u >= 4u ? kSplit4x2 : kSplit4x1;      /* a last round of 8 that is at least 5 full */
}

template <uint32_t S, uint32_t G, uint32_t Q>
static int launch_reduce_split(int dt, int out_dt, const ReduceArgs& a, hipStream_t s)
{
    const dim3 grid((uint32_t)((a.n + kGroup * G - 1) / (kGroup * G))), block(64u * S * G);
    const size_t lds_bytes = sizeof(uint32_t) * a.n_peers;
    const SlotLayout L = slot_layout(a.n, dt);
    const SplitArgs b = {a.comp, a.comp_capacity, a.slot_cap, a.out, a.status, (uint32_t)a.n, a.n_peers,
                         (uint32_t)L.lo, (uint32_t)L.p0, (uint32_t)L.plane_bytes, (uint32_t)L.idx, (uint32_t)L.esc};
    if (dt == ZIPCCL_BF16 && out_dt == ZIPCCL_BF16) hipLaunchKernelGGL((k_reduce_split<ZIPCCL_BF16, ZIPCCL_BF16, S, G, Q>), grid, block, lds_bytes, s, b);
    else if (dt == ZIPCCL_BF16) hipLaunchKernelGGL((k_reduce_split<ZIPCCL_BF16, ZIPCCL_FP32, S, G, Q>), grid, block, lds_bytes, s, b);
    else if constexpr (S == 4u && Q == 2u) return 1;      /* kSplit4x2 is a form for bf16 */
    else if (out_dt == ZIPCCL_BF16) hipLaunchKernelGGL((k_reduce_split<ZIPCCL_FP32, ZIPCCL_BF16, S, G, Q>), grid, block, lds_bytes, s, b);
    else hipLaunchKernelGGL((k_reduce_split<ZIPCCL_FP32, ZIPCCL_FP32, S, G, Q>), grid, block, lds_bytes, s, b);
    return (int)hipGetLastError();
}

int launch_decompress_reduce(int dt, int out_dt, const ReduceArgs& a, void* stream)
{
    hipStream_t s = (hipStream_t)stream;
    switch (split_form(a.n, dt, a.n_peers)) {
        case kSplit2x1: return launch_reduce_split<2, 4, 1>(dt, out_dt, a, s);
        case kSplit4x1: return launch_reduce_split<4, 2, 1>(dt, out_dt, a, s);
        case kSplit4x2: return launch_reduce_split<4, 2, 2>(dt, out_dt, a, s);
        case kSplit8x2: return launch_reduce_split<8, 1, 2>(dt, out_dt, a, s);
        case kNoSplit: break;
    }
    const dim3 block(kThreads);
    ReduceArgs b = a;
    b.gpw = reduce_groups_per_wave(a.n, dt, out_dt, a.n_peers);
    const uint64_t per = (uint64_t)kGroup * kWavesPerBlock * b.gpw;
    /* whole tiles with a dword-aligned output go through the form without bounds checks, the rest (under one
       tile, or everything when the output is only 2-byte aligned) through the general one, in the same launch */
    const size_t lds_bytes = sizeof(uint32_t) * a.n_peers;
    const bool aligned = (reinterpret_cast<uintptr_t>(a.out) & 3u) == 0;
    const uint64_t full = aligned ? a.n / per : 0;
    const uint64_t rest = a.n - full * per;
    b.n_full = (uint32_t)full;
    b.gpw_rest = full ? 1u : b.gpw;     /* under a tile is left: one group per wave, so that it is not one workgroup's crawl */
    const uint64_t per_rest = (uint64_t)kGroup * kWavesPerBlock * b.gpw_rest;
    uint64_t n_rest = (rest + per_rest - 1) / per_rest;
    if (a.n == 0) n_rest = 1;           /* one workgroup that only checks the headers */
    b.n_work = (uint32_t)(full + n_rest);
    const bool pair = dt == ZIPCCL_BF16 && b.gpw == 2u && full != 0;
    const dim3 grid(b.n_work + (pair || a.n == 0 ? 0u : 1u));      /* the last one: the slots' first index entries */
#define ZIPCCL_REDUCE(DT, ODT, PAIR)                                                                                   \
    do {                                                                                                               \
        if (n_rest) hipLaunchKernelGGL((k_decompress_reduce<DT, ODT, true, PAIR>), grid, block, lds_bytes, s, b);      \
        else hipLaunchKernelGGL((k_decompress_reduce<DT, ODT, false, PAIR>), grid, block, lds_bytes, s, b);            \
    } while (0)
    if (pair && out_dt == ZIPCCL_FP32) ZIPCCL_REDUCE(ZIPCCL_BF16, ZIPCCL_FP32, true);
    else if (pair) ZIPCCL_REDUCE(ZIPCCL_BF16, ZIPCCL_BF16, true);
    else if (dt == ZIPCCL_BF16 && out_dt == ZIPCCL_FP32) ZIPCCL_REDUCE(ZIPCCL_BF16, ZIPCCL_FP32, false);
    else if (dt == ZIPCCL_BF16) ZIPCCL_REDUCE(ZIPCCL_BF16, ZIPCCL_BF16, false);
    else if (out_dt == ZIPCCL_FP32) ZIPCCL_REDUCE(ZIPCCL_FP32, ZIPCCL_FP32, false);
    else ZIPCCL_REDUCE(ZIPCCL_FP32, ZIPCCL_BF16, false);
#undef ZIPCCL_REDUCE
    return (int)hipGetLastError();
}


} // namespace zipccl
