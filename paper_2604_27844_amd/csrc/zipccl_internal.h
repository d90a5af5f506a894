/* Internal declarations shared by the host logic and the HIP kernels of libzipccl.so. */
#ifndef ZIPCCL_INTERNAL_H
#define ZIPCCL_INTERNAL_H

#include <stddef.h>
#include <stdint.h>
#include "zipccl.h"

#if defined(__HIPCC__)
#define ZIPCCL_HD __host__ __device__ inline
#else
#define ZIPCCL_HD inline
#endif

namespace zipccl {

/* Work decomposition: a workgroup handles one TILE of 16 groups (of 4 waves, unless a kernel says otherwise); a wave handles
 * a group of 512 elements at a time, 8 consecutive elements per lane (one 16-byte bf16 load). */
constexpr uint32_t kLaneElems = 8;
constexpr uint32_t kGroup = ZIPCCL_GROUP;
constexpr uint32_t kWavesPerBlock = 4;
constexpr uint32_t kThreads = 64 * kWavesPerBlock;
constexpr uint32_t kGroupsPerWave = 4;
constexpr uint32_t kGroupsPerTile = kWavesPerBlock * kGroupsPerWave;
constexpr uint32_t kTile = kGroup * kGroupsPerTile; /* 8192 elements */
constexpr uint32_t kMaxBatch = 128;                 /* chunks per kernel launch */
constexpr uint32_t kVersion = 1;
constexpr uint32_t kMagic = 0x4C43505Au;            /* "ZPCL" little-endian */
constexpr uint32_t kWorkspaceHeader = 256;          /* reserved bytes before the per-tile arrays */
constexpr uint32_t kMaxPeers = 1024;                /* slots one zipccl_decompress_reduce call can sum */
constexpr uint32_t kFusedGroups = 508;              /* groups to count in a chunk up to which a second count of it is one workgroup's */
constexpr uint32_t kStashSlack = 64;                /* readable bytes past the last stash byte */

/* header words (u32 index): 0 magic, 1 version, 2 dtype, 3 G, 4-5 n, 6-7 n_esc, 8-9 chunk_bytes, 10-11 dec[8] */

ZIPCCL_HD uint64_t pad128(uint64_t x) { return (x + 127u) & ~(uint64_t)127u; }
ZIPCCL_HD uint32_t elem_size(int dt) { return dt == ZIPCCL_BF16 ? 2u : 4u; }

/* Byte offsets of the sections inside a slot of n elements (all multiples of 128). */
struct SlotLayout {
    uint64_t sm, lo, p0, plane_bytes, idx, esc, cap;
};

ZIPCCL_HD SlotLayout slot_layout(uint64_t n, int dt)
{
    SlotLayout L;
    L.sm = 128;
    L.lo = L.sm + pad128(n);
    L.p0 = L.lo + (dt == ZIPCCL_FP32 ? pad128(2 * n) : 0);
    L.plane_bytes = pad128((n + 7) / 8);
    L.idx = L.p0 + 3 * L.plane_bytes;
    L.esc = L.idx + pad128(4 * ((n + kGroup - 1) / kGroup));
    L.cap = L.esc + pad128(n);
    return L;
}

/*
 * Nonzero unless base <= next <= n_esc and next - base <= 512: what two consecutive index entries must be to bound a
 * group's slice of a list of n_esc zero-points.  The difference alone does not say that they ascend: it wraps, and a base
 * just below 2^32 is as little ahead of a small next as a good one.  A decoder of a whole chunk need ask so (`ascend`) of
 * the first group only: a later group's base is the next of the group before, inside the list, and if every group's
 * difference is its count of zero-points, the entries are the first one plus sums that stay below 2^32.
 */
ZIPCCL_HD uint32_t slice_bad(uint32_t base, uint32_t next, uint32_t n_esc, bool ascend)
{
    return (uint32_t)(next - base > kGroup) | (uint32_t)(next > n_esc) | (uint32_t)(ascend && base > next);
}

/*
 * The slices of the zero-point list that three consecutive index entries give two neighbouring groups, and how a wave
 * fetches both: lane l reads the 16 bytes at pair_list_offset(s, l) behind the 16 bytes in front of the list.  Entries
 * that are not base <= mid <= next <= n_esc, 512 apart at most, are bad: nothing of the list is fetched then.
 */
struct PairSlices {
    uint32_t count_a, count_b;   /* zero-points of the two groups (meaningless if bad) */
    uint32_t from;               /* base rounded down to 16, */
    uint32_t mis;                /* base - from, */
    uint32_t span;               /* and bytes from there to next, 0 for empty slices */
    uint32_t bad;
};

ZIPCCL_HD PairSlices pair_slices(uint32_t base, uint32_t mid, uint32_t next, uint32_t n_esc)
{
    PairSlices s;
    s.count_a = mid - base;
    s.count_b = next - mid;
    s.bad = (uint32_t)(s.count_a > kGroup) | (uint32_t)(s.count_b > kGroup) | (uint32_t)(next > n_esc) | (uint32_t)(base > next);
    s.from = s.bad ? 0u : base & ~15u;
    s.mis = s.bad ? 0u : base & 15u;
    s.span = s.bad || s.count_a + s.count_b == 0u ? 0u : next - s.from;
    return s;
}

ZIPCCL_HD uint32_t pair_list_offset(const PairSlices& s, uint32_t lane) { return 16u * lane < s.span ? 16u * lane + 16u : 0u; }

/* a slice of more than 64 aligned pieces (all but a few of the 1024 values are zero-points): one more, behind those */
constexpr uint32_t kPairLastPiece = 64u * 16u;
ZIPCCL_HD bool pair_has_last_piece(const PairSlices& s) { return !s.bad && s.mis + s.count_a + s.count_b > kPairLastPiece; }

ZIPCCL_HD uint64_t tiles_of(uint64_t n) { return n == 0 ? 1 : (n + kTile - 1) / kTile; }

/* Per-launch chunk table, passed by value in the kernel argument segment. */
struct ChunkTab {
    uint32_t n_chunks;
    uint32_t tile_start[kMaxBatch + 1]; /* first tile of chunk c in this launch */
    uint64_t elem_off[kMaxBatch + 1];   /* first element of chunk c, relative to the launch's input */
    uint64_t slot_off[kMaxBatch + 1];   /* byte offset of slot c, relative to the launch's output */
};

/*
 * The same in a few bytes, for the kernels of small calls: the host's part of a launch takes 2.8 us with at most 112 bytes of
 * kernel arguments, 3.5 from 120 on and 4.1 with a whole ChunkTab, and such a kernel itself runs 3 to 5 (32 x 4096 bf16
 * values in 8 chunks: compress call 4.9 -> 3.8 us of host time; two launches on 2^20 values 8.6 -> 6.6).
 */
struct EqualSplit {
    uint32_t n;                          /* elements of every chunk */
};
constexpr uint32_t kFewChunks = 8;
struct FewSplit {                        /* any split into at most kFewChunks chunks, 2^32 - 1 elements in all at most */
    uint32_t elem_off[kFewChunks + 1];
    uint32_t slot_line[kFewChunks];      /* slot_off / 128 */
};

/* The forms a launch's table allows. */
ZIPCCL_HD bool is_equal_split(const ChunkTab& t)
{
    for (uint32_t c = 1; c < t.n_chunks; ++c)
        if (t.elem_off[c + 1] - t.elem_off[c] != t.elem_off[1] - t.elem_off[0]) return false;
    return t.elem_off[0] == 0;
}

ZIPCCL_HD bool is_few_split(const ChunkTab& t)
{
    return t.n_chunks <= kFewChunks && t.elem_off[t.n_chunks] <= 0xFFFFFFFFull && t.slot_off[t.n_chunks] / 128u <= 0xFFFFFFFFull;
}

ZIPCCL_HD EqualSplit equal_split(const ChunkTab& t) { return EqualSplit{(uint32_t)t.elem_off[1]}; }

ZIPCCL_HD FewSplit few_split(const ChunkTab& t)
{
    FewSplit f = {};
    for (uint32_t c = 0; c < kFewChunks; ++c) {
        const uint32_t k = c < t.n_chunks ? c : t.n_chunks;
        f.elem_off[c] = (uint32_t)t.elem_off[k];
        f.slot_line[c] = (uint32_t)(t.slot_off[k] / 128u);
    }
    f.elem_off[kFewChunks] = (uint32_t)t.elem_off[t.n_chunks];
    return f;
}

/* Where chunk c of a launch lies, and its tiles: how many, and the number of the first among the launch's. */
struct ChunkPlace {
    uint64_t elem_off, n, slot_off;
    uint32_t tile, tiles;
};

ZIPCCL_HD ChunkPlace place_of(const ChunkTab& t, uint32_t c, int)
{
    return ChunkPlace{t.elem_off[c], t.elem_off[c + 1] - t.elem_off[c], t.slot_off[c], t.tile_start[c], t.tile_start[c + 1] - t.tile_start[c]};
}

ZIPCCL_HD ChunkPlace place_of(const EqualSplit& t, uint32_t c, int dt)
{
    const uint32_t tiles = (uint32_t)tiles_of(t.n);
    return ChunkPlace{(uint64_t)c * t.n, t.n, c * slot_layout(t.n, dt).cap, c * tiles, tiles};
}

ZIPCCL_HD ChunkPlace place_of(const FewSplit& t, uint32_t c, int)
{
    const uint64_t n = t.elem_off[c + 1] - t.elem_off[c];
    uint32_t tile = 0;
#pragma unroll
    for (uint32_t k = 0; k + 1u < kFewChunks; ++k)
        if (k < c) tile += (uint32_t)tiles_of((uint64_t)(t.elem_off[k + 1] - t.elem_off[k]));
    return ChunkPlace{t.elem_off[c], n, (uint64_t)t.slot_line[c] * 128u, tile, (uint32_t)tiles_of(n)};
}

/*
 * Chained compress: tiles tell one another their counts in 64-bit words, a count in the low 24 bits, the launch's tag in the others.
 * The tag of the launch of this number: 2^40 - 2 launches until one comes again, and neither 0 nor all ones, which the words of a
 * workspace that was cleared or filled hold.
 */
constexpr uint64_t kChainCount = 0xFFFFFFull;
constexpr uint64_t kChainTags = (1ull << 40) - 2u;
ZIPCCL_HD uint64_t chain_tag(uint64_t launch) { return (launch % kChainTags + 1u) * (kChainCount + 1u); }
ZIPCCL_HD bool chain_told(uint64_t word, uint64_t tag) { return (word ^ tag) <= kChainCount; }

struct CompressArgs {
    const uint8_t* in;       /* first element of the launch's first chunk */
    uint8_t* out;            /* compressed buffer base for this launch */
    uint64_t* chunk_bytes;   /* entry of the launch's first chunk, or null */
    uint32_t* tile_total;    /* one u32 per tile of this launch: its zero-point count */
    uint32_t* tile_prefix;   /* one u32 per tile: zero-points of its chunk before it */
    uint64_t* words;         /* chained form: one per tile of this launch */
    uint8_t* stash;          /* stash mode: one byte per input element of this launch (+ slack) */
    uint32_t dec_lo;         /* dec[0..3] packed little-endian: dec[1..7] are consecutive */
    const uint32_t* d_table; /* when not null: the table lives in device memory (two words), dec_lo unused */
    uint32_t table_stride;   /* words from one chunk's table to the next: 0 = one table for all chunks, 2 = one each */
    ChunkTab tab;
};

constexpr uint32_t kManyTiles = 8192;                /* of 8192 values: chained_pays, launch_chained_dt */

/*
 * Whether a call that is not captured compresses in the chained form rather than with a stash.  Always where the workspace has no room for
 * a stash, as the form without reads its input twice (us, twice / chained: 8 chunks of 21 * 2^20 values in all 26.4 / 17.6, 64 odd ones of
 * 120 million 117 / 77, 8 odd ones of 537 million 494 / 333).  Else not in launches of many bf16 tiles whose
 * chunks start off cache lines, where normal values lose by it, if rows with gains do not (us, with a stash / chained, normal values | rows with gains
 * among them | Student-t: 8 odd chunks of 70 million in all 48.2 / 50.7 | 53.5 / 52.2 | 49.2 / 50.9, of 120 million 75.7 / 77.1 | 80.3 / 78.7 | 77.0 / 77.2, of
 * 537 million 320.6 / 331.2 | 348.3 / 341.9 | 332.5 / 334.9; 64 of 120 million 76.5 / 77.1 | 83.4 / 78.7 | 78.6 / 77.5, of 300 million 180.3 / 185.1 |
 * 190.9 / 188.4 | 183.4 / 183.5).
 */
inline bool chained_pays(const CompressArgs& a, int dt)
{
    const uint32_t tiles = a.tab.tile_start[a.tab.n_chunks];
    if (a.stash == nullptr || dt != ZIPCCL_BF16) return true;
    uint64_t off = 0;
    if (tiles > kManyTiles) {
        off = reinterpret_cast<uintptr_t>(a.in) % 128u;
        for (uint32_t c = 0; c < a.tab.n_chunks; ++c) off |= a.tab.elem_off[c] * 2u % 128u;
    }
    return off == 0u;
}

constexpr uint32_t kPlaceScanTiles = 4096;            /* largest chunk (in tiles) for which k_place does the tile scan itself */
constexpr uint32_t kMomentBlocks = 2048;             /* workgroups (and partial sums) of the sigma estimate */

struct MomentArgs {
    const uint8_t* in;
    uint64_t n;
    double* partial;         /* 2 doubles per workgroup: sum d, sum d^2 with d = x - first value */
    uint32_t n_blocks;
    uint8_t* table;          /* device zipccl_table_t (8 bytes) */
    double* sigma;           /* may be null */
};

constexpr uint32_t kHistBlocks = 256;                /* workgroups of the robust estimate: one per compute unit */
constexpr uint32_t kHistBytes = 32768 * 8;           /* its workspace: one count per 15-bit magnitude, at most 64 bits each */

struct HistArgs {
    const uint8_t* in;       /* first element of the launch's first chunk */
    unsigned long long* hist;   /* the launch's first chunk's workspace, kHistBytes per chunk */
    uint32_t sample_stride;  /* 1: every value counts; a power of two S: one group of 512 values per S groups */
    uint8_t* table;          /* device zipccl_table_t (8 bytes) per chunk of the launch */
    double* sigma;           /* one per chunk of the launch; may be null */
    ChunkTab tab;            /* the launch's chunks (elem_off; the other fields are not used) */
};

/* Groups to count in the launch's largest chunk. */
ZIPCCL_HD uint64_t groups_to_count(const ChunkTab& t, uint32_t sample_stride)
{
    uint64_t largest = 0;
    for (uint32_t c = 0; c < t.n_chunks; ++c)
        if (t.elem_off[c + 1] - t.elem_off[c] > largest) largest = t.elem_off[c + 1] - t.elem_off[c];
    return ((largest + kGroup - 1) / kGroup + sample_stride - 1) / sample_stride;
}

/*
 * Whether one workgroup per chunk does it all in one kernel (k_robust_chunk_fused), or a windowed count in two (us, bf16, one / two): one chunk of 64 groups
 * to count 7.4 / 8.5, of 100 8.4 / 7.9, of 256 13 / 8.5; 8 chunks of 64 8.5 / 9.1, of 100 9.5 / 8.7, of 256 14 / 10.5; 64 chunks of 128 10.3 / 11.7, of 180
 * 13.0 / 12.7, of 448 22 / 17; 128 chunks of 180 13.7 / 15.3, of 448 22.9 / 22.1: the more chunks, the fewer workgroups are left for each of them.
 */
ZIPCCL_HD bool robust_in_one_kernel(const ChunkTab& t, uint32_t sample_stride)
{
    return groups_to_count(t, sample_stride) < (t.n_chunks <= 16u ? 100u : (t.n_chunks <= 64u ? 180u : 260u));
}

/* How the windowed count of a launch runs (k_window_count, k_window_finish). */
struct WindowPlan {
    uint32_t parts;          /* workgroups per chunk that count */
    uint32_t finish;         /* workgroups per chunk of the finish, and of a second count */
    bool wide;               /* the wide window */
    bool shared;             /* a second count goes to a histogram that the first kernel zeroes */
    bool stream;             /* loads past the caches */
};
constexpr uint32_t kWideParts = 16;                  /* workgroups per chunk up to which the window is the wide one */
constexpr uint32_t kManyChunks = 32, kManyChunksAlone = 2048;

ZIPCCL_HD WindowPlan window_plan(const ChunkTab& t, int dt, uint32_t sample_stride)
{
    WindowPlan p;
    const uint64_t groups = groups_to_count(t, sample_stride);
    /* two groups per wave at least (2^20 bf16 values 9.4 us, 10.4 with four), one workgroup per compute unit at most */
    const uint64_t want = (groups + 31) / 32, most = kHistBlocks / t.n_chunks;
    p.parts = (uint32_t)(want < 1 ? 1 : (want < most ? want : most));
    /* The wide window is never left by values that the narrow one loses 1 in 5 times (rows of scales spread by e^2), and where few
       workgroups share a chunk its counts are as quick to read.  us, bf16, tensors in turn, narrow / wide, normal values | rows spread by
       e^2: 64 chunks of 2^19 24.7 / 24.4 | 28.6 / 24.1, 8 of 2^21 from one group in 16 (8 workgroups each) 11.3 / 10.8 | 13.8 / 10.7; with 32 workgroups
       each normal values lose by it: 8 of 2^20 15.2 / 15.5 | 17.9 / 15.3, one of 2^19 10.8 / 11.1 | 13.1 / 10.8 */
    p.wide = p.parts <= kWideParts;
    /* 128 KiB zeroed per chunk are time in a launch of many small chunks (64 of 2^19 bf16 values 26.6 us with, 24.7 without), which fill the
       chip with one workgroup each should all of them be counted twice (64 of 2^20 110 us with, 95 without; 8 of 2^20 38 and 76) */
    p.shared = groups > (t.n_chunks >= kManyChunks ? kManyChunksAlone : kFusedGroups);
    /* workgroups for the case that the window does not hold the rank: most of the time they only start and end, which is worth
       a microsecond of a call on less than 2^25 values */
    p.finish = !p.shared ? 1u : (groups <= 65536u ? (p.parts + 7u) / 8u : p.parts);
    /* up to 64 MiB of counted values, 32 of sampled ones, stay in the caches for the compress that usually follows (us, estimate and compress, streamed
       loads / plain: 2^24 bf16 values 35.7 / 31.9, 64 experts of 512 x 7168 from one group in 16 156.0 / 152.6); larger tensors do
       not, and are read faster streamed (2^26: 33, 36; 64 MiB in scattered kilobytes, estimate alone, 25.9 / 28.8) */
    p.stream = t.elem_off[t.n_chunks] / sample_stride * elem_size(dt) > (sample_stride == 1u ? 64ull << 20 : 32ull << 20);
    return p;
}

struct DecompressArgs {
    const uint8_t* comp;
    uint64_t comp_capacity;  /* readable bytes from comp */
    uint8_t* out;
    uint32_t* status;        /* may be null */
    ChunkTab tab;
};

struct ReduceArgs {
    const uint8_t* comp;     /* n_peers slots of n values each, back to back */
    uint64_t comp_capacity;  /* readable bytes from comp */
    uint64_t slot_cap;       /* bytes from one slot to the next */
    uint8_t* out;            /* n sums */
    uint32_t* status;        /* may be null */
    uint64_t n;
    uint32_t n_peers;
    /* set by the launcher: */
    uint32_t gpw;            /* groups per wave in the workgroups that take whole tiles */
    uint32_t n_full;         /* how many those are: workgroups 0 .. n_full - 1 */
    uint32_t n_work;         /* workgroups that sum; one more may look at the slots' first index entries */
    uint32_t gpw_rest;       /* groups per wave in the workgroups after them, which take the rest of the shard */
};

/* kModeStash: single pass over the input; zero-point exponents go to a stash at a position that
 * does not depend on other tiles, and k_place moves them once the tile prefixes are known.
 * kModeCount + kModeEmit: the same without a stash, reading the input twice.
 * kModeDirect: one launch for small chunks; every workgroup counts the zero-points of its chunk's tiles before its own.
 * kModeChained: one launch; every workgroup adds up the counts that its chunk's tiles before have told. */
enum CompressMode { kModeCount = 0, kModeEmit = 1, kModeStash = 2, kModeDirect = 3, kModeChained = 4 };

/* launchers implemented next to their kernels (zipccl_compress.hip, zipccl_decompress.hip, zipccl_aux.hip);
 * they return a hipError_t as int */
int launch_estimate(int dt, const MomentArgs& a, void* stream);
int launch_estimate_robust(int dt, const HistArgs& a, void* stream);
int launch_compress(int dt, int mode, const CompressArgs& a, void* stream);
/* kModeChained, or kNotTaken and nothing is launched */
constexpr int kNotTaken = -1;
int launch_compress_chained(int dt, const CompressArgs& a, void* stream);
/* device address and size of the library's own workspace on the current GPU (zipccl_compress_static) */
int static_scratch(void** ptr, size_t* bytes);
int launch_tile_scan(const CompressArgs& a, void* stream);
int launch_place(int dt, bool scan, const CompressArgs& a, void* stream);
int launch_decompress(int dt, const DecompressArgs& a, void* stream);
int launch_decompress_reduce(int dt, int out_dt, const ReduceArgs& a, void* stream);

} // namespace zipccl
#endif
