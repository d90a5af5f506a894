/*
 * Sanitizer driver for the host side of libzipccl.so (csrc/zipccl_host.cpp): built with g++ under
 * -fsanitize=address,undefined together with stand-ins for the kernel launchers (no HIP, no GPU), and run by
 * tests/test_sanitizers.py.  It calls the pure-host entry points (table, sizes, offsets, switcher) on exact-size
 * host arrays, and the device entry points with arguments that must be rejected before anything is launched;
 * calls that pass the checks reach the stand-in launchers, which verify the geometry they are handed.
 */
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "zipccl_internal.h"

#define CHECK(c) do { if (!(c)) { std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)

namespace zipccl {

static int g_launches = 0;

/* the geometry every launch is handed must be consistent: tiles ascending, offsets ascending */
static void check_tab(const ChunkTab& t)
{
    CHECK(t.n_chunks >= 1 && t.n_chunks <= kMaxBatch);
    for (uint32_t c = 0; c < kMaxBatch; ++c) {
        CHECK(t.tile_start[c] <= t.tile_start[c + 1]);
        CHECK(t.elem_off[c] <= t.elem_off[c + 1]);
        CHECK(t.slot_off[c] <= t.slot_off[c + 1]);
        CHECK(t.slot_off[c] % ZIPCCL_ALIGN == 0);
    }
}

/* and the short forms of it that kernels are handed must say the same */
static int g_equal = 0, g_few = 0;
static void check_forms(const ChunkTab& t, int dt)
{
    const bool equal = is_equal_split(t), few = is_few_split(t);
    for (uint32_t c = 0; c < t.n_chunks; ++c) {
        const ChunkPlace want = place_of(t, c, dt);
        CHECK(want.n == t.elem_off[c + 1] - t.elem_off[c] && want.tiles == tiles_of(want.n));
        if (equal) {
            const ChunkPlace p = place_of(equal_split(t), c, dt);
            CHECK(p.elem_off == want.elem_off && p.n == want.n && p.slot_off == want.slot_off && p.tile == want.tile && p.tiles == want.tiles);
        }
        if (few) {
            const ChunkPlace p = place_of(few_split(t), c, dt);
            CHECK(p.elem_off == want.elem_off && p.n == want.n && p.slot_off == want.slot_off && p.tile == want.tile && p.tiles == want.tiles);
        }
    }
    g_equal += equal;
    g_few += few;
}

int launch_estimate(int, const MomentArgs& a, void*) { CHECK(a.n_blocks >= 1 && a.n_blocks <= kMomentBlocks); ++g_launches; return 0; }
/* one kernel, a workgroup per chunk; or two, whose workgroups and windows must fit the device and a chunk's workspace */
static int g_one_kernel = 0, g_wide = 0, g_narrow = 0, g_shared = 0, g_alone = 0;
int launch_estimate_robust(int dt, const HistArgs& a, void*)
{
    CHECK(a.tab.n_chunks >= 1 && a.tab.n_chunks <= kMaxBatch);
    CHECK(a.sample_stride >= 1 && a.sample_stride <= ZIPCCL_MAX_SAMPLE_STRIDE && (a.sample_stride & (a.sample_stride - 1)) == 0);
    for (uint32_t c = 0; c < kMaxBatch; ++c) CHECK(a.tab.elem_off[c] <= a.tab.elem_off[c + 1]);
    ++g_launches;
    uint64_t groups = 0;
    for (uint32_t c = 0; c < a.tab.n_chunks; ++c) {
        const uint64_t of = ((a.tab.elem_off[c + 1] - a.tab.elem_off[c] + kGroup - 1) / kGroup + a.sample_stride - 1) / a.sample_stride;
        groups = of > groups ? of : groups;
    }
    CHECK(groups_to_count(a.tab, a.sample_stride) == groups);
    if (robust_in_one_kernel(a.tab, a.sample_stride)) {
        CHECK(groups <= kFusedGroups);
        ++g_one_kernel;
        return 0;
    }
    const WindowPlan p = window_plan(a.tab, dt, a.sample_stride);
    CHECK(p.parts >= 1 && p.parts * a.tab.n_chunks <= kHistBlocks && p.finish >= 1 && p.finish <= p.parts);
    CHECK(p.wide == (p.parts <= kWideParts) && p.parts * (p.wide ? 2048u : 512u) <= kHistBytes / 2);
    CHECK(p.shared ? groups > kFusedGroups : (p.finish == 1 && groups <= kManyChunksAlone));
    ++(p.wide ? g_wide : g_narrow);
    ++(p.shared ? g_shared : g_alone);
    return 0;
}
/* kModeDirect has no workgroup wait for another: every one counts the tiles before its own, so they have to be few */
static int g_by_mode[4];
int launch_compress(int dt, int mode, const CompressArgs& a, void*)
{
    check_tab(a.tab);
    check_forms(a.tab, dt);
    if (mode == kModeDirect)
        for (uint32_t c = 0; c < a.tab.n_chunks; ++c)
            CHECK(a.tab.tile_start[c + 1] - a.tab.tile_start[c] <= (dt == ZIPCCL_BF16 ? 8u : 4u));
    if (mode == kModeStash) CHECK(a.stash != nullptr);
    ++g_by_mode[mode];
    ++g_launches;
    return 0;
}
/* kModeChained: not on a stream that is being captured, here where g_chains is not set; the words are 8 bytes per tile */
static bool g_chains = false, g_pays = false;
static int g_chained = 0;
int launch_compress_chained(int dt, const CompressArgs& a, void*)
{
    check_tab(a.tab);
    check_forms(a.tab, dt);
    CHECK(a.words != nullptr && reinterpret_cast<uintptr_t>(a.words) % 8 == 0);
    g_pays = chained_pays(a, dt);
    if (!g_chains) return kNotTaken;
    ++g_chained;
    ++g_launches;
    return 0;
}
int launch_tile_scan(const CompressArgs& a, void*) { check_tab(a.tab); ++g_launches; return 0; }
int launch_place(int, bool, const CompressArgs& a, void*) { check_tab(a.tab); ++g_launches; return 0; }
int launch_decompress(int dt, const DecompressArgs& a, void*) { check_tab(a.tab); check_forms(a.tab, dt); ++g_launches; return 0; }
int launch_decompress_reduce(int, int, const ReduceArgs& a, void*) { CHECK(a.n_peers >= 1 && a.n_peers <= kMaxPeers); ++g_launches; return 0; }
int static_scratch(void** ptr, size_t* bytes)
{
    static uint64_t fake[4];                        /* never dereferenced: the stand-in launchers touch no buffer */
    *ptr = fake;
    *bytes = ZIPCCL_STATIC_SCRATCH_BYTES;
    return 0;
}

/* The check of a group's two index entries; and what a wave of the fused reduce fetches of a slot's zero-point list for three consecutive index entries, whatever a
 * damaged stream holds in their place: every 16-byte read of the 64 lanes (and the last piece) lies between the 16
 * bytes in front of the list and its padded end, and entries that are not ascending positions of the list, at most a
 * group apart, are bad. */
static void check_pair_slices()
{
    const uint32_t ends[] = {0u, 1u, 13u, 30u, 512u, 1024u, 1040u, 100000u, 0x7FFFFFFFu, 0xFFFFFFFFu};
    const int64_t near[] = {0, 1, 14, 15, 16, 17, 511, 512, 513, 1007, 1008, 1009, 1023, 1024, 1025, 1040};
    for (uint32_t n_esc : ends) {
        std::vector<uint32_t> at;                     /* entries around 0, around n_esc and just below 2^32 */
        for (int64_t d : near)
            for (int64_t v : {d, (int64_t)n_esc - d, (int64_t)n_esc + d, ((int64_t)1 << 32) - 1 - d})
                if (v >= 0 && v <= 0xFFFFFFFFll) at.push_back((uint32_t)v);
        for (uint32_t base : at) {
            for (uint32_t next : at) {
                CHECK((slice_bad(base, next, n_esc, true) == 0u) == (base <= next && next <= n_esc && next - base <= kGroup));
                if (base <= next) CHECK(slice_bad(base, next, n_esc, false) == slice_bad(base, next, n_esc, true));
            }
        }
        const int64_t list_end = (int64_t)pad128(n_esc);
        for (uint32_t base : at) {
            for (uint32_t mid : at) {
                for (uint32_t next : at) {
                    const PairSlices s = pair_slices(base, mid, next, n_esc);
                    const bool good = base <= mid && mid <= next && next <= n_esc && mid - base <= kGroup && next - mid <= kGroup;
                    CHECK((s.bad == 0u) == good);
                    for (uint32_t lane = 0; lane < 64; ++lane) {
                        const int64_t off = -16 + (int64_t)s.from + (int64_t)pair_list_offset(s, lane);
                        CHECK(off >= -16 && off % 16 == 0 && off + 16 <= (list_end > 0 ? list_end : 0));
                    }
                    if (pair_has_last_piece(s)) CHECK((int64_t)s.from + kPairLastPiece + 16 <= list_end);
                    if (!good) continue;              /* the lanes' pieces cover the slice */
                    const uint32_t fetched = pair_has_last_piece(s) ? kPairLastPiece + 16u : kPairLastPiece;
                    CHECK(s.mis + s.count_a + s.count_b <= fetched && s.from + s.mis == base && s.count_a + s.count_b == next - base);
                    if (next != base) CHECK(s.span == next - s.from);
                }
            }
        }
    }
}

} // namespace zipccl

int main()
{
    using namespace zipccl;
    check_pair_slices();
    /* table builder over a wide sigma range, clamps and rejections */
    zipccl_table_t t;
    for (int k = -1100; k <= 1100; ++k) {
        const double s = std::ldexp(1.37, k);
        if (!(s > 0.0) || std::isinf(s)) continue;
        CHECK(zipccl_build_table(s, ZIPCCL_BF16, &t) == ZIPCCL_OK);
        CHECK(t.dec[1] >= 1 && t.dec[1] <= 248 && t.dec[7] == t.dec[1] + 6);
    }
    CHECK(zipccl_build_table(0.0, ZIPCCL_BF16, &t) == ZIPCCL_ERR_INVALID_ARG);
    CHECK(zipccl_build_table(NAN, ZIPCCL_BF16, &t) == ZIPCCL_ERR_INVALID_ARG);
    CHECK(zipccl_build_table(INFINITY, ZIPCCL_FP32, &t) == ZIPCCL_ERR_INVALID_ARG);
    CHECK(zipccl_build_table(1.0, ZIPCCL_BF16, nullptr) == ZIPCCL_ERR_INVALID_ARG);
    CHECK(zipccl_build_table(1.0, (zipccl_dtype_t)9, &t) == ZIPCCL_ERR_UNSUPPORTED_DTYPE);
    CHECK(zipccl_build_table(1.0, ZIPCCL_BF16, &t) == ZIPCCL_OK && t.dec[1] == 122);

    /* sizes and offsets: exact-size arrays, more chunks than one launch holds, empty chunks, bad splits */
    const uint32_t C = 300;
    std::vector<uint64_t> ce(C), off(C + 1), st(C);
    uint64_t n = 0;
    for (uint32_t c = 0; c < C; ++c) { ce[c] = (c * 7919u) % 20000u * (c % 5 != 0); n += ce[c]; }
    CHECK(zipccl_chunk_slot_offsets(n, ZIPCCL_FP32, C, ce.data(), off.data()) == ZIPCCL_OK);
    CHECK(zipccl_chunk_static_bytes(n, ZIPCCL_FP32, C, ce.data(), st.data()) == ZIPCCL_OK);
    CHECK(zipccl_max_compressed_size(n, ZIPCCL_FP32, C, ce.data()) == off[C]);
    for (uint32_t c = 0; c < C; ++c) CHECK(off[c] % 128 == 0 && st[c] <= off[c + 1] - off[c]);
    CHECK(zipccl_max_compressed_size(n + 1, ZIPCCL_FP32, C, ce.data()) == 0);
    CHECK(zipccl_max_compressed_size(10, ZIPCCL_BF16, 3, nullptr) == 0);
    CHECK(zipccl_max_compressed_size(10, ZIPCCL_BF16, 0, nullptr) == 0);
    ce[0] = ZIPCCL_MAX_CHUNK_ELEMS + 1;
    CHECK(zipccl_chunk_slot_offsets(n, ZIPCCL_FP32, C, ce.data(), off.data()) == ZIPCCL_ERR_INVALID_ARG);
    ce[0] = ~0ull; ce[1] = 2;                                         /* a sum that wraps */
    CHECK(zipccl_max_compressed_size(1, ZIPCCL_BF16, C, ce.data()) == 0);
    ce[0] = 0; ce[1] = (1 * 7919u) % 20000u;
    CHECK(zipccl_compress_workspace_size(n, ZIPCCL_FP32, C, ce.data()) > zipccl_compress_min_workspace_size(n, ZIPCCL_FP32, C, ce.data()));

    /* device entry points: rejected arguments never reach a launcher; accepted ones hand over consistent geometry.
       The pointers are only compared and aligned, never dereferenced by the stand-ins. */
    alignas(256) static uint8_t in[64], out[256], ws[256];
    const size_t big = (size_t)1 << 40;
    CHECK(zipccl_build_table(1.0, ZIPCCL_BF16, &t) == ZIPCCL_OK);
    g_launches = 0;
    CHECK(zipccl_compress(nullptr, 8, ZIPCCL_BF16, 1, nullptr, &t, out, big, nullptr, ws, big, nullptr) == ZIPCCL_ERR_INVALID_ARG);
    CHECK(zipccl_compress(in + 1, 8, ZIPCCL_BF16, 1, nullptr, &t, out, big, nullptr, ws, big, nullptr) == ZIPCCL_ERR_INVALID_ARG);
    CHECK(zipccl_compress(in, 8, ZIPCCL_BF16, 1, nullptr, &t, out + 64, big, nullptr, ws, big, nullptr) == ZIPCCL_ERR_INVALID_ARG);
    CHECK(zipccl_compress(in, 8, ZIPCCL_BF16, 1, nullptr, &t, out, 100, nullptr, ws, big, nullptr) == ZIPCCL_ERR_BUFFER_TOO_SMALL);
    CHECK(zipccl_compress(in, 8, ZIPCCL_BF16, 1, nullptr, &t, out, big, nullptr, ws, 16, nullptr) == ZIPCCL_ERR_BUFFER_TOO_SMALL);
    zipccl_table_t bad = t; bad.dec[3] = 7;
    CHECK(zipccl_compress(in, 8, ZIPCCL_BF16, 1, nullptr, &bad, out, big, nullptr, ws, big, nullptr) == ZIPCCL_ERR_INVALID_ARG);
    CHECK(zipccl_compress(in, 8, ZIPCCL_BF16, 1, nullptr, nullptr, out, big, nullptr, ws, big, nullptr) == ZIPCCL_ERR_INVALID_ARG);
    CHECK(zipccl_decompress(out, 100, in, 8, ZIPCCL_BF16, 1, nullptr, nullptr, nullptr) == ZIPCCL_ERR_BUFFER_TOO_SMALL);
    CHECK(zipccl_decompress(out + 1, big, in, 8, ZIPCCL_BF16, 1, nullptr, nullptr, nullptr) == ZIPCCL_ERR_INVALID_ARG);
    CHECK(zipccl_decompress_reduce(out, big, in, 8, ZIPCCL_BF16, 0, ZIPCCL_FP32, nullptr, nullptr) == ZIPCCL_ERR_INVALID_ARG);
    CHECK(zipccl_decompress_reduce(out, big, in, 8, ZIPCCL_BF16, 1025, ZIPCCL_FP32, nullptr, nullptr) == ZIPCCL_ERR_INVALID_ARG);
    CHECK(zipccl_decompress_reduce(out, 100, in, 8, ZIPCCL_BF16, 2, ZIPCCL_FP32, nullptr, nullptr) == ZIPCCL_ERR_BUFFER_TOO_SMALL);
    CHECK(zipccl_estimate_table(in, 8, ZIPCCL_BF16, (zipccl_table_t*)out, nullptr, ws, 8, nullptr) == ZIPCCL_ERR_BUFFER_TOO_SMALL);
    CHECK(zipccl_estimate_table_robust(in, 8, ZIPCCL_BF16, (zipccl_table_t*)out, nullptr, ws, 8, nullptr) == ZIPCCL_ERR_BUFFER_TOO_SMALL);
    CHECK(zipccl_compress_static(in, (size_t)16 << 31, ZIPCCL_BF16, 16, nullptr, &t, out, big * 1024, nullptr, nullptr) == ZIPCCL_ERR_BUFFER_TOO_SMALL);
    CHECK(g_launches == 0);
    /* accepted calls, with the 300-chunk split (three launches' worth of chunk tables) */
    CHECK(zipccl_compress(in, n, ZIPCCL_FP32, C, ce.data(), &t, out, big, nullptr, ws, big, nullptr) == ZIPCCL_OK);
    CHECK(zipccl_compress(in, n, ZIPCCL_FP32, C, ce.data(), &t, out, big, nullptr, ws,
                          zipccl_compress_min_workspace_size(n, ZIPCCL_FP32, C, ce.data()), nullptr) == ZIPCCL_OK);
    CHECK(zipccl_compress_static(in, n, ZIPCCL_FP32, C, ce.data(), &t, out, big, nullptr, nullptr) == ZIPCCL_OK);
    /* which form a compress takes: small chunks one kernel whatever the workspace, launch by launch; a chunk of more tiles
       the stash or, in the minimum workspace, two reads */
    auto forms = [&](zipccl_dtype_t dt, std::vector<uint64_t> split, bool least, int direct, int stash_launches, int emit) {
        uint64_t total = 0;
        for (uint64_t k : split) total += k;
        for (int& m : g_by_mode) m = 0;
        const uint32_t k = (uint32_t)split.size();
        const size_t ws_bytes = least ? zipccl_compress_min_workspace_size(total, dt, k, split.data()) : big;
        CHECK(zipccl_compress(in, total, dt, k, split.data(), &t, out, big, nullptr, ws, ws_bytes, nullptr) == ZIPCCL_OK);
        CHECK(g_by_mode[kModeDirect] == direct && g_by_mode[kModeStash] == stash_launches);
        CHECK(g_by_mode[kModeCount] == emit && g_by_mode[kModeEmit] == emit);
    };
    const uint64_t T = kTile;
    for (bool least : {false, true}) {
        const int s = least ? 0 : 1, e = least ? 1 : 0;
        forms(ZIPCCL_BF16, {8 * T}, least, 1, 0, 0);
        forms(ZIPCCL_BF16, {8 * T + 1}, least, 0, s, e);
        forms(ZIPCCL_FP32, {4 * T, 0, 1}, least, 1, 0, 0);
        forms(ZIPCCL_FP32, {4 * T + 1}, least, 0, s, e);
        forms(ZIPCCL_BF16, std::vector<uint64_t>(8, 8 * T), least, 1, 0, 0);
        forms(ZIPCCL_BF16, std::vector<uint64_t>(9, 8 * T), least, 0, s, e);
        forms(ZIPCCL_BF16, std::vector<uint64_t>(128, 4 * T), least, 1, 0, 0);
        forms(ZIPCCL_FP32, std::vector<uint64_t>(32, 4 * T), least, 1, 0, 0);
        forms(ZIPCCL_FP32, std::vector<uint64_t>(33, 4 * T), least, 0, s, e);
        std::vector<uint64_t> mixed(129, T);                          /* the second launch holds the one large chunk */
        mixed[128] = 9 * T;
        forms(ZIPCCL_BF16, mixed, least, 1, s, e);
    }
    /* and the chained form wherever it can be taken, but for chunks of one or two tiles, in either workspace */
    g_chains = true;
    for (bool least : {false, true}) {
        auto chained = [&](zipccl_dtype_t dt, std::vector<uint64_t> split, int direct, int want) {
            g_chained = 0;
            forms(dt, split, least, direct, 0, 0);
            CHECK(g_chained == want);
        };
        chained(ZIPCCL_BF16, {2 * T}, 1, 0);
        chained(ZIPCCL_BF16, {2 * T + 1}, 0, 1);
        chained(ZIPCCL_FP32, std::vector<uint64_t>(64, T), 1, 0);
        chained(ZIPCCL_FP32, std::vector<uint64_t>(32, 2 * T), 1, 0);
        chained(ZIPCCL_FP32, std::vector<uint64_t>(33, 2 * T), 0, 1);
        chained(ZIPCCL_BF16, std::vector<uint64_t>(128, 2 * T), 1, 0);
        chained(ZIPCCL_BF16, {0xFFFFFFFFull, 0xFFFFFFFFull}, 0, 1);
        std::vector<uint64_t> mixed(129, T);
        mixed[128] = 3 * T;
        chained(ZIPCCL_BF16, mixed, 1, 1);
    }
    /* where it pays: not for many bf16 tiles of chunks that start off cache lines, if there is room for a stash */
    for (bool least : {false, true}) {
        auto pays = [&](zipccl_dtype_t dt, std::vector<uint64_t> split, bool want) {
            forms(dt, split, least, 0, 0, 0);
            CHECK(g_pays == (want || least));
        };
        pays(ZIPCCL_BF16, {(kManyTiles - 1) * T - 1, T}, true);
        pays(ZIPCCL_BF16, {kManyTiles * T / 2 + 1, kManyTiles * T / 2 + 63}, false);
        pays(ZIPCCL_BF16, {kManyTiles * T / 2 + 64, kManyTiles * T / 2 + 64, 1}, true);
        pays(ZIPCCL_FP32, {kManyTiles * T / 2 + 1, kManyTiles * T / 2 + 63}, true);
        for (uint64_t tiles : {2048u, 2049u, 2304u, 2305u, 8191u}) {
            const uint64_t split[2] = {tiles * T - 77, 77};
            CHECK(zipccl_compress_device_table(in, tiles * T, ZIPCCL_BF16, 2, split, (const zipccl_table_t*)out, out, big, nullptr, ws,
                                               least ? zipccl_compress_min_workspace_size(tiles * T, ZIPCCL_BF16, 2, split) : big, nullptr) == ZIPCCL_OK);
            CHECK(g_pays);
        }
    }
    g_chains = false;
    /* a launch's tag: one of 2^40 - 2, from which what cleared and filled words hold differs as well as its neighbours' */
    for (uint64_t base : {0ull, 1ull << 24, (1ull << 40) - 4u, 1ull << 40, 0xFFFFFFFFFFFFFFF0ull})
        for (uint64_t k = base; k < base + 8u; ++k) {
            const uint64_t tag = chain_tag(k);
            CHECK((tag & kChainCount) == 0 && chain_told(tag, tag) && chain_told(tag | kChainCount, tag));
            for (uint64_t other : {(uint64_t)0, ~(uint64_t)0, chain_tag(k + 1u), chain_tag(k + 1u) | kChainCount}) CHECK(!chain_told(other, tag));
        }
    /* the short forms of the chunk table (check_forms): equal splits, given as such or chunk by chunk, and a few uneven chunks */
    const int equal0 = g_equal, few0 = g_few;
    for (zipccl_dtype_t dt : {ZIPCCL_BF16, ZIPCCL_FP32})
        for (uint32_t k : {1u, 2u, 7u, 8u, 9u, 128u, 130u})
            for (uint64_t each : {0ull, 1ull, 511ull, 512ull, 8191ull, 8192ull, 8193ull, 65537ull, 0x20000000ull, 0xFFFFFFFFull}) {
                std::vector<uint64_t> split(k, each);
                CHECK(zipccl_decompress(out, SIZE_MAX / 2, in, each * k, dt, k, nullptr, nullptr, nullptr) == ZIPCCL_OK);
                CHECK(zipccl_decompress(out, SIZE_MAX / 2, in, each * k, dt, k, split.data(), nullptr, nullptr) == ZIPCCL_OK);
                uint64_t total = 0;
                for (uint32_t c = 0; c < k; ++c) total += split[c] = (each >> (c % 5)) + c % 3;
                if (each < 0xFFFFFFFFull)
                    CHECK(zipccl_decompress(out, SIZE_MAX / 2, in, total, dt, k, split.data(), nullptr, nullptr) == ZIPCCL_OK);
            }
    CHECK(g_equal - equal0 >= 2 * 2 * 7 * 10 && g_few - few0 >= 2 * 2 * 4 * 9);
    CHECK(zipccl_decompress(out, big, in, n, ZIPCCL_FP32, C, ce.data(), nullptr, nullptr) == ZIPCCL_OK);
    CHECK(zipccl_decompress_reduce(out, big, in, 5000, ZIPCCL_BF16, 1024, ZIPCCL_BF16, nullptr, nullptr) == ZIPCCL_OK);
    CHECK(zipccl_estimate_table(in, 100000, ZIPCCL_BF16, (zipccl_table_t*)out, nullptr, ws, big, nullptr) == ZIPCCL_OK);
    CHECK(zipccl_estimate_table_robust(in, 100000, ZIPCCL_BF16, (zipccl_table_t*)out, nullptr, ws, big, nullptr) == ZIPCCL_OK);
    CHECK(zipccl_estimate_chunk_tables(in, n, ZIPCCL_FP32, C, ce.data(), (zipccl_table_t*)out, nullptr, ws, big, nullptr) == ZIPCCL_OK);
    for (zipccl_dtype_t dt : {ZIPCCL_BF16, ZIPCCL_FP32})
        for (uint32_t k : {1u, 2u, 7u, 8u, 9u, 16u, 17u, 31u, 32u, 64u, 65u, 127u, 128u, 130u})
            for (uint64_t groups : {0ull, 1ull, 99ull, 100ull, 179ull, 180ull, 259ull, 260ull, 508ull, 509ull, 1024ull, 1025ull, 2048ull, 2049ull, 65536ull, 65537ull, 0x7FFFFFull})
                for (uint32_t stride : {1u, 16u, 4096u}) {
                    std::vector<uint64_t> split(k, groups * kGroup / 2);
                    split[k / 2] = groups * kGroup;
                    uint64_t total = 0;
                    for (uint64_t v : split) total += v;
                    CHECK(zipccl_estimate_chunk_tables_sampled(in, total, dt, k, split.data(), stride, (zipccl_table_t*)out, nullptr, ws, SIZE_MAX / 2, nullptr) == ZIPCCL_OK);
                }
    CHECK(g_one_kernel && g_wide && g_narrow && g_shared && g_alone);
    CHECK(zipccl_estimate_chunk_tables(in, n, ZIPCCL_FP32, C, ce.data(), (zipccl_table_t*)out, nullptr, ws, 1000, nullptr) == ZIPCCL_ERR_BUFFER_TOO_SMALL);
    CHECK(zipccl_estimate_chunk_tables(in, n + 1, ZIPCCL_FP32, C, ce.data(), (zipccl_table_t*)out, nullptr, ws, big, nullptr) == ZIPCCL_ERR_INVALID_ARG);
    for (uint32_t stride : {1u, 2u, 16u, 4096u})
        CHECK(zipccl_estimate_chunk_tables_sampled(in, n, ZIPCCL_FP32, C, ce.data(), stride, (zipccl_table_t*)out, nullptr, ws, big, nullptr) == ZIPCCL_OK);
    for (uint32_t stride : {0u, 3u, 48u, 8192u, 0x80000000u})
        CHECK(zipccl_estimate_chunk_tables_sampled(in, n, ZIPCCL_FP32, C, ce.data(), stride, (zipccl_table_t*)out, nullptr, ws, big, nullptr) == ZIPCCL_ERR_INVALID_ARG);
    CHECK(zipccl_compress_chunk_tables(in, n, ZIPCCL_FP32, C, ce.data(), (const zipccl_table_t*)out, out, big, nullptr, ws, big, nullptr) == ZIPCCL_OK);
    CHECK(zipccl_compress_chunk_tables(in, n, ZIPCCL_FP32, C, ce.data(), nullptr, out, big, nullptr, ws, big, nullptr) == ZIPCCL_ERR_INVALID_ARG);
    CHECK(g_launches > 0);

    /* switcher */
    zipccl_link_model_t m{1e-5, 1e-10, 2e-5, 1e-10};
    double a = 0, b = 0;
    CHECK(zipccl_switch_prefers_zipped(&m, 1e9, 0.7, 1.0, &a, &b) == 1 && b < a);
    CHECK(zipccl_switch_prefers_zipped(&m, 1e3, 0.7, 1.0, nullptr, nullptr) == 0);
    CHECK(zipccl_switch_prefers_zipped(nullptr, 1e3, 0.7, 1.0, nullptr, nullptr) == -1);
    CHECK(zipccl_switch_prefers_zipped(&m, NAN, 0.7, 1.0, nullptr, nullptr) == -1);
    const double ds[4] = {1e6, 2e6, 4e6, 8e6}, ts[4] = {1.1e-3, 2.1e-3, 4.1e-3, 8.1e-3};
    CHECK(zipccl_fit_link_model(ds, ts, 4, &a, &b) == ZIPCCL_OK && std::fabs(a - 1e-4) < 1e-9 && std::fabs(b - 1e-9) < 1e-15);
    CHECK(zipccl_fit_link_model(ds, ts, 1, &a, &b) == ZIPCCL_ERR_INVALID_ARG);
    const double same[2] = {5.0, 5.0};
    CHECK(zipccl_fit_link_model(same, ts, 2, &a, &b) == ZIPCCL_ERR_INVALID_ARG);
    for (int s = 0; s <= 6; ++s) CHECK(zipccl_status_string((zipccl_status_t)s) != nullptr);
    std::puts("host sanitizer driver: ok");
    return 0;
}
