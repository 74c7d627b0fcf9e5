// The split-K shape of the attention kernels: how many workgroups of how many waves share the pages of a sequence and KV
// head.  Host code without anything of the GPU in it (the CPU tests run it over the whole range of shapes).
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

namespace chess {

// n_slots > 0: the workgroups of a KV head, dealt to the sequences by length, at most n_splits to one
struct SplitShape { int n_splits, waves, n_slots; };

struct SplitLimits {
    int n_cu;
    int resident;           // four-wave workgroups of the dense kernel that fit on the device at once
    int max_splits;
    int n_kv_heads, group;
    int tile_pages;         // pages of a 32-token tile
    int force_splits, force_waves;   // test hook; force_splits 0 = automatic
};

constexpr int kDealMost = 4096;   // most sequences whose every-page attention is dealt by length

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline int64_t clampi(int64_t x, int64_t lo, int64_t hi) { return x < lo ? lo : (x > hi ? hi : x); }

// Rows of split partials a workspace for `rows` (sequence, KV head) pairs holds, in units of G vectors.
inline int64_t partial_rows(int n_cu, int64_t rows) { return 4LL * n_cu + rows; }

// The fused step with rows of its own (one workgroup each): whether its lean kernel, made for three workgroups a compute unit, is the
// one to launch.  Only where the rows outnumber two a compute unit; and not where the levels are so long that what they keep in
// LDS (`level_bytes`; allocated in pieces of 1280) leaves no room for three in 160 KB: two of the lean kind score with half the
// vectors in flight.  us a layer, lean / not: 80 sequences of 64K at a budget of 10 % 690 / 669, with bf16 vectors 566 / 519.  (A long
// page list, which also takes LDS, says nothing about the levels: 96 sequences of 30-32K at 1 % with room for 1950 pages 75.7 / 78.3.)
inline bool lean_step(int n_cu, int64_t rows, int64_t level_bytes)
{
    return rows > 2LL * n_cu && 3 * cdiv(level_bytes, 1280) * 1280 <= 160 * 1024;
}

// Most splits of a page list: what its tiles can use.  A split more costs the last workgroup requests (up to eight splits are
// one round trip, beyond that it asks for eight or sixteen at a time), and pays as long as waves have several tiles: eight splits
// for up to 48 tiles, sixteen (twelve with more than four query heads, where sixteen would fill the chip) for up to some 200; then as
// many as leave each of eight waves a tile, up to 2 sqrt(tiles), in eights.  us of attention over a list (8 / 16 / 24 / 32 / 64 splits,
// the better of four and eight waves):
//   one (sequence, head), G = 4, pages of 16    48 pages   6.1 /  6.6 /  7.3              150 pages   8.3 /  7.7 /  8.0 /  8.1
//                                              500 pages  15.6 / 11.9 / 11.2 / 10.6      4000 pages  99.7 / 55.1 / 40.6 / 33.0 / 23.9
//   eight, G = 4, pages of 16                  260 pages  11.7 / 10.5 / 11.7 / 12.4      1000 pages  32.6 / 21.9 / 20.5 / 20.7
//   one, G = 7, pages of 32                     90 pages   9.9 /  9.0 /  9.3 /  9.5       500 pages  27.9 / 18.4 / 16.0 / 14.9 / 15.3
// (A fixed most of 8 / 16 took 63 us of the 4000 pages and 133 of 4000 pages of 32.)
inline int64_t list_cap(const SplitLimits& c, int64_t pairs, int64_t tiles)
{
    if (tiles <= 48) return 8;
    const int64_t grown = std::min(tiles / 8, (int64_t)(2.0 * std::sqrt((double)tiles))) / 8 * 8;
    return std::max<int64_t>(c.group > 4 && 64 * pairs > 3LL * c.n_cu ? 12 : 16, grown);
}

// A workgroup has four waves (eight where `wide` below says so); tiles are dealt round-robin over splits and waves.
// Dense (every page): enough workgroups to cover the chip a few times over; the workgroup that finishes last merges
// ns partial rows per output, tile time falls as 1/ns and merge time grows as G*ns/32 (in units of one memory
// round trip), so the best split count is about sqrt(8*tiles/G), within what is resident at once.  With several
// sequences that count is the most one of them gets, and the workgroups resident at once are dealt to them by their
// lengths on the device (share_slots), as soon as there are more of them than sequences: only the device knows the
// lengths, and splits chosen for the longest possible one cost a short sequence more than the dealing does (times there).
// A page list: the fixed latencies dominate, and the measured optimum (sweeps at 1 .. 128 (sequence, head) pairs, 16 .. 12000
// pages, G = 1 .. 7, both page sizes) is: no split once there is a (sequence, head) per compute unit; otherwise one workgroup per
// compute unit, at least two tiles per workgroup, at most 1.6 x the merge-balanced count, and at most list_cap.
inline SplitShape choose_splits(const SplitLimits& c, int batch, int64_t max_list_pages, bool listed)
{
    const int64_t tiles = std::max<int64_t>(1, cdiv(max_list_pages, c.tile_pages));
    const int64_t pairs = (int64_t)batch * c.n_kv_heads;
    const int64_t room = partial_rows(c.n_cu, pairs);
    if (c.force_splits > 0) return {c.force_splits, c.force_waves == 8 && !listed ? 4 : c.force_waves, 0};
    const int waves = 4;
    const double balanced = std::sqrt(8.0 * (double)tiles / c.group);
    const int64_t limit = std::min<int64_t>(c.max_splits, 1024 / c.group);
    int64_t ns;
    if (listed) {
        ns = std::min<int64_t>(c.n_cu / pairs, cdiv(tiles, 2));
        ns = std::min<int64_t>(ns, (int64_t)std::llround(1.6 * balanced));
        ns = std::min<int64_t>(ns, list_cap(c, pairs, tiles));
        ns = std::max<int64_t>(ns, 1);
    } else {
        // all workgroups resident at once: a second round of workgroups would double a short kernel
        ns = (int64_t)std::llround(balanced);
        ns = std::min<int64_t>(ns, std::max<int64_t>(1, c.resident / pairs));
        ns = clampi(ns, 1, cdiv(tiles, waves));
        const int64_t most = clampi(std::llround(balanced), 1, std::min<int64_t>(cdiv(tiles, waves), limit));
        const int64_t slots = std::min<int64_t>(std::min<int64_t>(c.resident, room) / c.n_kv_heads, batch * most);
        if (batch > 1 && batch <= kDealMost && slots > batch) return {(int)most, waves, (int)slots};
    }
    ns = std::min<int64_t>(ns, limit);
    while (ns > 1 && pairs * ns > room) --ns;                      // stay inside the workspace
    // Eight waves for a list whose workgroups leave each compute unit at most one of four waves: a wave's chain of tiles
    // halves and the rows in flight double, with no exchange through memory, but a workgroup takes about 0.2 us longer
    // to start and to combine.  Four against eight waves over batch 1 .. 32, 8 .. 256 (sequence, head) pairs, G = 1 .. 16,
    // both page sizes, sparse decode and reuse step:
    //   more than four query heads and more than one split (the merge of G * ns rows is shared by twice the threads):
    //     eight are faster from the first tile beyond four waves' (0.81 - 0.97 x the time), level beyond 64 tiles a split;
    //   otherwise only when each of eight waves has a tile (below that 1.00 - 1.04 x; from there 0.95 - 1.00 x), and with
    //     tiles of two pages while none has more than four (beyond that 1.01 - 1.07 x; with one-page tiles the reuse step
    //     still gains 2 - 5 % there).
    // 32 sequences of 16-32K, 8 layers and the monitor: 139.8 -> 135.0 us.
    const bool big_merge = c.group > 4 && ns > 1;
    const bool wide = listed && pairs * ns <= c.n_cu &&
                      (big_merge ? tiles > 4 * ns : tiles >= 8 * ns && (c.tile_pages == 1 || tiles <= 32 * ns));
    return {(int)ns, wide ? 8 : waves, 0};
}

}  // namespace chess
