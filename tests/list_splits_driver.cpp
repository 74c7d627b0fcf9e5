// The split rule of page lists (split_rule.h) against measured ranges: for each list, the split counts whose time was within some
// 6 % of the best one's, from sweeps on 256 compute units.  And over the range of shapes: no split without two tiles, none
// beyond a workgroup per compute unit, and waves that have many tiles only where the chip is full.  Exit code 0: all hold.
#include <cstdio>

#include "split_rule.h"

using namespace chess;

struct Range { int heads, batch, group, tile_pages; int64_t room; int from, to; };   // room: entries of a list's row

int main()
{
    const Range measured[] = {
        {1, 1, 4, 2, 64, 8, 12},    {1, 1, 4, 2, 106, 12, 16},  {1, 1, 4, 2, 166, 12, 24},  {1, 1, 4, 2, 276, 16, 32},  {1, 1, 4, 2, 516, 24, 48},
        {1, 1, 4, 2, 1016, 32, 64}, {1, 1, 4, 2, 2016, 48, 96}, {1, 1, 4, 2, 4016, 64, 128}, {1, 1, 4, 2, 12016, 128, 200},
        {4, 1, 4, 2, 516, 16, 48},  {4, 1, 4, 2, 1016, 32, 48}, {4, 1, 4, 2, 4016, 48, 64},
        {8, 1, 4, 2, 42, 6, 8},     {8, 1, 4, 2, 106, 8, 16},   {8, 1, 4, 2, 276, 16, 16},  {8, 1, 4, 2, 516, 16, 32},  {8, 1, 4, 2, 1016, 24, 32}, {8, 1, 4, 2, 4016, 24, 32},
        {8, 2, 4, 2, 516, 12, 16},  {8, 4, 4, 2, 516, 6, 8},    {8, 16, 4, 2, 516, 2, 2},   {8, 32, 4, 2, 516, 1, 1},
        {1, 1, 1, 2, 516, 24, 48},  {1, 1, 1, 2, 4016, 64, 128}, {8, 1, 1, 2, 1016, 24, 32},
        {1, 1, 7, 1, 106, 16, 24},  {1, 1, 7, 1, 276, 24, 48},  {1, 1, 7, 1, 516, 32, 64},  {1, 1, 7, 1, 4016, 96, 146}, {4, 1, 7, 1, 1016, 32, 64},
        {4, 4, 7, 1, 106, 8, 12},
    };
    for (const Range& r : measured) {
        const SplitLimits c{256, 768, 256, r.heads, r.group, r.tile_pages, 0, 4};
        const SplitShape s = choose_splits(c, r.batch, r.room, true);
        if (s.n_splits < r.from || s.n_splits > r.to) {
            std::printf("heads %d batch %d G %d tile pages %d room %lld -> %d splits, measured best %d to %d\n", r.heads, r.batch, r.group, r.tile_pages, (long long)r.room,
                        s.n_splits, r.from, r.to);
            return 1;
        }
    }
    for (int heads : {1, 2, 4, 8})
        for (int group : {1, 4, 5, 7, 16})
            for (int tile_pages : {1, 2})
                for (int batch : {1, 2, 7, 32, 200})
                    for (int64_t room = 1; room <= 1 << 20; room = room < 24 ? room + 1 : room * 5 / 4) {
                        const SplitLimits c{256, 768, 256, heads, group, tile_pages, 0, 4};
                        const SplitShape s = choose_splits(c, batch, room, true);
                        const int64_t tiles = cdiv(room, tile_pages), pairs = (int64_t)heads * batch, ns = s.n_splits;
                        const char* bad = nullptr;
                        if (ns > 1 && (2 * ns > tiles + 1 || pairs * ns > c.n_cu)) bad = "too many splits";
                        // with room for twice the workgroups: sixteen tiles a wave at most, or as many splits as the merge can have
                        else if (2 * pairs * ns <= c.n_cu && 2 * ns * group <= 1024 && tiles > 16 * ns * s.waves) bad = "idle compute units";
                        if (bad != nullptr) {
                            std::printf("%s: heads %d G %d tile pages %d batch %d room %lld -> %d splits of %d waves\n", bad, heads, group, tile_pages, batch, (long long)room,
                                        s.n_splits, s.waves);
                            return 1;
                        }
                    }
    std::printf("ok\n");
    return 0;
}
