// Runs the product's split rule (split_rule.h) over the range of shapes.  Exit code 0: all hold.
#include <cstdio>

#include "split_rule.h"

using namespace chess;

int main()
{
    for (int n_cu : {1, 64, 256, 304})
        for (int blocks : {1, 2, 3, 8})
            for (int heads : {1, 2, 4, 8, 16})
                for (int group : {1, 2, 4, 5, 7, 16})
                    for (int tile_pages : {1, 2})
                        for (int batch = 1; batch <= 1500; batch = batch < 40 ? batch + 1 : batch * 9 / 8)
                            for (int64_t pages = 1; pages <= 1 << 17; pages = pages < 24 ? pages + 1 : pages * 5 / 4)
                                for (bool listed : {false, true}) {
                                    const SplitLimits c{n_cu, blocks * n_cu, 256, heads, group, tile_pages, 0, 4};
                                    const SplitShape s = choose_splits(c, batch, pages, listed);
                                    const int64_t pairs = (int64_t)batch * heads, tiles = cdiv(pages, tile_pages), ns = s.n_splits;
                                    const int64_t used = s.n_slots > 0 ? (int64_t)s.n_slots * heads : pairs * ns;
                                    const char* bad = nullptr;
                                    if (ns < 1 || ns > 256 || ns * group > 1024) bad = "split count";
                                    else if ((ns > 1 || s.n_slots > 0) && used > partial_rows(n_cu, pairs)) bad = "partials outgrow the workspace";
                                    else if (s.n_slots > 0 && (listed || batch < 2 || batch > kDealMost || s.n_slots <= batch || used > blocks * n_cu)) bad = "dealt slots";
                                    else if (!listed && s.waves != 4) bad = "waves of every-page attention";
                                    else if (listed && ns > 1 && pairs * ns > n_cu) bad = "more list workgroups than compute units";
                                    else if (listed && s.waves == 8) {
                                        // eight waves only where they were faster than four (see split_rule.h)
                                        if (pairs * ns > n_cu) bad = "eight waves, shared compute units";
                                        else if (group > 4 && ns > 1) { if (tiles <= 4 * ns) bad = "eight waves without tiles for them"; }
                                        else if (tiles < 8 * ns) bad = "eight waves, fewer than eight tiles a split";
                                        else if (tile_pages == 2 && tiles > 32 * ns) bad = "eight waves, more than four tiles a wave";
                                    }
                                    if (bad != nullptr) {
                                        std::printf("%s: cu %d blocks %d heads %d G %d tile pages %d batch %d pages %lld listed %d -> ns %d waves %d slots %d\n",
                                                    bad, n_cu, blocks, heads, group, tile_pages, batch, (long long)pages, listed, s.n_splits, s.waves, s.n_slots);
                                        return 1;
                                    }
                                }
    // a forced shape is what it says, except that every-page attention has no eight-wave kernel
    for (int waves : {1, 4, 8})
        for (bool listed : {false, true}) {
            const SplitLimits c{256, 768, 256, 8, 4, 2, 3, waves};
            const SplitShape s = choose_splits(c, 4, 100, listed);
            if (s.n_splits != 3 || s.n_slots != 0 || s.waves != (waves == 8 && !listed ? 4 : waves)) { std::printf("forced shape\n"); return 1; }
        }
    std::printf("ok\n");
    return 0;
}
