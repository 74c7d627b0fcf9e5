// The split rule of page lists (split_rule.h): never more splits than the merge asks for in one round trip.  Exit code 0: all hold.
#include <cstdio>

#include "split_rule.h"

int main()
{
    using namespace chess;
    for (int heads : {1, 4, 8})
        for (int group : {1, 4, 5, 7, 16})
            for (int tile_pages : {1, 2})
                for (int batch : {1, 2, 7, 32})
                    for (int64_t pages : {1, 16, 48, 49, 96, 97, 98, 400, 5000}) {
                        const SplitLimits c{256, 768, 256, heads, group, tile_pages, 0, 4};
                        const SplitShape s = choose_splits(c, batch, pages, true);
                        const int most = cdiv(pages, tile_pages) <= 48 ? 8 : group > 4 ? 12 : 16;
                        if (s.n_splits > most) {
                            std::printf("heads %d G %d tile pages %d batch %d pages %lld -> %d splits\n", heads, group, tile_pages, batch, (long long)pages, s.n_splits);
                            return 1;
                        }
                    }
    std::printf("ok\n");
    return 0;
}
