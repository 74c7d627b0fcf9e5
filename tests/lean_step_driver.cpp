// Which launches of the fused step take the lean kernel (split_rule.h).  Exit code 0: all hold.
#include <cstdio>

#include "split_rule.h"

int main()
{
    using chess::lean_step;
    bool ok = !lean_step(256, 1, 40000) && !lean_step(256, 512, 40000);           // at most two workgroups a compute unit
    for (int64_t rows : {513, 768, 4096})
        for (int64_t bytes = 0; bytes <= 160 * 1024; bytes += 64) {
            int64_t fit = 0, used = 0;                                            // workgroups side by side, in pieces of 1280 bytes
            for (const int64_t each = (bytes + 1279) / 1280 * 1280; fit < 8 && used + each <= 160 * 1024; ++fit) used += each;
            ok = ok && lean_step(256, rows, bytes) == (fit >= 3);
        }
    if (ok) std::printf("ok\n");
    return ok ? 0 : 1;
}
