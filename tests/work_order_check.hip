// Host check of the work order of short samples (va_device.h): every (item, head) once, whichever rotation the items'
// samples give, query heads of a group on the kv head's XCD, and the tiles of a sample on the same XCD where the order
// promises it.
#include <cstdio>
#include <set>
#include <utility>

#include "../paper_2605_08962_amd/csrc/va_device.h"

int main() {
    const int shapes[][3] = {{908, 16, 16}, {1, 16, 16}, {300, 32, 8}, {15, 8, 8}, {16, 8, 8}, {17, 24, 24},
                             {5, 6, 3}, {100, 12, 12}, {129, 20, 4}, {33, 1, 1}, {40, 64, 16}};
    int bad = 0;
    for (auto& sh : shapes)
        for (int D : {64, 80, 96, 128}) {
            const int n = sh[0], heads = sh[1], kv = sh[2];
            const bool whole = va::short_whole_items(D, kv);
            std::set<std::pair<int, int>> seen;
            for (unsigned bid = 0; bid < (unsigned)(n * heads); ++bid) {
                int item = -1, hp = -1;
                va::short_item_head(bid, n, heads, kv, D, item, hp);
                if (item < 0 || item >= n) { ++bad; continue; }
                const int sample = item / 3 * 384;  // samples of three tiles
                const int h = va::short_rotated_head(hp, item, sample, heads, kv, D);
                if (h < 0 || h >= heads || !seen.insert({item, h}).second) ++bad;
                const unsigned first = (unsigned)n / (8 * va::kShortRun) * (8 * va::kShortRun);
                if (whole && (unsigned)item < first && (unsigned)item / va::kShortRun % 8 != bid % 8) ++bad;
                // same sample, same kv head: the XCD depends on the kv head and the sample only
                const int unrotated = (int)(((unsigned)h + heads - ((unsigned)sample * 2654435761u >> 16) % heads) % heads);
                if (!whole && (unrotated % kv) % 8 != (int)(bid % 8)) ++bad;
            }
            if ((int)seen.size() != n * heads) ++bad;
            if (bad) { std::printf("n=%d heads=%d kv=%d D=%d: %d errors\n", n, heads, kv, D, bad); return 1; }
        }
    std::printf("work order ok\n");
    return 0;
}
