// Host check of the order in which a small launch takes its samples (csrc/va_small.h): longest first, equal ones in the
// batch's order, every place once, for up to 64 samples with empty ones among them; and of causal tiles, by falling cost.
#include <cstdio>
#include <set>
#include <utility>
#include <vector>

#include "../paper_2605_08962_amd/csrc/va_small.h"

int main() {
    unsigned state = 12345;
    auto next = [&](unsigned m) { state = state * 1664525u + 1013904223u; return (state >> 8) % m; };
    int bad = 0;
    for (int trial = 0; trial < 400; ++trial) {
        const int n = trial < 64 ? trial + 1 : 1 + (int)next(64);
        std::vector<int> len(n), at(n, -1);
        for (int& x : len) x = (int)next(trial % 3 == 0 ? 3 : 5000);
        for (int s = 0; s < n; ++s) {
            const int place = va::length_rank(n, s, len[s], [&](int i) { return len[i]; });
            if (place < 0 || place >= n || at[place] >= 0) { ++bad; continue; }
            at[place] = s;
        }
        for (int k = 1; k < n && !bad; ++k)
            if (len[at[k - 1]] < len[at[k]] || (len[at[k - 1]] == len[at[k]] && at[k - 1] > at[k])) ++bad;
        // a lane without a sample (length 0 behind the last) comes behind all of them
        if (va::length_rank(n, n, 0, [&](int i) { return len[i]; }) != n) ++bad;
        // causal tiles by falling cost: the idx-th of the batch, as the kernels find it, takes every tile once
        std::vector<int> tiles(n);
        int total = 0, most = 0;
        for (int s = 0; s < n; ++s) { tiles[s] = (len[s] + 127) / 128; total += tiles[s]; if (tiles[s] > most) most = tiles[s]; }
        auto from = [&](int v) { int k = 0; for (int x : tiles) k += x - v + 1 > 0 ? x - v + 1 : 0; return k; };
        std::set<std::pair<int, int>> seen;
        for (int idx = 0, last = most; idx < total; ++idx) {
            const int v = va::cost_level(idx, most, from), place = idx - from(v + 1);
            int s = -1, before = 0;
            for (int i = 0; i < n; ++i)
                if (tiles[i] >= v && before++ == place) s = i;
            if (s < 0 || v > last || v < 1 || !seen.insert({s, tiles[s] - v}).second) ++bad;
            last = v;
        }
        if ((int)seen.size() != total) ++bad;
        if (bad) { std::printf("n=%d: %d errors\n", n, bad); return 1; }
    }
    std::printf("length order ok\n");
    return 0;
}
