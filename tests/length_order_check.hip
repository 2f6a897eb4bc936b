// Host check of the order in which a small launch takes its samples (csrc/va_small.h): longest first, equal ones in the
// batch's order, every place once, for up to 64 samples with empty ones among them.
#include <cstdio>
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
        if (bad) { std::printf("n=%d: %d errors\n", n, bad); return 1; }
    }
    std::printf("length order ok\n");
    return 0;
}
