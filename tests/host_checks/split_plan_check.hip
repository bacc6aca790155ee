// Host-side check of the split plan's candidates (swaa::split_length, swaa::split_count): the first one splits nothing,
// however far off the approximate reciprocal is; of the dies' shares of the units (swaa::die_share) and of their order (swaa::unit_of_rank).  Built and run by tests/test_host_split_plan.py; needs no GPU.
#include <cstdio>
#include <cstring>

#include "swaa_fwd_split.h"

int main() {
    long bad = 0, checked = 0;
    auto ulps = [](float x, int n) {
        unsigned u;
        std::memcpy(&u, &x, 4);
        u += (unsigned)n;
        std::memcpy(&x, &u, 4);
        return x;
    };
    // longest sequences of 1 .. 2^20 halves (33 million keys): no sequence of the batch is split by candidate 0
    for (int h_max = 1; h_max <= 1 << 20; h_max += h_max < 4096 ? 1 : 37)
        for (int off = -2; off <= 2; ++off) {
            const int L = swaa::split_length(h_max, 0, ulps(1.f, off));
            for (int h : {1, h_max / 2, h_max - 1, h_max}) {
                ++checked;
                if (h < 1 || swaa::split_count(h, L, 1.f / (float)L) == 1) continue;
                if (bad++ < 10) std::printf("candidate 0: %d of %d halves, reciprocal %d ulps off: L = %d\n", h, h_max, off, L);
            }
        }
    // the others are at least the shortest split, and no longer than an exact quotient by more than one
    for (int h_max = 1; h_max <= 20000; h_max += 7)
        for (int i = 1; i < 64; ++i)
            for (int off = -1; off <= 1; ++off) {
                const int L = swaa::split_length(h_max, i, ulps(1.f / (float)(i + 1), off)), exact = (h_max + i) / (i + 1);
                ++checked;
                const int want = exact > swaa::kSplitMinHalves ? exact : swaa::kSplitMinHalves;
                if (L >= swaa::kSplitMinHalves && L <= want + 1 && L >= want - 1) continue;
                if (bad++ < 10) std::printf("candidate %d of %d halves: L = %d, not %d\n", i, h_max, L, want);
            }
    // the dies' shares: every unit once, and over sequences of as many units each no die gets more than one unit more
    for (unsigned units = 0; units <= 70; ++units) {
        unsigned of_die[swaa::kXcds] = {};
        for (unsigned b = 0; b < swaa::kSplitMaxBatch; ++b) {
            unsigned most = 0, least = ~0u;
            bool whole = swaa::die_share(units, b * units, 0) == 0 && swaa::die_share(units, b * units, swaa::kXcds) == units;
            for (unsigned x = 0; x < swaa::kXcds; ++x) {
                const int share = (int)(swaa::die_share(units, b * units, x + 1) - swaa::die_share(units, b * units, x));
                whole = whole && share >= 0 && share <= (int)((units + swaa::kXcds - 1) / swaa::kXcds);
                of_die[x] += (unsigned)share;
                most = of_die[x] > most ? of_die[x] : most;
                least = of_die[x] < least ? of_die[x] : least;
            }
            ++checked;
            if (whole && most - least <= 1) continue;
            if (bad++ < 10) std::printf("%u sequences of %u units: dies get %u to %u\n", b + 1, units, least, most);
        }
    }
    // the order on a die: every unit once, and no two row tiles on a compute unit (ranks r and r + 32) while one
    // of few rows could be there
    for (unsigned n_rows = 0; n_rows <= 140; ++n_rows)
        for (unsigned n_few = 0; n_few <= 140; ++n_few) {
            const unsigned n = n_rows + n_few, pairs = n <= 32 ? 0 : n <= 64 ? n - 32 : 32;
            bool seen[2][140] = {}, kind[280] = {}, sound = true;
            for (unsigned r = 0; r < n; ++r) {
                bool few;
                unsigned at;
                swaa::unit_of_rank(r, n_rows, n_few, few, at);
                sound = sound && at < (few ? n_few : n_rows) && !seen[few][at];
                if (sound) seen[few][at] = true;
                kind[r] = few;
            }
            unsigned rows_alone = 0;
            for (unsigned r = 0; r < pairs; ++r) rows_alone += !kind[r] && !kind[r + 32];
            sound = sound && rows_alone <= (n_few < pairs ? pairs - n_few : 0);
            ++checked;
            if (sound) continue;
            if (bad++ < 10) std::printf("%u row tiles, %u of few rows: %u compute units with two row tiles\n", n_rows, n_few, rows_alone);
        }
    std::printf("checked %ld cases, %ld wrong\n", checked, bad);
    return bad != 0;
}
