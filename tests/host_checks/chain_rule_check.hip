// Host-side check of what the rules for long rows count (swaa::pairs_of_rows, swaa::longest_row) against the mask's definition, and of
// calls that the forwards take or leave by them (swaa::plan_fwd_short, head dimension 128, and swaa::plan_fwd_d64_short).  Built and run by
// tests/test_host_chain_rule.py; needs no GPU.
#include <cstdio>

#include "swaa_fwd_d64.hip"
#include "swaa_fwd_short.hip"

int main() {
    long bad = 0, checked = 0;
    for (int N : {1, 2, 33, 70})
        for (int W = 1; W <= N; ++W)
            for (int S = 0; S <= N; ++S)
                for (int P = 0; P <= N; ++P) {
                    swaa::FwdParams p{};
                    p.Nq = p.Nk = N, p.W = W, p.S = S, p.P = P;
                    long long pairs = 0, longest = 0;
                    for (int i = 0; i < N; ++i) {
                        long long row = 0;
                        for (int j = 0; j <= i; ++j) row += i >= P || j > i - W || j < S;
                        pairs += row;
                        longest = row > longest ? row : longest;
                    }
                    ++checked;
                    if (swaa::pairs_of_rows(p) == (double)pairs && swaa::longest_row(p) == longest) continue;
                    if (bad++ < 10)
                        std::printf("N %d W %d S %d P %d: %lld pairs, not %.0f, longest row %lld, not %lld\n", N, W, S, P, pairs, swaa::pairs_of_rows(p), longest,
                                    swaa::longest_row(p));
                }
    struct Call {
        int B, Hkv, G, N, W, S, P;
        bool takes;
        int D = 128;
    };
    const Call calls[] = {
        {1, 8, 1, 20000, 1024, 4, 19488, true},      // generated rows behind a prompt
        {1, 8, 4, 16384, 128, 8192, 16383, false},   // as long as the others, which see the sinks
        {1, 8, 4, 8000, 512, 1000, 7999, false},     // 324 us on 32 rows of a head, 215 on row tiles
        {2, 8, 4, 16384, 128, 1000, 16320, false},   // 1162 / 695
        {1, 8, 1, 4001, 512, 4096, 4001, true},      // full attention, by its sinks
        {8, 4, 4, 2285, 67, 4, 2284, false},         // narrow windows: 120 / 57.9
        {8, 4, 4, 6124, 123, 4, 6119, false},        // 339 / 166
        {8, 8, 4, 1600, 123, 4, 1586, false, 64},    // 79.4 / 43.5
        // head dimension 64, as include/swaa.h says: up to 512 tiles, or 1536 if a row sees 256 keys
        {1, 8, 2, 1024, 40, 4, 1024, true, 64},
        {1, 8, 2, 1025, 40, 4, 1025, false, 64},
        {1, 8, 2, 1025, 252, 3, 1025, false, 64},
        {1, 8, 2, 1025, 252, 4, 1025, true, 64},
        {1, 8, 2, 1025, 40, 4, 1024, true, 64},
        {1, 8, 2, 3072, 300, 4, 3072, true, 64},
        {1, 8, 2, 3073, 300, 4, 3073, false, 64},
    };
    for (const Call &c : calls) {
        swaa::FwdParams p{};
        p.B = c.B, p.Hkv = c.Hkv, p.G = c.G, p.Hq = c.Hkv * c.G, p.Nq = p.Nk = c.N, p.W = c.W, p.S = c.S < c.N ? c.S : c.N, p.P = c.P;
        swaa::FwdShortParams sp;
        ++checked;
        if ((c.D == 64 ? swaa::plan_fwd_d64_short(p, sp) : swaa::plan_fwd_short(p, false, sp)) == c.takes) continue;
        ++bad;
        std::printf("B %d Hkv %d G %d N %d W %d S %d P %d D %d: on the other kernel\n", c.B, c.Hkv, c.G, c.N, c.W, c.S, c.P, c.D);
    }
    std::printf("checked %ld cases, %ld wrong\n", checked, bad);
    return bad != 0;
}
