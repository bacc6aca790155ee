// Host-side check of the work list's order (swaa::work_place): whatever the plan, every row tile of every pair is one
// workgroup's and no workgroup has two; dies take a pair's tiles in turn only behind windows that
// make rows differ, and lists of one round with tiles of several kinds go pair after pair.  Built and run by tests/test_host_work_list.py; needs no GPU.
#include <cstdio>
#include <vector>

#include "swaa_common.h"

int main() {
    long bad = 0, checked = 0;
    for (int B : {1, 2, 3, 4, 5, 8, 16})
        for (int Hkv : {1, 2, 3, 4, 8, 12})
            for (int G : {1, 2, 4, 5, 7, 8})
                for (int rows : {1, 33, 128, 500, 1000, 2048, 2049, 6200, 9000})
                    for (int W : {64, rows / 9, rows / 6, rows / 2, rows})
                        for (int P : {rows, rows - 1})
                            for (int wg_rows : {128, 256})
                                for (bool fold : {true, false}) {
                                    swaa::FwdParams p{};
                                    p.B = B; p.Hkv = Hkv; p.G = G; p.Nq = p.Nk = rows; p.W = W > 0 ? W : 1; p.P = P;
                                    if (!swaa::plan_work(p, rows, wg_rows)) continue;
                                    if (!fold) p.fold = 0x7fffffff;
                                    std::vector<int> seen((size_t)p.total_items, 0);
                                    long items = 0;
                                    const bool mixed = (G > 3) + (G % 4 > 1) + G % 2 > 1;
                                    bool sound = (!mixed || p.chunk <= 44 || p.chunk >= 64 || p.die_pairs == 1) &&
                                                 (p.die_shift == 0 || (B * Hkv == 1 ? 4 : 8) * p.W >= rows);
                                    for (unsigned bid = 0; bid < (unsigned)(p.chunk * swaa::kXcds); ++bid) {
                                        unsigned pair, r;
                                        if (!swaa::work_place(p, bid, pair, r)) continue;
                                        sound = sound && pair < (unsigned)(B * Hkv) && r < (unsigned)p.tiles_per_pair;
                                        if (sound) sound = !seen[(size_t)pair * p.tiles_per_pair + r]++;
                                        ++items;
                                    }
                                    ++checked;
                                    if (sound && items == p.total_items) continue;
                                    if (bad++ < 10) std::printf("B %d Hkv %d G %d rows %d W %d P %d tile %d: %ld of %lld items\n", B, Hkv, G, rows, W, P, wg_rows, items, p.total_items);
                                }
    std::printf("checked %ld cases, %ld wrong\n", checked, bad);
    return bad != 0;
}
