// Host-side check of the plan of one packed sequence (swaa::plan_fwd_split): stating the number of rows decides whether there is a
// launch for splits at all, never whether or how often the keys are split.  Built and run by tests/test_host_split_plan.py; needs no GPU.
#include <cstdio>

#include "swaa_fwd_pipelined.hip"

int main() {
    long bad = 0, checked = 0, whole = 0, split = 0;
    for (int Hkv : {1, 2, 4, 8})
        for (int G : {1, 2, 4, 5, 8})
            for (int Nq : {1, 8, 33, 63, 64, 65, 200, 333, 512, 735, 1000, 2048})
                for (int Nk : {Nq + 1, 1100, 2500, 4000, 12000, 24000, 131072})
                    for (int W : {1, 500, 900, 1250, 1500, 2048, 2500, 3000, 4096, 8192, Nk})
                        for (int P : {Nk, Nk - Nq}) {
                            if (Nq > Nk) continue;
                            swaa::FwdParams by_rows[2] = {};
                            long long need[2];
                            bool planned = true;
                            for (int stated = 0; stated < 2; ++stated) {
                                swaa::FwdParams &p = by_rows[stated];
                                static const int offsets[2] = {0, 0};  // (only looked at for being there)
                                p.cu_q = p.cu_k = offsets;
                                p.B = 1, p.Hkv = Hkv, p.G = G, p.Hq = Hkv * G, p.Nq = Nq, p.Nk = Nk;
                                p.W = W < Nk ? W : Nk, p.S = 4, p.P = P;
                                planned = planned && (stated ? swaa::plan_work_packed(p, Nq, swaa::kFwdWgRows, Nq) : swaa::plan_work(p, Nq, swaa::kFwdWgRows));
                                need[stated] = swaa::plan_fwd_split(p);
                            }
                            if (!planned) continue;
                            const swaa::FwdParams &p = by_rows[0];
                            // splits of the sequence if it has Nq rows and Nk keys: the host's count, or by the device's rule for whole batches
                            const bool device_whole = swaa::whole_batch(p, Nq, swaa::least_units(p, Nq));
                            bool sound = need[1] > 0 ? need[0] > 0 && by_rows[1].bound_splits == p.bound_splits
                                                     : need[0] == 0 || (device_whole && p.bound_splits == 0);
                            // the launch has room for the row tiles, and for all partial results
                            for (int stated = 0; stated < 2; ++stated) {
                                const swaa::FwdParams &s = by_rows[stated];
                                if (need[stated] <= 0) continue;
                                const long long units = (long long)Hkv * swaa::split_seq(s, Nq, Nk, P).tiles;
                                sound = sound && s.split_cap >= units * s.bound_splits && s.chunk * swaa::kXcds >= units && s.chunk * swaa::kXcds >= s.split_cap;
                            }
                            whole += need[1] == 0 && need[0] > 0;
                            split += p.bound_splits > 1;
                            ++checked;
                            if (sound) continue;
                            if (bad++ < 10)
                                std::printf("Hkv %d G %d Nq %d Nk %d W %d P %d: %lld and %lld bytes, %d and %d splits, whole on the device %d\n", Hkv, G, Nq, Nk, W, P,
                                            need[0], need[1], p.bound_splits, by_rows[1].bound_splits, (int)device_whole);
                        }
    std::printf("checked %ld cases, %ld of them whole by the rows stated, %ld split by the host, %ld wrong\n", checked, whole, split, bad);
    return bad != 0 || !whole || !split;
}
