// Host-side check of the backward's plan (swaa::plan_bwd) and of the tiles its workgroups take (swaa::dkv_tiles): every row that
// sees a key of a key tile lies in exactly one query tile of one of that key tile's workgroups, the partial sums fit the
// workspace asked for, that is no more than include/swaa.h states, and the workgroups of whole key tiles (swaa::dkv_main_item) have
// each of them once.  Built and run by tests/test_host_bwd_plan.py; needs no GPU.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "swaa_bwd.hip"

namespace swaa {
hipError_t launch_bwd_dq_pipelined_d128(const BwdParams &, hipStream_t) { return hipErrorUnknown; }  // (never called here)
}  // namespace swaa

int main() {
    long bad = 0, checked = 0;
    for (int B : {1, 2, 8, 9, 16, 64, 65, 200})
        for (int Hkv : {1, 4, 8})
            for (int G : {1, 4})
                for (int N : {100, 129, 500, 1000, 4096, 6200})
                    for (int W : {1, 64, 256, 1000, N})
                        for (int S : {0, 4, 129, 1000, 4000})
                            for (int P : {N, N - 1, N / 2})
                                for (int D : {64, 128})
                                    for (bool pieces : {true, false}) {
                                        swaa::BwdParams p{};
                                        p.f.B = p.B = B; p.f.Hkv = p.Hkv = Hkv; p.f.Hq = p.Hq = G * Hkv; p.f.G = G;
                                        p.f.Nq = p.f.Nk = p.N = N;
                                        p.f.W = W < N ? W : N; p.f.S = S < N ? S : N; p.f.P = P;
                                        if (!swaa::plan_work(p.f, N, swaa::kWgRows)) continue;
                                        swaa::plan_bwd(p, D, pieces);
                                        const int n_kt = (N + 127) / 128, n_tiles = (N + swaa::kBq - 1) / swaa::kBq;
                                        bool sound = p.n_split >= 1 && p.n_seg >= 0 && (p.n_sink_kt == 0) == (p.n_seg == 0);
                                        long long parts = 0;
                                        for (int kt = 0; kt < n_kt && sound; ++kt) {
                                            const int k0 = kt * 128, k1 = k0 + 127 < N ? k0 + 127 : N - 1;
                                            std::vector<int> taken(n_tiles, 0);
                                            for (int seg = -1; seg < (kt < p.n_sink_kt ? p.n_seg : 0) && sound; ++seg) {
                                                const swaa::DkvTiles t = swaa::dkv_tiles(p, swaa::DkvItem{kt, 0, seg, 0});
                                                for (int i = 0; i < t.n && sound; ++i) {
                                                    sound = t.at(i) >= 0 && t.at(i) < n_tiles;
                                                    if (sound) ++taken[t.at(i)];
                                                }
                                            }
                                            for (int i = 0; i < n_tiles && sound; ++i) {
                                                const int r0 = i * swaa::kBq, r1 = r0 + swaa::kBq < N ? r0 + swaa::kBq - 1 : N - 1;
                                                // some row of the tile sees some key of the key tile
                                                const bool seen = r1 >= k0 && (r0 - p.f.W < k1 || k0 < p.f.S || r1 >= P);
                                                sound = taken[i] <= 1 && (taken[i] == 1 || !seen);
                                            }
                                            // (a key tile's slots begin where those of the one before end)
                                            if (p.parts(kt) > 0) sound = sound && p.first_part(0, kt) == parts;
                                            parts += p.parts(kt);
                                        }
                                        sound = sound && p.first_part(1, 0) == parts &&
                                                swaa::bwd_workspace_floats(p, D) >= (long long)B * Hkv * (G * (long long)N + parts * 2 * 128 * D);
                                        const long long T = (long long)B * Hkv * ((p.f.S + 127) / 128), few = T ? T + std::max(512LL, T) : 0;
                                        sound = sound && 4 * swaa::bwd_workspace_floats(p, D) <=
                                                             ((long long)B * Hkv * G * N + 3) / 4 * 16 + (pieces ? std::max(few, 1536LL) : few) * 1024 * D;
                                        if (p.n_split == 1) {
                                            const int pairs = B * Hkv, n_extra = pairs * p.n_sink_kt * p.n_seg;
                                            const unsigned n_main = (unsigned)(pairs * n_kt + 7) / 8 * 8;
                                            std::vector<int> dealt(pairs * n_kt, 0);
                                            for (unsigned i = 0; i < n_main; ++i) {
                                                const int id = swaa::dkv_main_item(p, (unsigned)n_extra + i, n_extra, n_main, n_kt);
                                                if (id >= 0 && id < pairs * n_kt) ++dealt[id];
                                            }
                                            for (int n : dealt) sound = sound && n == 1;
                                        }
                                        ++checked;
                                        if (sound) continue;
                                        if (bad++ < 10)
                                            std::printf("B %d Hkv %d G %d N %d W %d S %d P %d D %d pieces %d: %d sink tiles, %d segments of %d, split %d\n", B, Hkv, G,
                                                        N, W, S, P, D, (int)pieces, p.n_sink_kt, p.n_seg, p.seg_tiles, p.n_split);
                                    }
    std::printf("checked %ld cases, %ld wrong\n", checked, bad);
    return bad != 0;
}
