// Which dK/dV kernel of head dimension 128 does the backward run?  One line per call on standard input, B Hkv G N W S P and 0 or 1
// (may key tiles be cut into pieces?); one line out: pieces, segments, 1 for the eight-wave kernel (swaa::dkv_short).
// Built and run by tests/test_host_bwd_plan.py; needs no GPU.
#include <cstdio>

#include "swaa_bwd.hip"

namespace swaa {
hipError_t launch_bwd_dq_pipelined_d128(const BwdParams &, hipStream_t) { return hipErrorUnknown; }  // (never called here)
}  // namespace swaa

int main() {
    int B, Hkv, G, N, W, S, P, pieces;
    while (std::scanf("%d %d %d %d %d %d %d %d", &B, &Hkv, &G, &N, &W, &S, &P, &pieces) == 8) {
        swaa::BwdParams p{};
        p.f.B = p.B = B; p.f.Hkv = p.Hkv = Hkv; p.f.Hq = p.Hq = G * Hkv; p.f.G = G;
        p.f.Nq = p.f.Nk = p.N = N;
        p.f.W = W < N ? W : N; p.f.S = S < N ? S : N; p.f.P = P < N ? P : N;
        if (!swaa::plan_work(p.f, N, swaa::kWgRows)) return 1;
        swaa::plan_bwd(p, 128, pieces != 0);
        std::printf("%d %d %d\n", p.n_split, p.n_seg, (int)swaa::dkv_short(p));
    }
    return 0;
}
