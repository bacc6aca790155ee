// Host-side check of the masks that the forward and dQ kernels apply to 32 keys at once (swaa::visible_keys) against
// the comparisons of the mask's definition.  Built and run by tests/test_host_visible_keys.py; needs no GPU.
#include <cstdio>

#include "swaa_common.h"

int main() {
    long bad = 0, checked = 0;
    auto check = [&](int k0, int qpos, int W, int S) {
        const unsigned bits = swaa::visible_keys(k0, qpos, W, S);
        for (int j = 0; j < 32; ++j, ++checked) {
            const int key = k0 + j;
            const bool sees = key <= qpos && (key > qpos - W || key < S);
            if (sees != ((bits >> j & 1u) != 0u)) {
                if (bad < 10) std::printf("mismatch: key %d row %d W %d S %d\n", key, qpos, W, S);
                ++bad;
            }
        }
    };
    const int lengths[] = {0, 1, 2, 31, 32, 33, 63, 64, 65, 100, 200};
    for (int base : {0, 1 << 20, 0x7fffff00 - 512})  // (positions stay below 2^31)
        for (int half = 0; half < 6; ++half)
            for (int row = 0; row < 200; ++row)
                for (int W : lengths)
                    for (int S : lengths)
                        if (W > 0) check(base + 32 * half, base + row, W, S ? base + S : 0);
    for (int half = 0; half < 6; ++half)  // a window as long as the sequence, and longer than any
        for (int row = 0; row < 200; ++row)
            for (int W : {200, 0x7fffffff - 200}) check(32 * half, row, W, 0);
    std::printf("checked %ld pairs, %ld wrong\n", checked, bad);
    return bad != 0;
}
