// Host-side check of the tile order of launches with buckets of one row tile and of several (mixed_tile in csrc/ffn_tiles.h): every
// tile has one place and either kind keeps its order.  tile_schedule_check.hip has whole launches in that order.
// Runs on the CPU: no HIP call is made.  Built and run by tests/test_mixed_tiles.py.
#include "ffn_tiles.h"

#include <cstdio>

using namespace moe;

#define CHECK(cond, ...)                                                            \
    do {                                                                            \
        if (!(cond)) {                                                              \
            std::printf("FAILED %s (line %d): ", #cond, __LINE__);                  \
            std::printf(__VA_ARGS__);                                               \
            std::printf("\n");                                                      \
            return 1;                                                               \
        }                                                                           \
    } while (0)

static int check_order(int heavy_rows, int light_rows, int q, int cpx) {
    const int n = (heavy_rows + light_rows) * q, heavy = heavy_rows * q;
    int next_heavy = 0, next_light = heavy;
    for (int idx = 0; idx < n; ++idx) {
        const int t = mixed_tile(heavy_rows, q, n, idx, cpx);
        if (t < heavy) CHECK(t == next_heavy++, "heavy %d light %d q %d cpx %d: place %d holds %d", heavy_rows, light_rows, q, cpx, idx, t);
        else CHECK(t == next_light++, "heavy %d light %d q %d cpx %d: place %d holds %d", heavy_rows, light_rows, q, cpx, idx, t);
    }
    CHECK(next_heavy == heavy && next_light == n, "heavy %d light %d q %d cpx %d: %d and %d placed", heavy_rows, light_rows, q, cpx, next_heavy, next_light);
    return 0;
}

int main() {
    const int qs[] = {1, 2, 14, 56}, cpxs[] = {4, 32, 38};
    for (int heavy : {1, 2, 5, 11, 40})
        for (int light : {1, 2, 5, 11, 12, 64, 200})
            for (int q : qs)
                for (int cpx : cpxs)
                    if (check_order(heavy, light, q, cpx)) return 1;
    if (check_order(2, 65533, 1, 32) || check_order(32767, 32768, 1, 32)) return 1;         // the largest lists that are mixed
    std::printf("ok\n");
    return 0;
}
