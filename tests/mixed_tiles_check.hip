// Host-side check of the tile order of launches with buckets of one row tile and of several (mixed_tile in csrc/ffn_tiles.h): every
// tile has one place, either kind keeps its order, and a launch whose plan asks for that order owns every tile once.
// Runs on the CPU: no HIP call is made.  Built and run by tests/test_mixed_tiles.py.
#include "ffn_tiles.h"

#include <cstdio>
#include <random>
#include <set>
#include <tuple>
#include <vector>

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

static int check_launch_of(std::mt19937& rng, int NT, int KT, int cpx, bool split) {
    const int BM = kShortTileRows, n_heavy = 1 + rng() % 4, n_light = 4 + rng() % 20, n = n_heavy + n_light;
    std::vector<int32_t> plan(kPlanInts, 0);
    int start = 0, row_tiles = 0, heavy_rows = 0;
    plan[0] = n;
    for (int i = 0; i < n; ++i) {
        const int rows = i < n_heavy ? BM + 1 + rng() % BM : 1 + rng() % BM, tiles = (rows + BM - 1) / BM;
        plan[kPlanExpert + i] = i;
        plan[kPlanStart + i] = start;
        plan[kPlanCount + i] = rows;
        plan[kPlanTiles1 + i] = row_tiles;
        start += rows;
        row_tiles += tiles;
        heavy_rows += i < n_heavy ? tiles : 0;
    }
    plan[kPlanTiles1 + n] = row_tiles;
    plan[kPlanMixed] = heavy_rows;
    std::set<std::tuple<int, int, int, int>> owned;
    const long long grid = ffn_grid(start, n, NT, BM, split, cpx);
    for (long long block = 0; block < grid; ++block) {
        WorkItem w;
        if (!workgroup_item(plan.data(), plan.data() + kPlanTiles1, NT, KT, BM, (unsigned)block, cpx, 8, split, w)) continue;
        CHECK(owned.insert(std::make_tuple(w.bucket, w.first, w.nt, w.kt0)).second, "bucket %d, row %d, column %d owned twice", w.bucket, w.first, w.nt);
    }
    std::set<std::tuple<int, int, int>> tiles;
    for (const auto& o : owned) tiles.insert(std::make_tuple(std::get<0>(o), std::get<1>(o), std::get<2>(o)));
    CHECK((long long)tiles.size() == (long long)row_tiles * NT, "%zu of %lld tiles owned", tiles.size(), (long long)row_tiles * NT);
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
    std::mt19937 rng(1);
    for (int NT : {1, 7, 8, 16, 112})
        for (int cpx : cpxs)
            for (bool split : {false, true})
                for (int i = 0; i < 20; ++i)
                    if (check_launch_of(rng, NT, 64, cpx, split)) return 1;
    std::printf("ok\n");
    return 0;
}
