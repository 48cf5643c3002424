// Host-side exhaustive check of the grouped GEMM's work distribution (csrc/ffn_tiles.h): for random tile plans
// and launch shapes, walk every workgroup id of the launch exactly as the kernels do and verify that every
// (bucket, row tile, column tile, k tile) is owned exactly once, that partial-tile slots are unique and inside
// their XCD's range, that the fix-up finds exactly the split tiles with their parts in k order, and that the
// grid the host launches is large enough.  Runs on the CPU: no HIP call is made.
// Built and run by tests/test_tile_schedule.py.
#include "ffn_tiles.h"

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <map>
#include <random>
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

struct Part { int bucket, mt, nt, kt0, kt1; };

static long long mixed_launches = 0, mixed_cuts = 0;      // launches whose plan spreads buckets of one row tile among the others; with parts of such tiles

// Receives that were measured with their segments apart and merged (us): merged where that was the faster way.
static int check_measured_merges() {
    struct Measured { MergeShape m; Buckets apart, merged; bool streaming, merge; };
    const MergeShape fine = {11, 32, 8, 22, 32}, mixtral = {112, 64, 16, 224, 32};
    const Measured table[] = {
        {fine, {17, 27}, {3, 211}, false, false},        // 54 / 94
        {fine, {23, 99}, {10, 786}, false, false},       // 65 / 93
        {fine, {30, 39}, {9, 289}, false, false},        // 80 / 95
        {fine, {37, 53}, {9, 402}, false, true},         // 96 / 92
        {fine, {28, 21}, {11, 81}, false, true},         // 77 / 70
        {fine, {47, 40}, {8, 150}, false, true},         // 119 / 82
        {fine, {167, 2428}, {118, 19338}, false, true},  // 522 / 460
        {mixtral, {8, 40}, {2, 144}, false, true},       // 313 / 176
        {mixtral, {8, 147}, {5, 287}, false, true},      // 422 / 390
        {fine, {15, 9}, {6, 58}, true, false},           // 48 / 59
        {fine, {17, 7}, {9, 23}, true, true},            // 55 / 51
        {fine, {17, 9}, {12, 18}, true, false},          // 56 / 59
        {fine, {20, 7}, {13, 13}, true, true},           // 62 / 56
        {fine, {28, 18}, {12, 70}, true, false},         // 82 / 88
        {fine, {27, 27}, {16, 53}, true, true},          // 96 / 90
        {fine, {24, 15}, {9, 110}, true, true},          // 74 / 65
        {fine, {17, 12}, {4, 94}, true, true},           // 54.5 / 52
        {mixtral, {4, 4}, {3, 6}, true, false},          // 195 / 231
        {mixtral, {5, 4}, {4, 6}, true, true},           // 280 / 258
        {mixtral, {8, 10}, {2, 32}, true, true},         // 304 / 164
    };
    for (const Measured& c : table)
        CHECK(merge_pays(c.m, c.apart, c.merged, c.streaming) == c.merge, "%d tiles, at most %d rows, to %d, at most %d", c.apart.tiles,
              c.apart.max_rows, c.merged.tiles, c.merged.max_rows);
    return 0;
}

#ifdef WITH_ROUND_SPLIT
static long long chosen_cuts = 0, cut_launches = 0;

// round_split's choice (csrc/ffn_plan.h), candidate after candidate
static RoundCut choose(const RoundShape& r) {
    RoundCut best = round_candidate(r, 0);
    for (int c = 1; c < kRoundCandidates; ++c) best = better_cut(best, round_candidate(r, c));
    if (best.big == 0) return best;
    const RoundCut even = even_cut(r);
    if (!(launch_cost(r, best.big, best.small, best.rounds) < launch_cost(r, even.big, even.small, even.rounds) + kSearchCost)) best.big = 0;
    return best;
}

// Launches that were measured both ways: cut by cost only where that was the faster way (down projection of 256 compute
// units, us, even split or uncut / cut).
static int check_measured_choices() {
    struct Measured { int nb, ns, NT, KT; bool cut; };
    const Measured table[] = {
        {8, 4, 16, 112, false},    // d 4096, f 7168, 1000 tokens: 157 / 181
        {7, 4, 16, 112, false},    // ... 927 tokens: 159 / 174
        {8, 4, 16, 56, false},     // f 3584, 1000 tokens: 89 / 107
        {8, 4, 16, 224, false},    // f 14336, 1000 tokens: 296 / 312
        {5, 6, 16, 56, false},     // f 3584, 846 tokens: 82 / 85
        {5, 6, 16, 224, true},     // f 14336, 700 tokens: 288 / 266
        {5, 6, 16, 112, true},     // f 7168, 777 tokens: 153 / 145
        {3, 6, 8, 64, true},       // d 2048, f 4096, 600 tokens: 72 / 54
        {8, 4, 8, 64, true},       // ... 1000 tokens: 80 / 70
        {12, 11, 4, 64, true},     // d 1024, f 4096, 16 experts, 1500 tokens: 83 / 58
        {7, 4, 10, 42, true},      // d 2432, f 2688, 4 of 32 experts, 4000 tokens: 65 / 56 (the split is the same, it need not be searched)
        {0, 4, 16, 224, true},     // f 14336, 4 of 8 experts, 300 tokens: 102 / 97
    };
    for (const Measured& m : table) {
        const RoundCut c = choose(round_shape(m.nb, m.ns, m.NT, m.KT, 32));
        CHECK((c.big > 0) == m.cut, "%d big and %d small row tiles, NT %d, KT %d: cut (%d, %d)", m.nb, m.ns, m.NT, m.KT, c.big, c.small);
    }
    return 0;
}
#endif

static int check_case(std::mt19937& rng, long long& units) {
    const int bms[2] = {256, 384};
    const int nts[10] = {1, 2, 5, 8, 11, 16, 23, 32, 57, 112};
    const int kts[8] = {4, 9, 22, 32, 64, 100, 224, 448};
    const int cpxs[4] = {32, 38, 48, 4};
    const bool by_size = rng() % 2;                       // of buckets listed by size, as build_plan (csrc/ffn_plan.h) does, whose rule then says whether tiles are mixed
    const int BM = by_size ? kShortTileRows : bms[rng() % 2], NT = nts[rng() % 10], KT = kts[rng() % 8], cpx = cpxs[rng() % 4];
    const int row_chunk = (rng() % 2) ? 8 : 4;
    const bool split = rng() % 2;
    const int n = 1 + (int)(rng() % ((rng() % 8 == 0) ? 256 : 12));
    std::vector<int32_t> plan(kPlanInts, 0);
    std::vector<int> start(n), count(n), tiles(n);
    long long N = 0;
    for (int i = 0; i < n; ++i) {
        const int kind = rng() % 4;
        count[i] = kind == 0 ? 1 + rng() % 40 : (kind == 1 ? 1 + rng() % 400 : (kind == 2 ? 1 + rng() % 3000 : BM * (1 + rng() % 4)));
        if (n > 64) count[i] = 1 + rng() % 300;
    }
    if (by_size) {
        for (int i = 2; i < n; ++i) count[i] = 1 + count[i] % BM;        // mostly buckets of one row tile
        std::sort(count.begin(), count.end(), std::greater<int>());
    }
    for (int i = 0; i < n; ++i) {
        start[i] = (int)N + (int)(rng() % 3);            // gaps between buckets are allowed
        N = start[i] + count[i];
        tiles[i] = (count[i] + BM - 1) / BM;
    }
    plan[0] = n;
    int32_t* prefix = plan.data() + kPlanTiles0;
    int mt_total = 0;
    for (int i = 0; i < n; ++i) {
        plan[kPlanExpert + i] = 1000 + i;                 // any id: the check maps it back
        plan[kPlanStart + i] = start[i];
        plan[kPlanCount + i] = count[i];
        prefix[i] = mt_total;
        mt_total += tiles[i];
    }
    prefix[n] = mt_total;
    if (by_size) {
        const int single = (int)std::count_if(count.begin(), count.end(), [&](int c) { return c <= BM; });
        plan[kPlanMixed] = mixed_rows(mt_total, single);
        CHECK(plan[kPlanMixed] == (single >= mt_total - single ? prefix[n - single] : 0), "%d of %d row tiles by themselves: %d", single, mt_total, plan[kPlanMixed]);
    }
    const bool mixed = plan[kPlanMixed] > 0 && NT >= kXcds;
#ifdef WITH_ROUND_SPLIT
    // tiles of more than 128 rows and the others cut apart: as the plan would choose, or else into any numbers of parts that fit two per compute unit
    int n_small = 0;
    for (int i = 0; i < n; ++i) n_small += (count[i] - 1) % kShortTileRows < kSmallTileRows ? 1 : 0;
    if (BM == kShortTileRows) {
        const RoundShape r = round_shape(mt_total - n_small, n_small, NT, KT, cpx);
        const RoundCut chosen = choose(r);
        if (r.nbx + r.nsx <= cpx) {
            const int even = xcd_share(mt_total, NT, 0, KT, cpx, true).split;
            CHECK(even_cut(r).big == even, "even split priced as %d parts, run as %d", even_cut(r).big, even);
        }
        int big = 1 + rng() % kMaxSplit, small = 1 + rng() % kMaxSplit;
        if (chosen.big > 0) {
            big = chosen.big;
            small = chosen.small;
            ++chosen_cuts;
        }
        const bool fits = r.nbx + r.nsx <= cpx && r.nbx * big + r.nsx * small <= 2 * cpx && (big == 1 || KT / big >= kMinSplitKT) && (small == 1 || KT / small >= kMinSplitKT);
        CHECK(fits || chosen.big == 0, "cut (%d, %d) of %d and %d tiles on %d compute units, %d k tiles", big, small, r.nbx, r.nsx, cpx, KT);
        if (fits) {
            plan[kPlanSmallTiles] = 1 + n_small;
            plan[kPlanBigParts] = big;
            plan[kPlanSmallParts] = small;
            if (split) ++cut_launches;
        }
    }
#endif

    const long long grid = ffn_grid((int)N, n, NT, BM, split, cpx);
    CHECK(grid > 0 && grid < (1ll << 31), "grid %lld", grid);
    std::map<std::tuple<int, int, int>, std::vector<char>> covered;
    std::map<int, Part> partial_of;
    long long active = 0;
    for (long long block = 0; block < grid + 64; ++block) {      // a few ids past the grid must find no work either
        WorkItem w;
        if (!workgroup_item(plan.data(), prefix, NT, KT, BM, (unsigned)block, cpx, row_chunk, split, w)) continue;
        CHECK(block < grid, "work at block %lld beyond the launched grid %lld (BM %d NT %d KT %d cpx %d n %d split %d)", block, grid, BM, NT, KT, cpx, n, (int)split);
        ++active;
        const int i = w.expert - 1000;
        CHECK(i >= 0 && i < n, "expert %d", w.expert);
        const int off = w.row0 - start[i];
        CHECK(off >= 0 && off % BM == 0, "row0 %d of bucket %d", w.row0, i);
        const int mt = off / BM;
        CHECK(mt < tiles[i], "row tile %d of %d", mt, tiles[i]);
        const int want_rows = count[i] - mt * BM < BM ? count[i] - mt * BM : BM;
        CHECK(w.rows == want_rows && w.rows > 0, "rows %d, want %d", w.rows, want_rows);
        CHECK(w.nt >= 0 && w.nt < NT, "column tile %d of %d", w.nt, NT);
        CHECK(0 <= w.kt0 && w.kt0 < w.kt1 && w.kt1 <= KT, "k range %d..%d of %d", w.kt0, w.kt1, KT);
        const int x = (int)(block % kXcds);
        if (w.partial < 0) {
            CHECK(w.kt0 == 0 && w.kt1 == KT, "a whole tile with k range %d..%d", w.kt0, w.kt1);
        } else {
            CHECK(split, "partial tile without a split launch");
            CHECK(w.partial >= x * 2 * cpx && w.partial < (x + 1) * 2 * cpx, "slot %d outside XCD %d's range", w.partial, x);
            CHECK(!partial_of.count(w.partial), "slot %d used twice", w.partial);
            CHECK(w.kt1 - w.kt0 >= kMinSplitKT, "k part of %d tiles", w.kt1 - w.kt0);
            partial_of[w.partial] = Part{i, mt, w.nt, w.kt0, w.kt1};
        }
        auto& c = covered[std::make_tuple(i, mt, w.nt)];
        if (c.empty()) c.assign(KT, 0);
        for (int kt = w.kt0; kt < w.kt1; ++kt) {
            CHECK(!c[kt], "k tile %d of (bucket %d, row tile %d, column tile %d) owned twice", kt, i, mt, w.nt);
            c[kt] = 1;
            ++units;
        }
    }
    for (int i = 0; i < n; ++i)
        for (int mt = 0; mt < tiles[i]; ++mt)
            for (int nt = 0; nt < NT; ++nt) {
                auto it = covered.find(std::make_tuple(i, mt, nt));
                CHECK(it != covered.end(), "tile (bucket %d, row tile %d, column tile %d) has no owner (BM %d NT %d KT %d cpx %d n %d split %d)", i, mt, nt, BM, NT, KT, cpx, n, (int)split);
                for (int kt = 0; kt < KT; ++kt) CHECK(it->second[kt], "k tile %d of (%d, %d, %d) has no owner", kt, i, mt, nt);
            }
    CHECK((long long)covered.size() == (long long)mt_total * NT, "%zu tiles owned, %lld exist", covered.size(), (long long)mt_total * NT);

    // the fix-up: every split tile exactly once, its parts in consecutive slots and in k order from 0 to KT
    size_t parts_seen = 0;
    std::map<std::tuple<int, int, int>, int> fixed;
    for (int x = 0; x < kXcds; ++x)
        for (int q = 0; q < cpx; ++q) {                  // the host launches cpx fix-up tiles per XCD
            WorkItem w;
            int first = -1, parts = 0;
            if (!fixup_item(plan.data(), prefix, NT, KT, BM, x, q, cpx, row_chunk, w, first, parts)) continue;
            CHECK(split || partial_of.empty(), "fix-up work although nothing was split");
            if (!split) continue;                        // a launch without split never runs the fix-up's result: its tiles were written whole
            const int i = w.expert - 1000, mt = (w.row0 - start[i]) / BM;
            CHECK(++fixed[std::make_tuple(i, mt, w.nt)] == 1, "tile fixed up twice");
            int at = 0;
            for (int p = 0; p < parts; ++p) {
                auto it = partial_of.find(first + p);
                CHECK(it != partial_of.end(), "fix-up reads slot %d that nobody wrote", first + p);
                const Part& pt = it->second;
                CHECK(pt.bucket == i && pt.mt == mt && pt.nt == w.nt, "slot %d belongs to another tile", first + p);
                CHECK(pt.kt0 == at, "parts out of k order");
                at = pt.kt1;
                ++parts_seen;
            }
            CHECK(at == KT, "parts end at k tile %d of %d", at, KT);
        }
    if (split) CHECK(parts_seen == partial_of.size(), "%zu parts fixed up, %zu written", parts_seen, partial_of.size());
    mixed_launches += mixed;
    mixed_cuts += mixed && plan[kPlanBigParts] == 0 && !partial_of.empty();
    (void)active;
    return 0;
}

int main(int argc, char** argv) {
    const int cases = argc > 1 ? std::atoi(argv[1]) : 2000;
    std::mt19937 rng(20250209);
    long long units = 0;
#ifdef WITH_ROUND_SPLIT
    if (check_measured_choices()) return 1;
#endif
    if (check_measured_merges()) return 1;
    for (int c = 0; c < cases; ++c)
        if (check_case(rng, units)) {
            std::printf("case %d\n", c);
            return 1;
        }
#ifdef WITH_ROUND_SPLIT
    CHECK(chosen_cuts > 0 && cut_launches > 0, "%lld cuts chosen, %lld launches cut", chosen_cuts, cut_launches);
#endif
    CHECK(mixed_launches > cases / 10 && mixed_cuts > cases / 100, "%lld mixed launches, %lld cut", mixed_launches, mixed_cuts);
    std::printf("ok: %d launches, %lld k tiles owned exactly once\n", cases, units);
    return 0;
}
