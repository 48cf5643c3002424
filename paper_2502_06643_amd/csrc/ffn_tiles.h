// Which piece of the grouped GEMM does a workgroup own?  The index arithmetic
// that turns (workgroup id, tile plan) into (expert, rows, column tile, k range)
// for moe_expert_ffn_grouped (paper Section 2.2 / Fig. 2b, the expert FFN over
// ragged per-expert buckets), kept apart from the kernels so that it can also
// be compiled for the host and checked exhaustively there: every
// (bucket, row tile, column tile, k tile) must be owned exactly once.
#pragma once
#include "ffn_plan.h"

namespace moe {

constexpr int kMaxCusPerXcd = 48;               // two fp32 partial-tile slots exist per compute unit, for at most this many

struct WorkItem {
    int expert, row0, rows, nt;
    int bucket, first;   // listed bucket and the tile's first row in it (row0 is the buffer row unless buckets are merged)
    int kt0, kt1;        // k tile range
    int partial;         // slot of the fp32 partial tile, or -1 for a whole tile
};

// Tile order inside one expert: row tiles are taken in chunks of `row_chunk`, and within a chunk the
// column tile advances before the chunk does, so the ~32 tiles that run together on an XCD form a
// row_chunk x (32 / row_chunk) block that streams row_chunk activation panels and 32 / row_chunk
// weight panels through that XCD's L2 (a large expert would otherwise run as a 32 x 1 strip that
// re-reads its activations once per column tile).  Every chunk re-reads the expert's weights, which
// come from DRAM, while re-read activations come from the Infinity Cache as long as they fit there:
// chunks of 8 row tiles then, of 4 (the split that moves the fewest bytes) for larger batches.
constexpr size_t kActivationsFitCache = (size_t)128 << 20;
static inline int row_chunk_for(size_t activation_bytes) { return activation_bytes <= kActivationsFitCache ? 8 : 4; }

// tile number `tile` of a list that walks NT column tiles of every listed bucket.  The bucket is searched by halves: each step waits for a
// load, a walk took 90 to 130 ns a bucket by where the compiler had put the loop, and many experts have many buckets.  Down projection, us, walk
// (in either place) / halves: 256 experts, top-8, 8000 tokens, d 1024, f 512 183, 205 / 132; top-4, 200 tokens, d 1664, f 1280 263, 283 / 208; 64 experts,
// top-6, 400 tokens, d 2048, f 1408 95 / 90; 8 experts as before.
__host__ __device__ __forceinline__ void locate_tile(const int32_t* __restrict__ plan, const int32_t* __restrict__ prefix, int NT,
                                                     long long tile, int BM, int row_chunk, WorkItem& w) {
    int i = 0;
    for (int last = plan[0] - 1; i < last;) {            // the last bucket that begins at or before the tile
        const int mid = (i + last + 1) >> 1;
        if ((long long)prefix[mid] * NT <= tile) i = mid; else last = mid - 1;
    }
    const int mt_e = prefix[i + 1] - prefix[i];
    const int rem = (int)(tile - (long long)prefix[i] * NT);
    const int per_chunk = row_chunk * NT;
    const int q = rem / per_chunk;                       // chunk of row tiles
    const int in_chunk = rem - q * per_chunk;
    const int left = mt_e - q * row_chunk;
    const int rows_here = row_chunk < left ? row_chunk : left;
    w.nt = in_chunk / rows_here;
    const int mt = q * row_chunk + (in_chunk - w.nt * rows_here);
    w.expert = plan[kPlanExpert + i];
    w.bucket = i;
    w.first = mt * BM;
    w.row0 = plan[kPlanStart + i] + mt * BM;
    const int rows_left = plan[kPlanCount + i] - mt * BM;
    w.rows = BM < rows_left ? BM : rows_left;
}

// Place `idx` of an XCD's list of `n` tiles -> tile number, when the plan says so (kPlanMixed).  A bucket of several row tiles is
// bound by the matrix pipes (its row tiles share a weight panel), a bucket of one by its weights; buckets being listed by
// size, all of the first kind would run before all of the second.  They are spread evenly among the others instead, but for
// the last round, which is the others'.
// Measured, layer, us, by size / spread: Mixtral shape, 380 tokens 604 / 593, 640 689 / 684, 777 722 / 711, 900 776 / 767; 64 experts, top-6,
// d 2048, f 1408, 1500 tokens 364 / 353.  With fewer tiles of the second kind than of the first: 2000 tokens 1295 / 1309, 16
// experts, top-4, d 1024, f 2048, 2500 tokens 191.5 / 193.5, one of 4 GPUs' share of 3000 Mixtral tokens 500 / 505.
__host__ __device__ __forceinline__ int mixed_tile(int heavy_rows, int q, int n, int idx, int cus_per_xcd) {
    const unsigned heavy = (unsigned)heavy_rows * (unsigned)q, light = (unsigned)n - heavy, at = (unsigned)idx;
    const unsigned span = (unsigned)n - (light < (unsigned)cus_per_xcd ? light : (unsigned)cus_per_xcd), rate = (heavy << 16) / span;
    const unsigned here = at < span ? at : span, before = here * rate >> 16;         // heavy tiles before place `here`
    if (at < span) return (int)((here + 1) * rate >> 16 > before ? before : heavy + at - before);
    return (int)(at - span < heavy - before ? before + at - span : at);
}

// tile `idx` of XCD x's list: first the tiles of its own column tiles, then its share of the left-over ones
__host__ __device__ __forceinline__ void locate_xcd_tile(const int32_t* __restrict__ plan, const int32_t* __restrict__ prefix,
                                                         const XcdShare& sh, int x, int idx, int BM, int cus_per_xcd, int row_chunk, WorkItem& w) {
    if (idx < sh.main) {
        const int heavy = BM == kShortTileRows && sh.main < 1 << 16 ? plan[kPlanMixed] : 0;
        locate_tile(plan, prefix, sh.q, heavy > 0 ? mixed_tile(heavy, sh.q, (int)sh.main, idx, cus_per_xcd) : idx, BM, row_chunk, w);
        w.nt += x * sh.q;
    } else {
        locate_tile(plan, prefix, sh.rem, sh.rem_begin + (idx - sh.main), BM, row_chunk, w);
        w.nt += kXcds * sh.q;
    }
}

// A launch whose tiles all run in one round and are cut by cost; the plan says into how many parts (round_split in
// ffn_plan.h: only with tiles of kShortTileRows rows).
struct RoundSplit {
    bool on;
    int q, rem;               // column tiles owned outright by every XCD; left-over ones
    int nb, ns;               // row tiles of more than kSmallTileRows rows, and of at most that
    int big, small;           // k parts of either kind
    int nbx, nsx;             // tiles of either kind on this XCD
    int rb0, rs0;             // ... and its first ones in the lists of left-over-column tiles
};

__host__ __device__ __forceinline__ RoundSplit round_share(const int32_t* __restrict__ plan, int MT, int NT, int x, int BM) {
    RoundSplit s;
    s.big = plan[kPlanBigParts];
    s.on = BM == kShortTileRows && s.big > 0;
    if (!s.on) return s;
    s.small = plan[kPlanSmallParts];
    s.q = NT / kXcds;
    s.rem = NT - s.q * kXcds;
    s.ns = plan[kPlanSmallTiles] - 1;
    s.nb = MT - s.ns;
    const int cb = (s.nb * s.rem + kXcds - 1) / kXcds, cs = (s.ns * s.rem + kXcds - 1) / kXcds;
    s.rb0 = x * cb;
    s.rs0 = x * cs;
    const int rb = s.nb * s.rem - s.rb0, rs = s.ns * s.rem - s.rs0;
    s.nbx = s.nb * s.q + (rb < 0 ? 0 : (rb < cb ? rb : cb));
    s.nsx = s.ns * s.q + (rs < 0 ? 0 : (rs < cs ? rs : cs));
    return s;
}

// tile number `tile` of either kind, of a list that walks NT column tiles of every listed bucket
__host__ __device__ __forceinline__ void locate_kind(const int32_t* __restrict__ plan, const int32_t* __restrict__ prefix, int NT, int tile,
                                                     int BM, bool small, WorkItem& w) {
    for (int i = 0; i < plan[0]; ++i) {
        const int tiles = prefix[i + 1] - prefix[i], last = plan[kPlanCount + i] - (tiles - 1) * BM;
        const int has_small = last <= kSmallTileRows ? 1 : 0, here = small ? has_small : tiles - has_small;
        if (tile >= here * NT) {
            tile -= here * NT;
            continue;
        }
        w.nt = tile / here;
        const int mt = small ? tiles - 1 : tile - w.nt * here;
        w.expert = plan[kPlanExpert + i];
        w.bucket = i;
        w.first = mt * BM;
        w.row0 = plan[kPlanStart + i] + mt * BM;
        w.rows = mt == tiles - 1 ? last : BM;
        return;
    }
}

// tile idx (big ones first) of XCD x
__host__ __device__ __forceinline__ void locate_round_tile(const int32_t* __restrict__ plan, const int32_t* __restrict__ prefix,
                                                           const RoundSplit& s, int x, int idx, int BM, WorkItem& w) {
    const bool small = idx >= s.nbx;
    if (small) idx -= s.nbx;
    const int own = (small ? s.ns : s.nb) * s.q;
    if (idx < own) {
        locate_kind(plan, prefix, s.q, idx, BM, small, w);
        w.nt += x * s.q;
    } else {
        locate_kind(plan, prefix, s.rem, (small ? s.rs0 : s.rb0) + idx - own, BM, small, w);
        w.nt += kXcds * s.q;
    }
}

// The work of workgroup `block` of a GEMM launch (blocks are dealt round-robin to the XCDs by the hardware:
// XCD = block % 8, and `slot` = block / 8 counts within the XCD): a whole tile, or one k part of a tail tile
// with its partial-tile slot.  False when the launch holds more workgroups than this XCD has work.
__host__ __device__ __forceinline__ bool workgroup_item(const int32_t* __restrict__ plan, const int32_t* __restrict__ prefix,
                                                        int NT, int KT, int BM, unsigned block, int cus_per_xcd, int row_chunk,
                                                        bool allow_split, WorkItem& w) {
    const int x = (int)(block % kXcds), slot = (int)(block / kXcds);
    if (allow_split) {
        const RoundSplit rs = round_share(plan, prefix[plan[0]], NT, x, BM);
        if (rs.on) {
            const int big_slots = rs.nbx * rs.big;
            if (slot >= big_slots + rs.nsx * rs.small) return false;
            const int parts = slot < big_slots ? rs.big : rs.small, j = slot < big_slots ? slot : slot - big_slots;
            const int part = j % parts;
            locate_round_tile(plan, prefix, rs, x, (slot < big_slots ? 0 : rs.nbx) + j / parts, BM, w);
            w.kt0 = (int)((long long)part * KT / parts);
            w.kt1 = (int)((long long)(part + 1) * KT / parts);
            w.partial = parts > 1 ? x * 2 * cus_per_xcd + slot : -1;
            return true;
        }
    }
    const XcdShare sh = xcd_share(prefix[plan[0]], NT, x, KT, cus_per_xcd, allow_split);
    if (slot >= sh.full + sh.tail * sh.split) return false;
    if (slot < sh.full) {
        locate_xcd_tile(plan, prefix, sh, x, slot, BM, cus_per_xcd, row_chunk, w);
        w.kt0 = 0; w.kt1 = KT; w.partial = -1;
    } else {
        const int j = slot - sh.full;
        const int part = j % sh.split;
        locate_xcd_tile(plan, prefix, sh, x, sh.full + j / sh.split, BM, cus_per_xcd, row_chunk, w);
        w.kt0 = (int)((long long)part * KT / sh.split);
        w.kt1 = (int)((long long)(part + 1) * KT / sh.split);
        w.partial = x * 2 * cus_per_xcd + j;
    }
    return true;
}

// Tail tile q of XCD x, for the fix-up that adds its k parts: the tile, the slot of its first partial tile
// and the number of parts (their slots follow each other).  False when the XCD has fewer tail tiles.
__host__ __device__ __forceinline__ bool fixup_item(const int32_t* __restrict__ plan, const int32_t* __restrict__ prefix, int NT,
                                                    int KT, int BM, int x, int q, int cus_per_xcd, int row_chunk, WorkItem& w,
                                                    int& first_partial, int& parts) {
    const RoundSplit rs = round_share(plan, prefix[plan[0]], NT, x, BM);
    if (rs.on) {
        if (q >= rs.nbx + rs.nsx) return false;
        parts = q < rs.nbx ? rs.big : rs.small;
        if (parts == 1) return false;
        locate_round_tile(plan, prefix, rs, x, q, BM, w);
        first_partial = x * 2 * cus_per_xcd + (q < rs.nbx ? q * rs.big : rs.nbx * rs.big + (q - rs.nbx) * rs.small);
        return true;
    }
    const XcdShare sh = xcd_share(prefix[plan[0]], NT, x, KT, cus_per_xcd, true);
    if (q >= sh.tail) return false;
    locate_xcd_tile(plan, prefix, sh, x, sh.full + q, BM, cus_per_xcd, row_chunk, w);
    first_partial = x * 2 * cus_per_xcd + q * sh.split;
    parts = sh.split;
    return true;
}

// Workgroups a GEMM launch needs for N rows in E buckets, whatever the bucket sizes (only the device knows
// them): the sum of ceil(n_e / bm) never exceeds N / bm + min(E, N), and the split tail adds at most two
// parts per compute unit.
static inline long long ffn_grid(int N, int E, long long nt, int bm, bool split, int cus_per_xcd) {
    const long long mt_max = (N + bm - 1) / bm + (E < N ? E : N);
    const long long per_xcd = mt_max * (nt / kXcds) + (mt_max * (nt % kXcds) + kXcds - 1) / kXcds;
    return (long long)kXcds * (per_xcd + (split ? 2 * cus_per_xcd : 0));
}

}  // namespace moe
