// Send rows copied during the expert FFN.  In a layer call on one GPU of several most rows of the send buffer go to other
// GPUs (paper Section 2.2, the first all-to-all): nothing of this call reads them.  A layer of many small experts has
// fewer output tiles here than the chip has compute units, so those rows are left to the workgroups that would be
// idle in the two projections, as many as these copy in the time of a tile.
//
// 8192 tokens, 64 experts, top-6, 8 of them here, d 2048, f 1408: row copy 39 -> 14 us (9 since it looks this GPU's rows up in the sorted
// order), projections 50 + 37 -> 59 + 50 (the copies take bandwidth from the tiles), layer 151 -> 143 (139).  Stores that stay out of the caches: 3 us less than without.  Random layers, with
// buffers that change from call to call, so that the weights are not in a cache: 246 that leave rows to the projections 1.040
// times as fast as without (geometric mean), the worst 0.984, 54 that ask and leave none 0.999.
#pragma once
#include "ffn_plan.h"

namespace moe {

// What a copying workgroup moves in the time of a k tile (1.3 us), bytes read and written.  80 KB made the layer above 4 us slower, 20
// KB 6.  20 KB in the down projection alone, whose tiles wait for memory more: the same 246 layers 1.037, the layer above 145, though where
// one layer is called over and over with its weights in the Infinity Cache 141.
constexpr int kLateBytesPerKTile = 40 << 10;

// Per XCD: compute units without a tile in a launch of MT x NT tiles that runs in one round; 0 when it takes longer.
__host__ __device__ __forceinline__ int late_copiers(int MT, int NT, int cus_per_xcd) {
    if (MT > kXcds * cus_per_xcd) return 0;
    const int tiles = MT * (NT / kXcds) + (MT * (NT % kXcds) + kXcds - 1) / kXcds;     // of the first XCD, which has the largest share (xcd_share)
    return tiles < cus_per_xcd ? cus_per_xcd - tiles : 0;
}

// How many tokens' rows the two projections take: what fits beside their tiles, while a quarter of the compute units has none in the up
// projection and if it is at least half of all (with 192 to 224 tiles on 256 compute units 25 layers 1.004 times as fast, the worst
// 0.97, with less than half of the tokens 30 0.998, 0.97; else 0.99 at worst).  The row copy works this out, in every thread: in
// the index kernels it would lengthen a serial chain that everything waits for (rank kernel 1.2 to 1.7 us, one-workgroup kernel 0.2 to 0.7).
struct LateTokens { int up, down; };
__device__ __forceinline__ LateTokens late_tokens(const LateShape& l, const int32_t* __restrict__ plan, int own_rows) {
    const int MT = plan[3] == 0 ? plan[1] : plan[2], foreign = l.T * l.k - own_rows;
    // a token's rows: one read, and one written for each of its routes of other GPUs
    const float tokens = __builtin_amdgcn_rcpf(__builtin_fmaf((float)foreign, l.per_token, 1.0f));
    const auto fit = [&](int copiers, float rows, int left) {
        const float n = (float)copiers * rows * tokens;
        return n < (float)left ? (int)n : left;
    };
    const int idle = late_copiers(MT, l.nt_up, l.cus_per_xcd), T = foreign > 0 && 4 * idle >= l.cus_per_xcd ? l.T : 0;
    LateTokens t;
    t.up = fit(idle, l.rows_up, T);
    t.down = fit(late_copiers(MT, l.nt_down, l.cus_per_xcd), l.rows_down, T - t.up);
    if (2 * (t.up + t.down) < T) t.up = t.down = 0;      // the token's rows are looked at once more, for little
    return t;
}

struct LateRows { const uint4* x; uint4* send; const int32_t* inv_perm; int k, N, units; };

typedef __attribute__((ext_vector_type(4))) uint32_t late_u32x4;

// Workgroup `block` of the up or the down projection, which has no tile: the rows of that launch's tokens outside this GPU's range.
// A wavefront takes a token at a time: its row once, its positions one a lane.
__device__ __forceinline__ void copy_late_rows(const LateRows& l, const int32_t* __restrict__ plan, bool up, int MT, int NT, int cus_per_xcd,
                                               unsigned block) {
    const int of_up = plan[kPlanLateUp], begin = up ? 0 : of_up, end = up ? of_up : of_up + plan[kPlanLateDown];
    if (begin == end) return;
    const int x = (int)(block % kXcds), idle = (int)(block / kXcds) - xcd_share(MT, NT, x, 0, cus_per_xcd, false).full;
    const int copiers = late_copiers(MT, NT, cus_per_xcd);
    if (idle < 0 || idle >= copiers) return;
    const int own0 = plan[kPlanOwnBegin], own1 = plan[kPlanOwnEnd];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    for (int t = begin + (idle * kXcds + x) * waves + wave; t < end; t += copiers * kXcds * waves) {
        const int at = lane < l.k ? l.inv_perm[(long long)t * l.k + lane] : -1;
        const late_u32x4* row = reinterpret_cast<const late_u32x4*>(l.x) + (long long)t * l.units;
        for (int c0 = lane; c0 - lane < l.units; c0 += 4 * 64) {
            late_u32x4 v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = c0 + 64 * i < l.units ? row[c0 + 64 * i] : late_u32x4{0u, 0u, 0u, 0u};
            for (int j = 0; j < l.k; ++j) {
                const int p = __builtin_amdgcn_readlane(at, j);
                if ((unsigned)p >= (unsigned)l.N || (p >= own0 && p < own1)) continue;
                late_u32x4* out = reinterpret_cast<late_u32x4*>(l.send) + (long long)p * l.units;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (c0 + 64 * i < l.units) __builtin_nontemporal_store(v[i], out + c0 + 64 * i);      // nothing here reads them
            }
        }
    }
}

}  // namespace moe
