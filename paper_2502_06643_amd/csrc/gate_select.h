// The top-k selection of moe_topk_gate (paper Section 2.1) for one token whose E logits are spread over L
// neighbouring lanes of a wavefront, VPL logits per lane: shared by the gate kernel (logits from memory) and by the
// fused router (logits from LDS, where the projection left them).  The lanes take turns in pieces of four logits
// (lane sub holds pieces sub, sub + L, ...), so that the lanes of one load read neighbouring 16-byte pieces.
#pragma once
#include "common.h"

namespace moe {

__device__ __forceinline__ uint32_t orderable(float v) {
    if (v == 0.0f) v = 0.0f;                       // -0.0 and +0.0 tie
    const uint32_t u = __float_as_uint(v);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float from_orderable(uint32_t o) {
    const uint32_t u = (o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o;
    return __uint_as_float(u);
}

// ---- two or more lanes per token: sorted lists ------------------------------------------------------------------
// A candidate is one double whose bit pattern orders as (key, lower expert first): a biased exponent of 1, then the 32
// bits of the key and 255 - expert.  No two are equal, so the selection is nothing but v_max_f64 / v_min_f64 (full
// rate on this chip) without an index beside the value; an empty slot has a biased exponent of 0, below every candidate.
// flipped = 255 - expert.  Nothing here branches: a logit that is not there is made an empty slot at the end.
__device__ __forceinline__ double candidate(float v, uint32_t flipped, bool have) {
    const uint32_t u = __float_as_uint(v + 0.0f);             // -0.0 and +0.0 tie
    const uint32_t key = u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
    const uint32_t hi = 0x00100000u | (key >> 24);
    return __builtin_bit_cast(double, ((uint64_t)(have ? hi : 0u) << 32) | ((key << 8) | flipped));
}
__device__ __forceinline__ int candidate_expert(double c) { return 255 - (int)(__builtin_bit_cast(uint64_t, c) & 255u); }
__device__ __forceinline__ float candidate_logit(double c) { return from_orderable((uint32_t)(__builtin_bit_cast(uint64_t, c) >> 8)); }

// The larger and the smaller of two candidates.  Written out because the compiler, for which they may be signalling NaNs,
// would pass what comes from another lane or from integer arithmetic through an instruction of its own first.
__device__ __forceinline__ double larger(double a, double b) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double smaller(double a, double b) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ void order_pair(double& hi, double& lo) {
    const double a = hi, b = lo;
    hi = larger(a, b);
    lo = smaller(a, b);
}

// bitonic a[0..K) -> descending
template <int K>
__device__ __forceinline__ void merge_bitonic(double (&a)[K]) {
#pragma unroll
    for (int st = K / 2; st > 0; st >>= 1)
#pragma unroll
        for (int i = 0; i < K; ++i)
            if ((i & st) == 0) order_pair(a[i], a[i | st]);
}

// Batcher's odd-even merge sort (Knuth, The Art of Computer Programming, volume 3, 5.2.2, Algorithm M): 19 exchanges for 8
// values, a bitonic sort has 24
template <int K>
__device__ __forceinline__ void sort_descending(double (&a)[K]) {
#pragma unroll
    for (int p = 1; p < K; p <<= 1)
#pragma unroll
        for (int st = p; st > 0; st >>= 1)
#pragma unroll
            for (int i = 0; i + st < K; ++i)
                if (i >= st % p && (i - st % p) % (2 * st) < st && i / (2 * p) == (i + st) / (2 * p)) order_pair(a[i], a[i + st]);
}

// the K largest of two descending lists, descending
template <int K>
__device__ __forceinline__ void keep_largest(double (&a)[K], const double (&b)[K]) {
#pragma unroll
    for (int i = 0; i < K; ++i) a[i] = larger(a[i], b[K - 1 - i]);
    merge_bitonic<K>(a);
}

// the value of the lane across from this one in the group of 2 M lanes: with its quad neighbours for M = 1 and 2, mirrored
// for M = 4 and 8 (every half holds one list by then, so any pairing of the halves does)
template <int M>
__device__ __forceinline__ double lane_across(double v) {
    constexpr int ctrl = M == 1 ? 0xB1 : (M == 2 ? 0x4E : (M == 4 ? 0x141 : 0x140));
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)u, ctrl, 0xF, 0xF, true);
    const uint32_t hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), ctrl, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// lane i's value, in every lane of its group of L
template <int L>
__device__ __forceinline__ float of_lane(float v, int i) {
    if constexpr (L == 2 || L == 4) {
        const int w = __float_as_int(v);
        const int r = L == 2 ? (i == 0 ? __builtin_amdgcn_mov_dpp(w, 0xA0, 0xF, 0xF, true) : __builtin_amdgcn_mov_dpp(w, 0xF5, 0xF, 0xF, true))
                    : i == 0 ? __builtin_amdgcn_mov_dpp(w, 0x00, 0xF, 0xF, true) : i == 1 ? __builtin_amdgcn_mov_dpp(w, 0x55, 0xF, 0xF, true)
                    : i == 2 ? __builtin_amdgcn_mov_dpp(w, 0xAA, 0xF, 0xF, true) : __builtin_amdgcn_mov_dpp(w, 0xFF, 0xF, 0xF, true);
        return __int_as_float(r);
    } else {
        return __shfl(v, ((threadIdx.x & 63) & ~(L - 1)) + i, 64);
    }
}

template <int M, int L, int K>
__device__ __forceinline__ void merge_lanes(double (&a)[K]) {
    if constexpr (M < L) {
        double b[K];
#pragma unroll
        for (int i = 0; i < K; ++i) b[i] = lane_across<M>(a[i]);
        keep_largest<K>(a, b);
        merge_lanes<2 * M, L, K>(a);
    }
}

// slots of the result that a lane hands out: sub, sub + L, ...
template <int L, int KMAX> constexpr int kGateSlots = (KMAX + L - 1) / L;

// row: the token's E logits (global memory or LDS; 16-byte aligned when E % 4 == 0 or `padded`); sub = this lane's
// index among the token's L lanes; live = the token exists.  `padded`: the row holds L * VPL readable floats and the
// ones from E on are ignored (the fused router's LDS rows).  Every lane of the L-lane group must call this (lane
// exchange); every lane of a live token hands slots sub, sub + L, ... of the k experts (e_sel), their exponentials
// (p_sel) and the denominator to `emit`.  KMAX >= k is a compile-time bound: the lists stay in registers.
//
// Bound by instructions: one lane alone (E <= 8) takes k rounds of a scan that carries the index; several lanes sort
// their candidates in lists of KMAX, merge the lists across lanes and share the exponentials, divisions and stores.
// Rounds of a scan and a shuffle butterfly took 18.9 us for 100003 tokens, E = 64, k = 6; bitonic sorts, a branch for each logit
// and doubles that the compiler had quieted 11.1; candidates without branches, fewer exchanges and those written out 9.3; and without the
// question which logits exist where all do (FULL) 8.7.
// FULL: E == L * VPL.  Where one copy of the selection can be had, the caller knows on the host: two of them and a branch in the kernels of
// the front cost spilled scalar registers (44, 76 and 69 for 12, 55 and 35 with 4 lanes top-2 and top-8 and 16 lanes top-8) and cold
// instruction fetches, layers of 1 to 64 tokens, 16 to 64 experts, top-2, 6.2 to 7.4 us for 5.8 to 7.0.
template <int L, int VPL, int KMAX, bool ALL, bool FULL, class Emit>
__device__ __forceinline__ void gate_select_emit(const float* row, bool padded, int sub, bool live, int E, int k, Emit emit) {
    static_assert(L >= 1 && L <= 16 && (KMAX & (KMAX - 1)) == 0 && MOE_MAX_EXPERTS <= 256, "DPP rows of 16 lanes, bitonic lists, 8-bit experts");
    constexpr int S = kGateSlots<L, KMAX>;
    const int e0 = sub * 4;                         // first logit of this lane; its i-th one is e0 + (i / 4) * 4 L + i % 4
    float v[VPL];
    bool have[VPL];
#pragma unroll
    for (int i = 0; i < VPL; ++i) { v[i] = 0.f; have[i] = FULL || (live && e0 + (i / 4) * (4 * L) + i % 4 < E); }
    if (FULL) {                                     // a lane without a token selects from a row that exists, for nobody
#pragma unroll
        for (int c = 0; c < VPL / 4; ++c) {
            const float4 q = *reinterpret_cast<const float4*>(row + e0 + 4 * L * c);
            v[4 * c] = q.x; v[4 * c + 1] = q.y; v[4 * c + 2] = q.z; v[4 * c + 3] = q.w;
        }
    } else if (live) {
        if (padded || (E & 3) == 0) {
#pragma unroll
            for (int c = 0; c < VPL / 4; ++c) {
                const int e = e0 + 4 * L * c;
                if (e < E) {
                    const float4 q = *reinterpret_cast<const float4*>(row + e);
                    v[4 * c] = q.x; v[4 * c + 1] = q.y; v[4 * c + 2] = q.z; v[4 * c + 3] = q.w;
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < VPL; ++i)
                if (have[i]) v[i] = row[e0 + (i / 4) * (4 * L) + i % 4];
        }
    }
    float denom = 0.f, p_sel[S];
    int e_sel[S];
    if constexpr (L == 1) {
        uint32_t key[VPL];
#pragma unroll
        for (int i = 0; i < VPL; ++i) key[i] = have[i] ? orderable(v[i]) : 0u;
        float top = 0.f;
#pragma unroll
        for (int j = 0; j < KMAX; ++j) {
            p_sel[j] = 0.f;
            e_sel[j] = 0;
            if (j < k) {
                uint32_t best = key[0];
                int be = 0;
#pragma unroll
                for (int i = 1; i < VPL; ++i)
                    if (key[i] > best) { best = key[i]; be = i; }
                const float lj = from_orderable(best);
                if (j == 0) {
                    top = lj;
                    if (ALL) {
#pragma unroll
                        for (int i = 0; i < VPL; ++i)
                            if (key[i] != 0u) denom += expf(from_orderable(key[i]) - top);
                    }
                }
#pragma unroll
                for (int i = 0; i < VPL; ++i)
                    if (i == be) key[i] = 0u;
                const float p = expf(lj - top);     // exp(0) = 1 for the top-1 expert
                if (!ALL) denom += p;
                p_sel[j] = p;
                e_sel[j] = be;
            }
        }
    } else {
        static_assert((L & (L - 1)) == 0, "the lane and the place in it are bits of their own in an expert's number");
        const auto slot = [&](int i) { return i < VPL ? candidate(v[i < VPL ? i : 0], (uint32_t)(255 ^ e0) ^ (uint32_t)((i / 4) * (4 * L) + i % 4), have[i < VPL ? i : 0]) : 0.0; };
        double best[KMAX];
#pragma unroll
        for (int i = 0; i < KMAX; ++i) best[i] = slot(i);
        sort_descending<KMAX>(best);
#pragma unroll
        for (int i0 = KMAX; i0 < VPL; i0 += KMAX) {
            double more[KMAX];
#pragma unroll
            for (int u = 0; u < KMAX; ++u) more[u] = slot(i0 + u);
            sort_descending<KMAX>(more);
            keep_largest<KMAX>(best, more);
        }
        merge_lanes<1, L, KMAX>(best);
        const float top = candidate_logit(best[0]);
        if (ALL) {
#pragma unroll
            for (int i = 0; i < VPL; ++i)
                if (have[i]) denom += expf(v[i] - top);
#pragma unroll
            for (int m = 1; m < L; m <<= 1) denom += __shfl_xor(denom, m, 64);
        }
#pragma unroll
        for (int i = 0; i < S; ++i) {
            double mine = best[i * L];
#pragma unroll
            for (int u = 1; u < L; ++u)
                if (i * L + u < KMAX && u == sub) mine = best[i * L + u < KMAX ? i * L + u : 0];
            e_sel[i] = candidate_expert(mine);
            p_sel[i] = expf(candidate_logit(mine) - top);
        }
        if (!ALL) {
#pragma unroll
            for (int j = 0; j < KMAX; ++j) {        // summed in slot order, in every lane
                const float p = of_lane<L>(p_sel[j / L], j % L);
                if (j < k) denom += p;
            }
        }
    }
    if (live) emit(e_sel, p_sel, denom);
}

// writes this lane's slots of topk_idx[t][0..k) and topk_w[t][0..k)
template <int L, int S>
__device__ __forceinline__ void gate_store(long long t, int sub, int k, const int (&e_sel)[S], const float (&p_sel)[S], float denom,
                                           int32_t* __restrict__ topk_idx, float* __restrict__ topk_w) {
    if (L == 1 && S == 2 && k == 2) {               // the common top-2 case: one 8-byte store each
        *reinterpret_cast<int2*>(topk_idx + t * 2) = make_int2(e_sel[0], e_sel[S - 1]);
        *reinterpret_cast<float2*>(topk_w + t * 2) = make_float2(p_sel[0] / denom, p_sel[S - 1] / denom);
    } else {
#pragma unroll
        for (int i = 0; i < S; ++i)
            if (sub + L * i < k) {
                topk_idx[t * k + sub + L * i] = e_sel[i];
                topk_w[t * k + sub + L * i] = p_sel[i] / denom;
            }
    }
}

template <int L, int VPL, int KMAX, bool ALL, bool FULL>
__device__ __forceinline__ void gate_select(const float* row, bool padded, int sub, bool live, long long t, int E, int k,
                                            int32_t* __restrict__ topk_idx, float* __restrict__ topk_w) {
    constexpr int S = kGateSlots<L, KMAX>;
    gate_select_emit<L, VPL, KMAX, ALL, FULL>(row, padded, sub, live, E, k,
                                        [&](const int (&e_sel)[S], const float (&p_sel)[S], float denom) {
                                            gate_store<L, S>(t, sub, k, e_sel, p_sel, denom, topk_idx, topk_w);
                                        });
}

}  // namespace moe
