// Placement evaluators: the quantities the paper's two ILPs are built from,
// computed on the GPU from the profiled statistics and a given expert->GPU map
// (the solve itself is not here).
//   moe_accumulate_counts : P_{e,l} += expert_counts of one batch      (ILP 1 input)
//   moe_placement_loads   : T_{c,l} = sum_e P_{e,l} x_{c,e,l}          (Eq. 2)
//                           sum_c |T_{c,l} - mean_l|, mean_l = sum_e P_{e,l} / G   (Eq. 1, Eq. 3)
//   moe_placement_traffic : C_{c1,c2,l} = sum R_{e1,e2,l} x_{c1,e1,l} x_{c2,e2,l+1}   (Eq. 9)
//                           max over GPU pairs of C / B                 (Eq. 8, one layer's term)
// The tables are tiny (E <= 256, G <= 256), so each call is one workgroup, bound by its launch and by how many
// dependent rounds of memory latency it makes (placement_loads with the tables in LDS: 5.4 -> 2.4 us at E = 64).
#include <algorithm>
#include "common.h"

namespace moe {

__global__ __launch_bounds__(256) void accumulate_counts_kernel(const int32_t* __restrict__ counts, int E, long long* __restrict__ P) {
    const int e = threadIdx.x;
    if (e < E) P[e] += (long long)counts[e];
}

__global__ __launch_bounds__(256) void placement_loads_kernel(const long long* __restrict__ P, const int32_t* __restrict__ placement,
                                                              int E, int G, long long* __restrict__ T_c, double* __restrict__ imbalance) {
    __shared__ long long p_e[MOE_MAX_EXPERTS];
    __shared__ int pl[MOE_MAX_EXPERTS];
    __shared__ double dev[MOE_MAX_GPUS];
    const int g = threadIdx.x;
    // both tables through LDS: one round of memory latency instead of one per expert
    p_e[g] = g < E ? P[g] : 0;
    pl[g] = g < E ? placement[g] : -1;
    __syncthreads();
    long long mine = 0, total = 0;
#pragma unroll 8
    for (int e = 0; e < E; ++e) {                        // every thread walks the E experts: E <= 256
        const long long p = p_e[e];
        total += p;
        mine += pl[e] == g ? p : 0;
    }
    if (g < G) {
        T_c[g] = mine;
        dev[g] = fabs((double)mine - (double)total / (double)G);
    }
    __syncthreads();
    if (g == 0 && imbalance) {
        double s = 0.0;
        for (int c = 0; c < G; ++c) s += dev[c];         // fixed order
        *imbalance = s;
    }
}

// One workgroup reads R once, all its loads independent, and adds every entry to its GPU pair's bin in LDS.
// The G x G bins are done in stripes of g1 of at most kTrafficBins bins (one stripe up to G = 90); a small
// table gets several copies, picked by lane, so that the lanes of a row, which mostly belong to few GPU
// pairs, do not queue on one address.  Bound by the read of R (at most
// 512 KB by one compute unit) and one LDS atomic per entry; for the small tables of a layer by latency: launch, R, barriers.
// A thread per GPU pair that walked R's rows itself, load after load, took 408 us for 64 experts on 8 GPUs.
// FEW: at most as many counters as threads, so that neighbouring lanes add up the copies of a bin, and the first rows asked for
// before it is known who needs them: 64 experts on 8 GPUs 5.1 us without, 4.7 with.  Where that leaves the lanes of a GPU pair, whose
// experts lie side by side in the usual map, less than a counter for two, they queue, and a thread adds up more copies of a bin
// faster than lanes do in several rounds (256 contiguous experts on 32 GPUs 14.0 us; with a counter a bin 31, with 8 and lanes 17.2).
constexpr int kTrafficThreads = 1024;
constexpr int kTrafficBins = 8192;       // 64 KB of int64
constexpr int kTrafficInFlight = 8;      // rows of R a thread fetches together

template <bool FEW>
__global__ __launch_bounds__(kTrafficThreads) void placement_traffic_kernel(const long long* __restrict__ R, const int32_t* __restrict__ pl_l,
                                                                            const int32_t* __restrict__ pl_l1, int E_l, int E_l1, int G,
                                                                            int col_bits, int stripe, int copies,
                                                                            long long* __restrict__ C, const double* __restrict__ B,
                                                                            double* __restrict__ max_cost) {
    __shared__ unsigned long long bins[kTrafficBins];
    __shared__ int row_gpu[MOE_MAX_EXPERTS];
    __shared__ double best[kTrafficThreads / 64];
    const int tid = threadIdx.x;
    // thread -> (row, column) of R with the column padded to a power of two
    const int e2 = tid & ((1 << col_bits) - 1), first_row = tid >> col_bits, rows_per_step = kTrafficThreads >> col_bits;
    const int g2 = e2 < E_l1 ? pl_l1[e2] : -1;
    const bool col_ok = (unsigned)g2 < (unsigned)G;
    if (tid < E_l) row_gpu[tid] = pl_l[tid];
    long long first[kTrafficInFlight];
    if (FEW) {
#pragma unroll
        for (int u = 0; u < kTrafficInFlight; ++u) {
            const int row = first_row + u * rows_per_step;
            first[u] = row < E_l && e2 < E_l1 ? R[(size_t)row * E_l1 + e2] : 0;
        }
    }
    double local_max = 0.0;
    for (int s0 = 0; s0 < G; s0 += stripe) {
        const int rows = min(stripe, G - s0), n_bins = rows * G;
        for (int i = tid; i < n_bins * copies; i += kTrafficThreads) bins[i] = 0ull;
        __syncthreads();
        if (col_ok) {
            const auto add = [&](int g, long long r) {
                if ((unsigned)g < (unsigned)rows && r != 0)
                    atomicAdd(&bins[(g * G + g2) * copies + (tid & (copies - 1))], (unsigned long long)r);
            };
            int e1 = first_row;
            if (FEW) {
#pragma unroll
                for (int u = 0; u < kTrafficInFlight; ++u) {
                    const int row = e1 + u * rows_per_step;
                    add(row < E_l ? row_gpu[row] - s0 : -1, first[u]);
                }
                e1 += rows_per_step * kTrafficInFlight;
            }
            for (; e1 < E_l; e1 += rows_per_step * kTrafficInFlight) {
                long long r[kTrafficInFlight];
                int g[kTrafficInFlight];
#pragma unroll
                for (int u = 0; u < kTrafficInFlight; ++u) {
                    const int row = e1 + u * rows_per_step;
                    g[u] = row < E_l ? row_gpu[row] - s0 : -1;
                    r[u] = (unsigned)g[u] < (unsigned)rows ? R[(size_t)row * E_l1 + e2] : 0;
                }
#pragma unroll
                for (int u = 0; u < kTrafficInFlight; ++u) add(g[u], r[u]);
            }
        }
        __syncthreads();
        const auto put = [&](int p, unsigned long long s) {
            const size_t pair = (size_t)s0 * G + p;
            C[pair] = (long long)s;
            const double cost = B ? (double)(long long)s / B[pair] : (double)(long long)s;
            local_max = cost > local_max ? cost : local_max;
        };
        if (FEW) {                                       // copies: a power of two up to 32
            unsigned long long s = tid < n_bins * copies ? bins[tid] : 0ull;
            for (int m = 1; m < copies; m <<= 1) s += __shfl_xor(s, m, 64);
            if (tid < n_bins * copies && (tid & (copies - 1)) == 0) put(tid / copies, s);
        } else {
            for (int p = tid; p < n_bins; p += kTrafficThreads) {
                unsigned long long s = 0;
                for (int c = 0; c < copies; ++c) s += bins[p * copies + ((c + tid) & (copies - 1))];
                put(p, s);
            }
        }
        __syncthreads();                                 // the bins have been read before the next stripe clears them
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        const double o = __shfl_xor(local_max, m, 64);
        local_max = o > local_max ? o : local_max;
    }
    if ((tid & 63) == 0) best[tid >> 6] = local_max;
    __syncthreads();
    if (tid == 0 && max_cost) {
        double m = 0.0;
        for (int i = 0; i < kTrafficThreads / 64; ++i) m = best[i] > m ? best[i] : m;
        *max_cost = m;
    }
}

int launch_accumulate_counts(const int32_t* counts, int E, int64_t* P, hipStream_t s) {
    hipLaunchKernelGGL(accumulate_counts_kernel, dim3(1), dim3(256), 0, s, counts, E, (long long*)P);
    return check_launch("moe_accumulate_counts launch");
}

int launch_placement_loads(const int64_t* P, const int32_t* placement, int E, int G, int64_t* T_c, double* imbalance, hipStream_t s) {
    hipLaunchKernelGGL(placement_loads_kernel, dim3(1), dim3(256), 0, s, (const long long*)P, placement, E, G, (long long*)T_c, imbalance);
    return check_launch("moe_placement_loads launch");
}

int launch_placement_traffic(const int64_t* R, const int32_t* pl_l, const int32_t* pl_l1, int E_l, int E_l1, int G, int64_t* C,
                             const double* B, double* max_cost, hipStream_t s) {
    int col_bits = 0;
    while ((1 << col_bits) < E_l1) ++col_bits;
    const int stripe = G * G <= kTrafficBins ? G : kTrafficBins / G;
    const auto copies_in = [&](int counters) {
        int copies = 1;
        while (copies < 32 && G * G * copies * 2 <= counters) copies *= 2;
        return copies;
    };
    // lanes of a wavefront with the same bin where a GPU's experts are neighbours: its columns, and its rows as far as the wavefront has them
    const int cols = (E_l1 + G - 1) / G, rows = std::min((E_l + G - 1) / G, std::max(64 >> col_bits, 1));
    const bool few = G * G <= kTrafficThreads && 2 * copies_in(kTrafficThreads) >= cols * rows;
    hipLaunchKernelGGL(few ? &placement_traffic_kernel<true> : &placement_traffic_kernel<false>, dim3(1), dim3(kTrafficThreads), 0, s, (const long long*)R,
                       pl_l, pl_l1, E_l, E_l1, G, col_bits, stripe, copies_in(few ? kTrafficThreads : kTrafficBins), (long long*)C, B, max_cost);
    return check_launch("moe_placement_traffic launch");
}

}  // namespace moe
