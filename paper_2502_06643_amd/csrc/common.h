// Internal helpers shared by the HIP sources of libmoetuner_hip (not part of
// the public interface, which is include/moetuner.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include "moetuner.h"

namespace moe {

// printf-style message for moe_last_error(); returns `code` for tail calls.
int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
int hip_fail(hipError_t e, const char* what);

// Brackets one kernel launch with a pair of events when a timing session has
// selected this kernel id; otherwise does nothing.
class LaunchTimer {
public:
    LaunchTimer(int kernel_id, hipStream_t stream);
    ~LaunchTimer();
    LaunchTimer(const LaunchTimer&) = delete;
    LaunchTimer& operator=(const LaunchTimer&) = delete;
private:
    int slot_;
    hipStream_t stream_;
    hipEvent_t start_ = nullptr, stop_ = nullptr;
};

inline int check_launch(const char* what) {
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? MOE_OK : hip_fail(e, what);
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
inline int elt_bytes(moe_dtype_t dt) { return dt == MOE_BF16 ? 2 : 4; }

// ---- launchers implemented in the .hip files --------------------------------
int launch_gate(const float* logits, int T, int E, int k, bool all_norm, int32_t* idx, float* w, hipStream_t s);

constexpr int kDispatchBlock = 256;
constexpr int kDispatchItems = 4;
void dispatch_geometry(long long N, int* items, int* nblocks);      // of the workspace: routes per thread and number of chunks
// How the expert FFN wants its tile plan built for N rows in E groups: the two tile heights, which of them (see
// launch_ffn_plan), and the column and k tiles of the down projection and the compute units per XCD (kt_down = 0: the
// path that follows does not split it).
struct PlanShape { int bm0, bm1, choice, nt_down, kt_down, cus_per_xcd; };
// Rows of other GPUs' experts that the tiled bf16 projections copy on the compute units that they leave idle (ffn_late.h):
// column tiles of both projections, rows that an idle compute unit of every XCD reads or writes meanwhile (rows_down = 0: the down
// projection fills the chip); tokens, routes a token, 1 / tokens.
struct LateShape { int nt_up, nt_down; float rows_up, rows_down; int T, k; float per_token; int cus_per_xcd; };
// The tile plan as a by-product of the dispatch's index kernels, which hold all it needs; plan == NULL: none wanted.
// late.T = 0: every row is copied before the FFN.
struct PlanTask { int32_t* plan; int local_gpu; PlanShape shape; LateShape late; };
int launch_dispatch(const void* x, int row_bytes, const int32_t* topk_idx, int T, int E, int k,
                    const int32_t* placement, int G, void* send_buf, int32_t* perm, int32_t* inv_perm,
                    int32_t* expert_counts, int32_t* expert_start, int32_t* gpu_counts,
                    int32_t* gpu_offsets, int32_t* block_counts, const PlanTask& plan_task, hipStream_t s);

// moe_dispatch_noalloc: the per-chunk histograms live in a file-scope device array of this many bytes;
// dispatch_static_scratch returns the current device's copy of it (looked up once per device)
constexpr size_t kDispatchStaticScratchBytes = (size_t)256 << 10;
int dispatch_static_scratch(int32_t** scratch);

int launch_combine(const void* ffn_out, moe_dtype_t dt, const int32_t* inv_perm, const int32_t* topk_idx,
                   const float* topk_w, const int32_t* placement, int local_gpu, int T, int d, int E, int k,
                   void* y, hipStream_t s);

int launch_transition(const int32_t* idx_l, const int32_t* idx_l1, int T, int k_l, int k_l1, int E_l,
                      int E_l1, bool top1_only, int64_t* R, hipStream_t s);

size_t router_packed_bytes(int d, int E, moe_dtype_t dt);
int launch_pack_router(const void* w_g, int d, int E, moe_dtype_t dt, void* packed, hipStream_t s);
int launch_router_gate(const void* x, moe_dtype_t dt, const void* packed, const float* bias, int T, int d, int E, int k,
                       float* logits, int32_t* idx, float* w, hipStream_t s);
int launch_accumulate_counts(const int32_t* counts, int E, int64_t* P, hipStream_t s);
int launch_placement_loads(const int64_t* P, const int32_t* placement, int E, int G, int64_t* T_c, double* imbalance, hipStream_t s);
int launch_placement_traffic(const int64_t* R, const int32_t* pl_l, const int32_t* pl_l1, int E_l, int E_l1, int G, int64_t* C,
                             const double* B, double* max_cost, hipStream_t s);

int launch_receive_segments(const int32_t* counts_all, const int32_t* placement, int E, int G, int dest, int max_seg,
                            int32_t* seg_expert, int32_t* seg_counts, int32_t* seg_start, int32_t* src_offset, int32_t* n_seg_out,
                            hipStream_t s);

// FFN: the workspace starts with a small plan area, followed by H [N,f].
constexpr size_t kPlanBytes = 8192;
size_t packed_bytes_f32(int E, int d, int f);
size_t packed_bytes_bf16(int E, int d, int f);
size_t ffn_bf16_scratch_bytes();      // fp32 partial tiles of the split tail, sized for the largest supported XCD
int launch_pack_f32(const float* w1, const float* w3, const float* w2, int E, int d, int f, float* packed, hipStream_t s);
int launch_pack_bf16(const void* w1, const void* w3, const void* w2, int E, int d, int f, void* packed, hipStream_t s);
bool ffn_streams(int N, int d, int f, int E, bool segments);
int ffn_plan_shape(moe_dtype_t dt, int N, int d, int f, int E, bool every_row_resident, bool segments, PlanShape* shape);
// T = 0: no rows are left to the projections
LateShape ffn_late_shape(moe_dtype_t dt, int N, int d, int f, int E, int T, int k, int G, int cus_per_xcd);
int ffn_bf16_device_setup(int* cus_per_xcd);      // of the tiled bf16 kernels, done by the first call on a device
// E row groups (counts/starts); group g uses the weights of expert group_expert[g] of n_weights
// (g itself when group_expert is NULL).  plan_ready: the plan has been built already (ffn_plan_shape's way)
int launch_ffn_f32(const float* a, int N, int d, int f, int E, const float* packed, const int32_t* counts,
                   const int32_t* starts, const int32_t* placement, int local_gpu, const int32_t* group_expert,
                   int n_weights, float* out, int32_t* plan, bool plan_ready, float* H, hipStream_t s);
// bf16, ffn_streams(): weight-streaming kernels for batches of few rows (plan already built).
// kFfnSkinnyMaxRows counts all routes, resident or not, whatever the shape.  Whole layer, us, tiled / streaming kernels: Mixtral
// shape, top-2, skewed, all experts, N = 72 476 / 448, 160 498 / 508, 256 504 / 558 (tasks of 64 rows of the largest buckets); two of the
// eight experts 149 / 139, 149 / 142, 148 / 146, with the most popular one among them 145 / 143, 153 / 174, 156 / 214; d 1024, f 4096,
// 16 experts 85 / 76, 95 / 89, 93 / 90; 8 of 64 experts, d 2048, f 1408, top-6 55 / 28, 55 / 28, 55 / 31.
constexpr int kFfnSkinnyMaxRows = 160;
// What the combine needs besides ffn_out; done: set when the FFN launches have written y as well.
struct CombineTail {
    const int32_t* inv_perm; const int32_t* topk_idx; const float* topk_w; const int32_t* placement;
    int local_gpu, T, E, k; void* y; bool done;
    const void* late_x;          // the tokens' rows, when the plan may leave some of them to the projections; NULL: it does not
};
int launch_ffn_skinny(const void* a, int N, int d, int f, int E, const void* packed, size_t s13, size_t expert_stride,
                      const int32_t* plan, void* H, float* partial, size_t scratch_bytes, void* out, CombineTail* tail, hipStream_t s);
int launch_ffn_bf16(const void* a, int N, int d, int f, int E, const void* packed, const int32_t* counts,
                    const int32_t* starts, const int32_t* placement, int local_gpu, const int32_t* group_expert,
                    int n_weights, void* out, int32_t* plan, bool plan_ready, void* H, CombineTail* tail, hipStream_t s);

}  // namespace moe
