// Declarations shared by the translation units of libulorl (not part of the public ABI).
#ifndef ULORL_INTERNAL_HPP
#define ULORL_INTERNAL_HPP

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "ulorl.h"

namespace ulorl_detail {

constexpr int kTokBlock = 1024;  // tokens per workgroup of the O(N) epilogue kernels
constexpr int kTokWaves = kTokBlock / 64;

// Workgroups per response that sum its token entropies: about 4096 rows each for responses of average
// length, at most 16.
inline int32_t entropy_slices(int64_t N, int32_t R)
{
    const int64_t s = N / ((int64_t)4096 * R);
    return s < 1 ? 1 : s > 16 ? 16 : (int32_t)s;
}

// Sum over the 64 lanes of a wave in a fixed order, in every lane.  In-register lane permutations instead of
// shuffles through the LDS unit: a double takes about 100 clocks instead of 1000.
__device__ __forceinline__ double wave_sum_f64(double x)
{
    auto add = [](double a, auto perm) {
        const int lo = perm(__double2loint(a)), hi = perm(__double2hiint(a));
        return a + __hiloint2double(hi, lo);
    };
    x = add(x, [](int v) { return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true); });    // lane ^ 1
    x = add(x, [](int v) { return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true); });    // lane ^ 2
    x = add(x, [](int v) { return __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true); });   // 7 - lane in each 8
    x = add(x, [](int v) { return __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, true); });   // 15 - lane in each 16
    double r[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
        r[q] = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), 16 * q), __builtin_amdgcn_readlane(__double2loint(x), 16 * q));
    return (r[0] + r[1]) + (r[2] + r[3]);
}
__device__ __forceinline__ double wave_max_f64(double x)
{
    auto mx = [](double a, auto perm) {
        const int lo = perm(__double2loint(a)), hi = perm(__double2hiint(a));
        return fmax(a, __hiloint2double(hi, lo));
    };
    x = mx(x, [](int v) { return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true); });
    x = mx(x, [](int v) { return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true); });
    x = mx(x, [](int v) { return __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true); });
    x = mx(x, [](int v) { return __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, true); });
    double r[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
        r[q] = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), 16 * q), __builtin_amdgcn_readlane(__double2loint(x), 16 * q));
    return fmax(fmax(r[0], r[1]), fmax(r[2], r[3]));
}

// Partial results that one workgroup hands to the last one of the same launch: relaxed agent-scope
// accesses, which every XCD sees without cache maintenance.  The writer waits for its stores
// (publish_done) before it takes a ticket.
__device__ __forceinline__ void publish(double* p, double v)
{
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), (unsigned long long)__double_as_longlong(v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish(int64_t* p, int64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double published(const double* p)
{
    return __longlong_as_double((long long)__hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ int64_t published(const int64_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// All threads of the workgroup call it after their publish() calls; true in every thread of the workgroup
// that took the last of `count` tickets.  Nothing published is read before the ticket.
__device__ __forceinline__ bool last_workgroup(uint32_t* ticket, uint32_t count)
{
    __shared__ uint32_t mine;
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0);          // this thread's stores have been acknowledged
    __syncthreads();
    if (threadIdx.x == 0)
        mine = count == 1 ? 0u : __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    asm volatile("" ::: "memory");
    return mine == count - 1;
}

}  // namespace ulorl_detail

#include "segment_stats.hpp"

namespace ulorl_detail {

// Arguments of the O(N) epilogue (per-response entropy, token terms, loss reduction).
struct TokenArgs {
    const float* logp;
    const float* entropy;
    const float* lse;
    const int32_t* token_ids;
    const int32_t* cu;
    const int32_t* segment_ids;
    const float* old_logp;
    const float* adv;
    float* gcoef;
    float* loss;        // [1]
    int64_t* counters;  // [4], may be NULL
    uint8_t* mask;
    float* ratio;
    int32_t* seg_out;
    float* resp_entropy;
    uint8_t* resp_gate;
    const uint32_t* sync_fail;  // one word (may be NULL): a wait of the row-cooperative kernel expired
    const uint8_t* defer;       // [N] (may be NULL): rows whose gradient waits for the entropy gate, to be listed
    uint32_t* defer_list;       // [N] workspace, used with defer
    uint32_t* defer_count;      // one word, zero before the epilogue
    uint32_t* ticket;           // one word of workspace: workgroups that have delivered their partial sums
    double* hsum;       // [R * slices] workspace
    int32_t slices;     // entropy_slices(N, R)
    uint32_t* rflags;   // [R] workspace
    double* part_sum;   // [nblk] workspace
    int64_t* part_cnt;  // [nblk * 2] workspace: masked | clipped << 32, positive | status bits << 32
    int64_t N;
    int32_t V, R;
    int32_t is_mode, gate_mode, seg_len;
    double eps_low, eps_high, tau, sigma, D;
    double log_tau, inv_D;   // ln(tau), 1 / D
    SegStatsArgs seg;        // per-segment diagnostics as a by-product (seg.K == 0: not wanted)
};

struct WorkspaceLayout {
    size_t slots, syncfail, hsum, rflags, part_sum, part_cnt, ticket, defer, badcu, zy, defer_list, defer_count, total;
    int64_t nblk;
};

struct ClusterShape {
    int vpt;      // 16-byte vectors per thread
    int pieces;   // workgroups per row (0: shape not supported)
};
ClusterShape cluster_shape(int64_t V, int32_t dt);

// V = 0: no exchange slots (callers that never run the row-cooperative kernel).
WorkspaceLayout workspace_layout(int64_t N, int64_t V, int32_t R);

// Host-side validation of the objective's scalar parameters and required pointers.
int32_t check_objective_args(const int32_t* cu_seqlens, int32_t R, const float* old_logp, const ulorl_params* p,
                             const float* loss, const float* gcoef);

TokenArgs make_token_args(int64_t N, int64_t V, const int32_t* token_ids, const int32_t* cu_seqlens, int32_t R,
                          const int32_t* segment_ids, const float* old_logp, const float* advantages,
                          const ulorl_params* p, float* logp, float* entropy, float* lse, float* gcoef,
                          uint8_t* mpt_mask, float* ratio, int32_t* segment_out, float* resp_entropy,
                          uint8_t* resp_gate, float* loss, int64_t* counters, void* workspace, const WorkspaceLayout& wl,
                          const SegStatsArgs& seg);

// Enqueues response_entropy_kernel and token_terms_kernel.
void launch_token_epilogue(const TokenArgs& a, const WorkspaceLayout& wl, hipStream_t st);

// Launch options of one call, validated and with the defaults filled in.
struct LaunchOpts {
    bool per_row = false;         // ULORL_LAUNCH_PER_ROW
    bool dense_rows = false;      // ULORL_LAUNCH_DENSE_ROWS
    int sync_spins = 1 << 24;
    int gemm_tile = 0;
    int gemm_group_m = 4;
};
int32_t resolve_launch(const ulorl_launch* launch, LaunchOpts* out);

// Validates an optional ulorl_segment_stats against N and turns it into kernel arguments
// (out->K == 0 when st is NULL).
int32_t resolve_segment_stats(const ulorl_segment_stats* st, int64_t N, SegStatsArgs* out);

}  // namespace ulorl_detail

#endif
