// Per-segment training-dynamics diagnostics (Sec. 3.1.2: drift of the importance ratio of older
// segments, share of clipped tokens; Sec. 3.2: entropy and MPT share): device code shared by the
// O(N) epilogue of the forward calls, which produces them from the values it holds in registers,
// and by the standalone ulorl_segment_diagnostics call, which reads them back from a forward call's
// outputs.  Both go through the same functions in the same order, so they give the same bits.
//
// Per workgroup of kSegBlock consecutive tokens: a table [K][7] in LDS; each wave walks the distinct
// segment ids of its lanes (in order of the first lane holding one) and the waves' fixed-tree sums are
// added to the table in a fixed order.  One workgroup then sums the tables.  No floating-point
// atomics: the result depends on the inputs only.
#ifndef ULORL_SEGMENT_STATS_HPP
#define ULORL_SEGMENT_STATS_HPP

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ulorl_detail {

constexpr int kSegBlock = 1024;     // tokens per workgroup (that of the O(N) epilogue)
constexpr int kSegStats = 7;        // count, ratio_sum, ratio_max, clipped, kl_sum, ent_sum, masked
constexpr int kSegMaxK = 1024;      // the table [K][7] of doubles has to fit the default LDS limit

struct SegStatsArgs {
    int32_t K;              // 0: diagnostics not wanted
    double* part;           // [nblk][K][7] workspace
    double* part_oor;       // [nblk] workspace
    int64_t* count;
    double* ratio_sum;
    float* ratio_max;
    int64_t* clipped;
    double* kl_sum;
    double* ent_sum;
    int64_t* masked;
    int64_t* out_of_range;  // may be NULL
};

// One token's seven values from what a forward call stores (fp32 ratio / log-probs / entropy,
// the mask byte, the advantage): v[] and its segment id k (-1: no token, or id outside [0, K),
// then *oor = 1).
__device__ __forceinline__ void seg_token_values(bool valid, int32_t seg, int32_t K, float ratio, float logp,
                                                 bool have_old, float old_logp, float entropy, uint8_t mask,
                                                 float adv, double eps_low, double eps_high, int& k, double (&v)[kSegStats],
                                                 double& oor)
{
    k = -1;
    oor = 0.0;
#pragma unroll
    for (int s = 0; s < kSegStats; ++s) v[s] = 0.0;
    if (!valid) return;
    if (seg < 0 || seg >= K) {
        oor = 1.0;
        return;
    }
    k = seg;
    const double r = (double)ratio;
    const double A = (double)adv;
    const double c = fmin(fmax(r, 1.0 - eps_low), 1.0 + eps_high);
    v[0] = 1.0;
    v[1] = r;
    v[2] = r;
    v[3] = (r * A <= c * A) ? 0.0 : 1.0;
    v[4] = have_old ? (double)old_logp - (double)logp : 0.0;
    v[5] = (double)entropy;
    v[6] = mask ? 1.0 : 0.0;
}

// Adds the workgroup's tokens to table (LDS, [K][7]) and hands it to `out` (global, [K][7], publish());
// returns the workgroup's count of out-of-range tokens on every thread.  All kSegBlock threads must call.
// Every wave forms the sums of up to kSegEntries distinct ids of its lanes at a time (counts by ballot); then the
// wave that holds the first entry of an id adds all entries of that id to the table, in the entries' order.  A pass
// costs what the ids present cost, not the size of the table.  The call on 65536 tokens, the waves taking turns /
// every slot of the table scanning all entries / this, us: 8 ids in runs 26 / 11.1 / 10.6, in no order 103 / 20.4 / 19.2;
// 1024 ids in runs 165 / 196 / 73, in no order 837 / 993 / 165.
constexpr int kSegEntries = 4;
__device__ __forceinline__ double seg_block_partials(int k, const double (&v)[kSegStats], double oor, int32_t K,
                                                     double* table, double* __restrict__ out)
{
    constexpr int NW = kSegBlock / 64;
    constexpr int NE = NW * kSegEntries;
    static_assert(NE == 64, "a ballot covers the entries");
    __shared__ double entry[NE][8];                  // a row per entry: a wave reads or writes one at a time
    __shared__ int entry_key[NE];
    __shared__ int oor_wave[NW];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slots = K * kSegStats;
    for (int i = tid; i < slots; i += kSegBlock) table[i] = 0.0;
    const int oor_count = __popcll(__ballot(oor != 0.0));
    if (lane == 0) oor_wave[wave] = oor_count;
    unsigned long long remaining = __ballot(k >= 0);
    int more;
    do {
#pragma unroll 1
        for (int e = 0; e < kSegEntries; ++e) {
            const int at = e * NW + wave;          // the waves' first ids, then their second ones, ...: an id's sums then fall to different waves
            int key = -1;
            if (remaining != 0ull) {
                key = __builtin_amdgcn_readlane(k, __ffsll((long long)remaining) - 1);
                const bool mine = k == key;
                const unsigned long long members = __ballot(mine);
                remaining &= ~members;
                const double ratio = wave_sum_f64(mine ? v[1] : 0.0), top = wave_max_f64(mine ? v[2] : 0.0);
                const double kl = wave_sum_f64(mine ? v[4] : 0.0), ent = wave_sum_f64(mine ? v[5] : 0.0);
                const int clipped = __popcll(__ballot(mine && v[3] != 0.0)), masked = __popcll(__ballot(mine && v[6] != 0.0));
                if (lane == 0) {
                    entry[at][0] = (double)__popcll(members);
                    entry[at][1] = ratio;
                    entry[at][2] = top;
                    entry[at][3] = (double)clipped;
                    entry[at][4] = kl;
                    entry[at][5] = ent;
                    entry[at][6] = (double)masked;
                }
            }
            if (lane == 0) entry_key[at] = key;
        }
        more = __syncthreads_or(remaining != 0ull);
        const int key_of_lane = entry_key[lane];
#pragma unroll 1
        for (int e = 0; e < kSegEntries; ++e) {
            const int at = e * NW + wave;
            const int key = __builtin_amdgcn_readlane(key_of_lane, at);
            unsigned long long same = __ballot(key_of_lane == key);
            if (key < 0 || __ffsll((long long)same) - 1 != at) continue;      // uniform: no entry, or not the id's first
            if (lane < kSegStats) {
                double t = table[key * kSegStats + lane];
                while (same != 0ull) {                                        // four reads in flight; 0 changes neither sums nor maxima
                    double x[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        x[u] = same != 0ull ? entry[__ffsll((long long)same) - 1][lane] : 0.0;
                        same &= same - 1ull;
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) t = lane == 2 ? fmax(t, x[u]) : t + x[u];
                }
                table[key * kSegStats + lane] = t;
            }
        }
        __syncthreads();
    } while (more);
    for (int i = tid; i < slots; i += kSegBlock) publish(out + i, table[i]);
    int total = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) total += oor_wave[w];
    return (double)total;
}

// Final sums over the workgroups' tables, by ONE workgroup of kSegBlock threads.  Slot (k, s) is
// summed by a group of T threads (T = the largest power of two with K * 7 * T <= kSegBlock, between 1 and
// 16), each over the blocks b = j, j + T, ... in order, then the T partial sums in order.
__device__ __forceinline__ void seg_finalize(const SegStatsArgs& a, int64_t nblk, double* scratch /* [kSegBlock] */)
{
    const int tid = threadIdx.x;
    const int slots = a.K * kSegStats;
    int T = 1;
    while (T < 16 && slots * T * 2 <= kSegBlock) T *= 2;
    for (int base = 0; base < slots; base += kSegBlock / T) {
        const int slot = base + tid / T;
        const int j = tid % T;
        double acc = 0.0;
        const bool is_max = (slot % kSegStats) == 2;
        if (slot < slots && tid / T < kSegBlock / T) {
            const double* p = a.part + (int64_t)j * slots + slot;
            const int64_t step = (int64_t)T * slots;
            int64_t b = j;
            for (; b + 7 * T < nblk; b += 8 * T) {              // eight loads in flight
                double x[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    x[q] = published(p);
                    p += step;
                }
#pragma unroll
                for (int q = 0; q < 8; ++q) acc = is_max ? fmax(acc, x[q]) : acc + x[q];
            }
            for (; b < nblk; b += T) {
                const double x = published(p);
                p += step;
                acc = is_max ? fmax(acc, x) : acc + x;
            }
        }
        __syncthreads();
        scratch[tid] = acc;
        __syncthreads();
        if (slot < slots && j == 0) {
            double s = scratch[tid];
            for (int q = 1; q < T; ++q) s = is_max ? fmax(s, scratch[tid + q]) : s + scratch[tid + q];
            const int k = slot / kSegStats;
            switch (slot % kSegStats) {
            case 0: a.count[k] = (int64_t)s; break;
            case 1: a.ratio_sum[k] = s; break;
            case 2: a.ratio_max[k] = (float)s; break;
            case 3: a.clipped[k] = (int64_t)s; break;
            case 4: a.kl_sum[k] = s; break;
            case 5: a.ent_sum[k] = s; break;
            default: a.masked[k] = (int64_t)s; break;
            }
        }
    }
    // out-of-range tokens
    double o = 0.0;
    for (int64_t b = tid; b < nblk; b += kSegBlock) o += published(a.part_oor + b);
    o = wave_sum_f64(o);
    __syncthreads();
    if ((tid & 63) == 0) scratch[tid >> 6] = o;
    __syncthreads();
    if (tid == 0 && a.out_of_range) {
        double s = 0.0;
        for (int q = 0; q < kSegBlock / 64; ++q) s += scratch[q];
        *a.out_of_range = (int64_t)s;
    }
}

inline size_t seg_align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

inline size_t seg_workspace_bytes(int64_t N, int32_t K)
{
    const size_t nblk = (size_t)((N + kSegBlock - 1) / kSegBlock);
    return seg_align_up(nblk * (size_t)K * kSegStats * sizeof(double), 256) + seg_align_up(nblk * sizeof(double), 256);
}

}  // namespace ulorl_detail

#endif
