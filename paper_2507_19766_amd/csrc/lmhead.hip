// lm_head variant of the UloRL token loss for gfx950: logits = hidden . W are produced tile by
// tile on the matrix cores (gemm_tile.hpp) and consumed in registers; the [N, V] logits tensor never
// exists in memory.
//
// Products (acc[m, n] = sum_k A[m, k] B[n, k], see gemm_tile.hpp for the two operand layouts):
//   forward   z^T[v, t]        A = W (K_COLS), B = hidden (K_ROWS)       online softmax statistics per token
//   backward  z^T again                                                  dz = g (onehot - softmax), stored per
//                                                                        vocabulary chunk as dZ[t, v]
//             dHidden[t, k]    A = W (K_ROWS), B = dZ (K_ROWS)           fp32 accumulation across chunks
//             dW[k, v]         A = dZ (K_COLS), B = hidden (K_COLS)      each element written once
// Every operand is read in the layout it has: no transposed copies of W, hidden or dZ exist.  In the z^T
// orientation a lane of a result block holds one token column and four vocabulary rows, which makes
// the softmax reductions mostly lane-local and dZ[t, v] rows contiguous per lane.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <mutex>
#include <type_traits>
#include <unordered_map>

#include "gemm_tile.hpp"
#include "lmhead_plan.hpp"
#include "ulorl.h"
#include "ulorl_internal.hpp"

using namespace ulorl_detail;

#pragma clang fp contract(off)

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kEmpty = -1.0e30f;
constexpr float kWide = 536870912.0f;        // 2^29, see lmhead_stats_kernel

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

#define ULORL_TILE_KERNEL(NT, WAVES_PER_SIMD) \
    __global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WAVES_PER_SIMD, WAVES_PER_SIMD)))

// ---------------------------------------------------------------------------------------------
// storing a result tile: element (n, m) at C[n * ldc + m]
// ---------------------------------------------------------------------------------------------
// fp32, straight from the registers: a lane's four rows m are one 16-byte access (C 16-byte aligned,
// ldc a multiple of 4, when `wide`); ACCUM adds to what is there.
template <bool ACCUM, class Tile>
__device__ __forceinline__ void store_tile_f32(const Tile& T, float* __restrict__ C, int64_t ldc, int M, int N, int m0, int n0, bool wide)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < Tile::NJ; ++j) {
        if (j >= T.blocks()) continue;
        const int n = n0 + T.col_off(wave, j) + (lane & 15);
        if (n >= N) continue;
#pragma unroll
        for (int i = 0; i < Tile::MI; ++i) {
            const int m = m0 + Tile::row_off(wave, i) + 4 * (lane >> 4);
            float* dst = C + (int64_t)n * ldc + m;
            if (wide && m + 4 <= M) {
                f32x4 x = T.acc[i][j];
                if (ACCUM) x += *reinterpret_cast<const f32x4*>(dst);
                *reinterpret_cast<f32x4*>(dst) = x;
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (m + r < M) dst[r] = ACCUM ? dst[r] + T.acc[i][j][r] : T.acc[i][j][r];
            }
        }
    }
}

// bf16 tiles, straight from the registers too.  A lane of a result block holds four rows m of a column n, packed 8 bytes; of
// two blocks below each other (x: rows m .. m + 15, y: the next 16) lanes trade halves so that each has eight rows in
// one 16-byte vector and four lanes 64 contiguous bytes.  A dz tile's work after its product took 20400 clocks with its
// terms fetched column by column and its values stored through an image in LDS (5300 of them), and takes 10000 now;
// 32768 x 8192 x 2048 dz alone 924 us before, 826 now.
__device__ __forceinline__ void store_bf16_pair(bf16_t* __restrict__ column, int m, int m_end, bool valid, u32x2 x, u32x2 y)
{
    const auto lo = __builtin_amdgcn_permlane16_swap(x[0], y[0], false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(x[1], y[1], false, false);
    const int row = ((int)threadIdx.x >> 4) & 3;
    m += (row & 1) * 16 + (row >> 1) * 8;
    if (valid && m < m_end) *reinterpret_cast<u32x4*>(column + m) = u32x4{lo[0], hi[0], lo[1], hi[1]};
}

// ---------------------------------------------------------------------------------------------
// the product on its own: C[m, n] = sum_k A[m, k] B[n, k], fp32, row-major
// ---------------------------------------------------------------------------------------------
struct GemmArgs {
    Operand a, b;
    int K;
    float* C;
    int64_t ldc;
    int wide;           // C allows 16-byte accesses
};

template <class Tile>
ULORL_TILE_KERNEL(Tile::NT, Tile::WAVES_PER_SIMD)
void gemm_tn_kernel(const GemmArgs g, int group_m)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    int tile_m, tile_n;
    if (!tile_coords((int)blockIdx.x, (g.a.count + Tile::BN - 1) / Tile::BN, (g.b.count + Tile::BM - 1) / Tile::BM, group_m, tile_m, tile_n))
        return;
    // C has n contiguous: B takes the engine's m side
    const int m0 = tile_n * Tile::BM;
    const ColumnTile c = Tile::columns(g.a.count, tile_m);
    Tile T;
    T.init(lds_raw);
    T.run(g.b, m0, g.a, c, g.K);
    store_tile_f32<false>(T, g.C, g.ldc, g.b.count, g.a.count, m0, c.first, g.wide != 0);
}

// d_hidden[t, :] = bf16(sum over slabs of acc[slab][pos[t], :]) (pos == NULL: row t itself); rows without a
// live position are zero.  One thread converts 8 elements (Hd is a multiple of 8; both buffers
// 16-byte aligned).
__global__ void dhidden_finish_kernel(const float* __restrict__ acc, int slabs, const int* __restrict__ pos, int64_t N, int Hd,
                                      bf16_t* __restrict__ dst)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int vpr = Hd / 8;
    const int64_t t = i / vpr;
    if (t >= N) return;
    const int c = (int)(i - t * vpr) * 8;
    const int64_t j = pos != nullptr ? (int64_t)pos[t] : t;
    u32x4 out = {0u, 0u, 0u, 0u};
    if (j >= 0) {
        const float* q = acc + j * Hd + c;
        f32x4 lo = *reinterpret_cast<const f32x4*>(q), hi = *reinterpret_cast<const f32x4*>(q + 4);
        for (int s = 1; s < slabs; ++s) {
            q += N * Hd;
            lo += *reinterpret_cast<const f32x4*>(q);
            hi += *reinterpret_cast<const f32x4*>(q + 4);
        }
        out = u32x4{pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3]), pack_bf16x2(hi[0], hi[1]), pack_bf16x2(hi[2], hi[3])};
    }
    *reinterpret_cast<u32x4*>(dst + t * Hd + c) = out;
}

// ---------------------------------------------------------------------------------------------
// live rows of the backward pass
// ---------------------------------------------------------------------------------------------
// A token whose coefficient is zero (masked as a well-mastered positive token, on the clipped
// branch, zero advantage, or flagged) contributes nothing to d_W and has a zero d_hidden row.  The
// backward pass therefore runs its three products over the LIVE rows only: their indices are
// collected in order (so that every sum keeps a fixed order), hidden is gathered, and the kernels
// take the live count from device memory.  The dynamic mask of the method makes this count
// much smaller than N whenever many positive tokens are mastered.
__device__ __forceinline__ bool row_has_gradient(float g, float l, int32_t y, int32_t V)
{
    return (g != 0.0f) && (fabsf(g) <= 3.0e38f) && (fabsf(l) <= 3.0e38f) && y >= 0 && y < V;
}

// Inclusive prefix sum over a workgroup of kLiveBlock threads; *total = the workgroup's sum.
__device__ __forceinline__ int live_block_scan(int v, int* wave_tot, int* total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int up = __shfl_up(v, off);
        if (lane >= off) v += up;
    }
    __syncthreads();
    if (lane == 63) wave_tot[wave] = v;
    __syncthreads();
    int before = 0, all = 0;
    for (int w = 0; w < kLiveBlock / 64; ++w) {
        const int x = wave_tot[w];
        before += w < wave ? x : 0;
        all += x;
    }
    *total = all;
    return v + before;
}

__global__ __launch_bounds__(kLiveBlock) void live_count_kernel(const float* __restrict__ gcoef, const float* __restrict__ lse,
                                                                const int32_t* __restrict__ token_ids, float grad_out,
                                                                int64_t N, int32_t V, int* __restrict__ block_count)
{
    __shared__ int wave_tot[kLiveBlock / 64];
    const int64_t t = (int64_t)blockIdx.x * kLiveBlock + threadIdx.x;
    const int live = t < N && row_has_gradient(gcoef[t] * grad_out, lse[t], token_ids[t], V);
    int total;
    live_block_scan(live, wave_tot, &total);
    if (threadIdx.x == 0) block_count[blockIdx.x] = total;
}

// One workgroup: exclusive prefix sums of the blocks' counts (in place) and the total.
__global__ __launch_bounds__(kLiveBlock) void live_scan_kernel(int* __restrict__ block_count, int nblk, int* __restrict__ n_live)
{
    __shared__ int wave_tot[kLiveBlock / 64];
    int base = 0;
    for (int b0 = 0; b0 < nblk; b0 += kLiveBlock) {
        const int b = b0 + threadIdx.x;
        const int c = b < nblk ? block_count[b] : 0;
        int total;
        const int incl = live_block_scan(c, wave_tot, &total);
        if (b < nblk) block_count[b] = base + incl - c;
        base += total;
    }
    if (threadIdx.x == 0) *n_live = base;
}

// pos[t] = position of row t among the live rows (-1: not live); row_map[position] = t.
__global__ __launch_bounds__(kLiveBlock) void live_fill_kernel(const float* __restrict__ gcoef, const float* __restrict__ lse,
                                                               const int32_t* __restrict__ token_ids, float grad_out,
                                                               int64_t N, int32_t V, const int* __restrict__ block_offset,
                                                               int* __restrict__ pos, int* __restrict__ row_map)
{
    __shared__ int wave_tot[kLiveBlock / 64];
    const int64_t t = (int64_t)blockIdx.x * kLiveBlock + threadIdx.x;
    const int live = t < N && row_has_gradient(gcoef[t] * grad_out, lse[t], token_ids[t], V);
    int total;
    const int incl = live_block_scan(live, wave_tot, &total);
    if (t < N) {
        const int p = block_offset[blockIdx.x] + incl - 1;
        pos[t] = live ? p : -1;
        if (live) row_map[p] = (int)t;
    }
}

// The three kernels above in one launch, for up to kLiveRecountRows rows: every workgroup counts the rows
// before its own itself (three independent loads from cache per row, at most 3 * kLiveRecountRows / kLiveBlock
// per thread), which is cheaper than two more launches of 4.5 us each: 32 x 1024 rows are recounted in about 7 us.
constexpr int64_t kLiveRecountRows = 32768;
__global__ __launch_bounds__(kLiveBlock) void live_rows_kernel(const float* __restrict__ gcoef, const float* __restrict__ lse,
                                                               const int32_t* __restrict__ token_ids, float grad_out,
                                                               int64_t N, int32_t V, int* __restrict__ pos,
                                                               int* __restrict__ row_map, int* __restrict__ n_live)
{
    __shared__ int wave_tot[kLiveBlock / 64];
    int before = 0;
#pragma unroll 4
    for (int b = 0; b < (int)blockIdx.x; ++b) {
        const int64_t t = (int64_t)b * kLiveBlock + threadIdx.x;
        before += row_has_gradient(gcoef[t] * grad_out, lse[t], token_ids[t], V) ? 1 : 0;
    }
    int base, total;
    live_block_scan(before, wave_tot, &base);
    const int64_t t = (int64_t)blockIdx.x * kLiveBlock + threadIdx.x;
    const int live = t < N && row_has_gradient(gcoef[t] * grad_out, lse[t], token_ids[t], V);
    const int incl = live_block_scan(live, wave_tot, &total);
    if (t < N) {
        const int p = base + incl - 1;
        pos[t] = live ? p : -1;
        if (live) row_map[p] = (int)t;
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *n_live = base + total;
}

// dst[j, c] = src[row_map[j], c] (row_map == NULL: src[j, c]) for j < rows (*n_rows if given) and c < cols;
// zeros up to the next multiple of 64 rows and up to dst_cols columns: contractions run over whole K
// tiles of 64.  cols, dst_cols multiples of 8, 16-byte aligned rows; grid over (rows + 63) / 64 * 64 rows.
__global__ __launch_bounds__(256) void copy_rows_padded_kernel(const bf16_t* __restrict__ src, int64_t ld_src, int cols,
                                                               const int* __restrict__ row_map, const int* __restrict__ n_rows,
                                                               int64_t rows, bf16_t* __restrict__ dst, int64_t dst_cols)
{
    const int64_t vpr = dst_cols / 8;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t j = i / vpr;
    if (n_rows != nullptr) rows = min(rows, (int64_t)*n_rows);
    if (j >= (rows + 63) / 64 * 64) return;
    const int64_t v = i - j * vpr;
    u32x4 x = {0u, 0u, 0u, 0u};
    if (j < rows && v * 8 < cols)
        x = *reinterpret_cast<const u32x4*>(src + (row_map != nullptr ? (int64_t)row_map[j] : j) * ld_src + v * 8);
    *reinterpret_cast<u32x4*>(dst + j * dst_cols + v * 8) = x;
}

// ---------------------------------------------------------------------------------------------
// forward: softmax statistics from z^T tiles
// ---------------------------------------------------------------------------------------------
// (m, S, T) with T = sum e^(z-m) (z-m) in natural units; exact when the maxima coincide.
__device__ __forceinline__ void merge_nat(float& m, float& S, float& T, float m2, float S2, float T2)
{
    const float M = fmaxf(m, m2);
    const float d1 = m - M, d2 = m2 - M;
    const float s1 = fast_exp2(d1 * kLog2e), s2 = fast_exp2(d2 * kLog2e);
    T = s1 * fmaf(d1, S, T) + s2 * fmaf(d2, S2, T2);
    S = s1 * S + s2 * S2;
    m = M;
}

// f(integral_constant i) for i = 0 .. N - 1.
template <int N, int I = 0, class F>
__device__ __forceinline__ void each_index(F f)
{
    f(std::integral_constant<int, I>{});
    if constexpr (I + 1 < N) each_index<N, I + 1>(f);
}

// One workgroup: the statistics of one tile of tokens over one slice of the vocabulary.
template <class Tile>
ULORL_TILE_KERNEL(Tile::NT, Tile::WAVES_PER_SIMD)
void lmhead_stats_kernel(const Operand W, const Operand H, int K, const int32_t* __restrict__ token_ids, int v_per_split,
                         int splits, StatQuad* __restrict__ partial, int group_m)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    __shared__ float red[Tile::WAVES_M][Tile::BN][3];
    __shared__ float chosen[Tile::BN];
    __shared__ int32_t token[Tile::BN];
    const int V = W.count, Ntok = H.count;
    int t_tile, split;
    if (!tile_coords((int)blockIdx.x, (Ntok + Tile::BN - 1) / Tile::BN, splits, group_m, t_tile, split)) return;
    const ColumnTile cols = Tile::columns(Ntok, t_tile);
    const int t0 = cols.first;
    const int vb = split * v_per_split;
    const int ve = min(V, vb + v_per_split);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int quad = lane >> 4;
    constexpr int MI = Tile::MI, NJ = Tile::NJ;

    // Per token column of this lane: running max m, S + Sc = sum 2^(z log2e - fl(m log2e)), T = the same weighted
    // with its exponent (log2 units).  The exponents carry the rounding residual of fl(m log2e), the
    // same for every term; it is taken out once at the end.  The residual grows with m: from kWide on it
    // exceeds 32 and soon the range of 2^x, so a workgroup that met such a maximum (S is 0 or not finite, or the last
    // maximum is one; its S is handed on as NaN) walks its tiles again and takes those columns' sums from exponents of z - m.
    float m[NJ], S[NJ], Sc[NJ], T[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        m[j] = kEmpty; S[j] = 0.0f; Sc[j] = 0.0f; T[j] = 0.0f;
    }
    Tile G;
    G.init(lds_raw);
    G.begin(W, vb, H, cols, K);
    for (int c = threadIdx.x; c < Tile::BN; c += Tile::NT) {
        chosen[c] = kEmpty;
        token[c] = t0 + c < Ntok ? token_ids[t0 + c] : -1;
    }
    __syncthreads();

    // One tile, finished, and the next one begun: its first copies go along with the work on this one's results.  That work has no
    // branch in it: the accumulators of TileLarge lie in registers that only moves can read, and what a second block
    // uses is moved at once, all 256.  RAGGED: the tile reaches past the end of this workgroup's vocabulary range.
    auto absorb_tile = [&](int v0, auto ragged_c) {
        constexpr bool RAGGED = decltype(ragged_c)::value;
        G.finish_keep(m, S, Sc, T);
        int col0 = lane & 15, my_rows = Tile::wave_m(wave) * 64 + quad * 4;      // my rows of a tile: bits 2, 3 and 6 are these
        asm volatile("" : "+v"(col0), "+v"(my_rows));         // nothing formed from them is kept over the loop, in registers it needs
        const bool last = v0 + Tile::BM >= ve;
        G.begin(W, last ? v0 : v0 + Tile::BM, H, cols, last ? 0 : K);
        each_index<NJ>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            // the chosen token's logit, if it is one of this lane's (rare); otherwise the store goes nowhere
            const int col = G.col_off(wave, j) + col0;
            const int dy = token[col] - v0;
            const int rows = j < G.blocks() ? min(Tile::BM, ve - v0) : 0;
            const bool mine = ((uint32_t)dy < (uint32_t)rows) & ((dy & 0x4c) == my_rows);
            const float zy = G.template pick<j>(mine ? ((dy >> 3) & 16) | ((dy >> 2) & 12) | (dy & 3) : -1);
            *(mine ? &chosen[col] : &red[0][0][0]) = zy;
            float z[MI][4];
            each_index<MI>([&](auto ic) { G.template take<decltype(ic)::value, j>(z[decltype(ic)::value]); });
            float cm = kEmpty;
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (!RAGGED || v0 + Tile::row_off(wave, i) + 4 * quad + r < ve) cm = fmaxf(cm, z[i][r]);
            const float mn = fmaxf(m[j], cm);
            const float mL = mn * kLog2e;
            const float d = m[j] * kLog2e - mL;               // <= 0
            const float sc = fast_exp2(d);
            const float Tn = sc * fmaf(d, S[j], T[j]);
            const float Sn = sc * S[j];
            const float Scn = sc * Sc[j];
            float ps[4] = {0.0f, 0.0f, 0.0f, 0.0f}, pt[4] = {0.0f, 0.0f, 0.0f, 0.0f};   // this tile's terms first, then one TwoSum
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float x = fmaf(z[i][r], kLog2e, -mL);
                    float e = fast_exp2(x);
                    if (RAGGED && v0 + Tile::row_off(wave, i) + 4 * quad + r >= ve) { x = 0.0f; e = 0.0f; }
                    ps[r] += e;
                    pt[r] = fmaf(e, x, pt[r]);
                }
            const float part = (ps[0] + ps[1]) + (ps[2] + ps[3]);
            const float tsum = Sn + part;
            const float bv = tsum - Sn;
            const float err = (Sn - (tsum - bv)) + (part - bv);
            S[j] = tsum; Sc[j] = Scn + err; T[j] = Tn + ((pt[0] + pt[1]) + (pt[2] + pt[3])); m[j] = mn;
            __builtin_amdgcn_sched_barrier(0);                // no column's values are taken before the last one's are used up
        });
    };
    int v0 = vb;
    for (; v0 + Tile::BM <= ve; v0 += Tile::BM) absorb_tile(v0, std::false_type{});
    if (v0 < ve) absorb_tile(v0, std::true_type{});
    ULORL_WAIT_VMEM(0);                                       // the zeros that the last begin() copied
    __syncthreads();
    // four lanes (L, L ^ 16, L ^ 32, L ^ 48) share a token column; then the waves stacked along the vocabulary
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        if (j >= G.blocks()) continue;
        const float delta = m[j] > 0.5f * kEmpty ? fmaf(m[j], kLog2e, -(m[j] * kLog2e)) : 0.0f;
        const float un = fast_exp2(-delta);
        // a lane without a row inside the vocabulary has met nothing: m is kEmpty and S 0
        const bool wide = m[j] > kEmpty && (!(S[j] > 0.0f && S[j] < 3.0e38f) || fabsf(m[j]) >= kWide);
        float mm = m[j], SS = wide ? __builtin_nanf("") : un * (S[j] + Sc[j]), TT = un * fmaf(-delta, S[j], T[j]) * kLn2;
#pragma unroll
        for (int off = 16; off <= 32; off <<= 1) {
            const float m2 = __shfl_xor(mm, off), S2 = __shfl_xor(SS, off), T2 = __shfl_xor(TT, off);
            merge_nat(mm, SS, TT, m2, S2, T2);
        }
        if (lane < 16) {
            float* q = red[Tile::wave_m(wave)][G.col_off(wave, j) + lane];
            q[0] = mm; q[1] = SS; q[2] = TT;
        }
    }
    __syncthreads();
    bool any_wide = false;
    for (int c = threadIdx.x; c < Tile::BN; c += Tile::NT) {
        float mm = red[0][c][0], SS = red[0][c][1], TT = red[0][c][2];
#pragma unroll
        for (int w = 1; w < Tile::WAVES_M; ++w) merge_nat(mm, SS, TT, red[w][c][0], red[w][c][1], red[w][c][2]);
        const int t = t0 + c;
        const bool mine = c < cols.width && t < Ntok;
        if (mine) partial[(int64_t)split * Ntok + t] = StatQuad{mm, SS, TT, chosen[c]};
        chosen[c] = mm;
        token[c] = mine && !(SS > 0.0f && SS < 3.0e38f);
        any_wide |= token[c] != 0;
    }
    // The OR over the waves goes through a stage, which no wave reads any more: __syncthreads_or brings LDS of its own, after
    // which the stages no longer start at a multiple of 8 KB, and that costs 1.5 % of the kernel.
    const int wave_wide = __any(any_wide);
    int* flags = reinterpret_cast<int*>(lds_raw);
    if (lane == 0) flags[wave] = wave_wide;
    __syncthreads();
    if (!__any(lane < Tile::NW && flags[lane] != 0)) return;
    // Rare: the tiles once more, for the columns marked in token[], whose maxima (in chosen[]) are known now.
    __syncthreads();
    float S2[NJ], T2[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) S2[j] = T2[j] = 0.0f;
#pragma unroll 1
    for (v0 = vb; v0 < ve; v0 += Tile::BM) {
        G.run(W, v0, H, cols, K);
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const float top = chosen[G.col_off(wave, j) + (lane & 15)];
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float x = (G.acc[i][j][r] - top) * kLog2e;
                    const float e = fast_exp2(x);
                    if (v0 + Tile::row_off(wave, i) + 4 * quad + r < ve) {
                        S2[j] += e;
                        T2[j] = fmaf(e, x, T2[j]);
                    }
                }
        }
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        if (j >= G.blocks()) continue;
#pragma unroll
        for (int off = 16; off <= 32; off <<= 1) {
            S2[j] += __shfl_xor(S2[j], off);
            T2[j] += __shfl_xor(T2[j], off);
        }
        if (lane < 16) {
            float* q = red[Tile::wave_m(wave)][G.col_off(wave, j) + lane];
            q[1] = S2[j]; q[2] = T2[j];
        }
    }
    __syncthreads();
    for (int c = threadIdx.x; c < Tile::BN; c += Tile::NT) {
        if (token[c] == 0) continue;
        float SS = 0.0f, TT = 0.0f;
#pragma unroll
        for (int w = 0; w < Tile::WAVES_M; ++w) {
            SS += red[w][c][1];
            TT += red[w][c][2];
        }
        StatQuad& q = partial[(int64_t)split * Ntok + t0 + c];
        q.S = SS;
        q.T = TT * kLn2;
    }
}

// LANES lanes per token: each merges every LANES-th slice in order, then a fixed shuffle tree.  (One thread per token walked up
// to 128 slices one dependent load after the other: 22 us at 64 slices, 5 with eight lanes.)  32 lanes beyond 64 slices.
template <int LANES>
__global__ __launch_bounds__(256) void lmhead_stats_merge_kernel(const StatQuad* __restrict__ partial, int splits, int Ntok, int V,
                                                                 const int32_t* __restrict__ token_ids, float* __restrict__ lse,
                                                                 float* __restrict__ logp, float* __restrict__ entropy)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int t = (int)(i / LANES), part = (int)(i % LANES);
    StatQuad q = {kEmpty, 0.0f, 0.0f, kEmpty};
    if (t < Ntok) {
#pragma unroll 4
        for (int s = part; s < splits; s += LANES) {
            const StatQuad p = partial[(int64_t)s * Ntok + t];
            merge_nat(q.m, q.S, q.T, p.m, p.S, p.T);
            q.zy = fmaxf(q.zy, p.zy);
        }
    }
#pragma unroll
    for (int off = 1; off < LANES; off <<= 1) {
        const float m2 = __shfl_xor(q.m, off), S2 = __shfl_xor(q.S, off), T2 = __shfl_xor(q.T, off), z2 = __shfl_xor(q.zy, off);
        merge_nat(q.m, q.S, q.T, m2, S2, T2);
        q.zy = fmaxf(q.zy, z2);
    }
    if (t >= Ntok || part != 0) return;
    const float lnS = logf(q.S);
    const int32_t y = token_ids[t];
    lse[t] = q.m + lnS;
    logp[t] = (y >= 0 && y < V) ? (q.zy - q.m) - lnS : __builtin_nanf("");
    entropy[t] = lnS - q.T / q.S;
}

// ---------------------------------------------------------------------------------------------
// backward
// ---------------------------------------------------------------------------------------------
// dz of one vocabulary chunk [vc0, vc0 + cw) (cw a multiple of 64; columns at or beyond V are written as
// zero).  H holds the token rows of the product; with a row map they are the gathered live rows and
// token column t stands for row row_map[t] of the per-token arrays.
struct DzArgs {
    Operand W, H;                    // W.count = V
    int K;                           // padded hidden size
    int vc0, cw;
    const int32_t* token_ids;
    const float* lse;
    const float* gcoef;
    float grad_out;
    bf16_t* dZ;                      // [token, v - vc0]
    int64_t ld;
    const int* row_map;
};

struct DzTerm {
    float g_mag, c;                  // -|g| (0: no gradient), log2|g| - lse log2e
    uint32_t flip;                   // sign bits of a packed pair, set for g > 0
    int dy;                          // row of the chosen token in the tile, or -1
};

// The tile of workgroup `bid`.  Ntok: the number of token rows; rows up to the next multiple of 64 are
// written as zeros (the d_W product contracts over whole K tiles of 64 tokens).
template <class Tile>
__device__ __forceinline__ void lmhead_dz_block(int bid, const DzArgs& a, int Ntok, int group_m, unsigned char* lds_raw)
{
    int v_tile, t_tile;
    if (!tile_coords(bid, (a.cw + Tile::BM - 1) / Tile::BM, (Ntok + Tile::BN - 1) / Tile::BN, group_m, v_tile, t_tile)) return;
    const int v0 = a.vc0 + v_tile * Tile::BM;
    const ColumnTile cols = Tile::columns(Ntok, t_tile);
    const int t0 = cols.first;
    const int V = a.W.count;
    const int vend = min(V, a.vc0 + a.cw);
    // Per token column:  dz = g (onehot - e^(z - lse)) = s (2^(z log2e + c) - |g| onehot)  with s = -sign(g),
    // c = log2|g| - lse log2e.  The magnitudes are computed and rounded; a negative s is applied to the packed pair by
    // flipping sign bits (rounding to nearest even is symmetric); a column without a gradient (zero coefficient, flagged row,
    // padding) is zeroed on the packed pair; the chosen token's element is rewritten by the one lane that holds it.
    // Per element that leaves one FMA, one exponential and half a conversion in the common path.
    // The terms of the tile's columns are fetched while its first copies are in flight: fetched by each lane for its eight columns
    // after the product, two loads deep, they took 6 us of a tile's 58 (one wave per SIMD covers no wait).
    DzTerm* terms = reinterpret_cast<DzTerm*>(lds_raw + Tile::LDS_BYTES);
    Tile G;
    G.init(lds_raw);
    Operand H = a.H;
    H.count = Ntok;
    G.begin(a.W, v0, H, cols, a.K);          // v0 < V: the padding columns of a chunk never fill a tile
    for (int n = threadIdx.x; n < Tile::BN; n += Tile::NT) {
        DzTerm q = {0.0f, 0.0f, 0u, -1};
        const int t = t0 + n;
        if (t < Ntok) {
            const int tt = a.row_map != nullptr ? a.row_map[t] : t;
            const float gg = a.gcoef[tt] * a.grad_out;
            const float l = a.lse[tt];
            const int32_t yy = a.token_ids[tt];
            if (row_has_gradient(gg, l, yy, V)) {
                q.g_mag = -fabsf(gg);
                q.c = fmaf(-l, kLog2e, log2f(fabsf(gg)));
                q.flip = gg > 0.0f ? 0x80008000u : 0u;
                if (yy >= v0 && yy < min(vend, v0 + Tile::BM)) q.dy = yy - v0;
            }
        }
        terms[n] = q;
    }
    G.finish();                              // its barriers stand between the terms' stores and their use

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int quad = lane >> 4;
    const int my_rows = Tile::wave_m(wave) * 64 + quad * 4;       // of the tile: those whose bits 2, 3 and 6 are these
    const bool ragged = v0 + Tile::BM > vend;     // uniform: the tile reaches past the end of the vocabulary
    const int n_end = min(cols.width, (Ntok + 63) / 64 * 64 - t0), m_end = a.vc0 + a.cw - v0;
    bf16_t* const dst = a.dZ + (int64_t)t0 * a.ld + (v0 - a.vc0);
#pragma unroll
    for (int j = 0; j < Tile::NJ; ++j) {
        if (j >= G.blocks()) continue;
        const int n = G.col_off(wave, j) + (lane & 15);
        const DzTerm q = terms[n];
        const uint32_t keep = q.g_mag != 0.0f ? 0xffffffffu : 0u;
        const bool mine = q.dy >= 0 && (q.dy & 0x4c) == my_rows;
        // CARE: with columns beyond the vocabulary, or the chosen token of one of the wave's columns (one block of 40)
        auto column = [&](auto care_c) {
            constexpr bool CARE = decltype(care_c)::value;
            u32x2 packed[Tile::MI];
#pragma unroll
            for (int i = 0; i < Tile::MI; ++i) {
                const int mrow = Tile::row_off(wave, i) + 4 * quad;
                float e[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    e[r] = fast_exp2(fmaf(G.acc[i][j][r], kLog2e, q.c));
                    if (CARE && mine && mrow + r == q.dy) e[r] += q.g_mag;
                    if (CARE && v0 + mrow + r >= vend) e[r] = 0.0f;
                }
                packed[i] = u32x2{(pack_bf16x2(e[0], e[1]) ^ q.flip) & keep, (pack_bf16x2(e[2], e[3]) ^ q.flip) & keep};
            }
#pragma unroll
            for (int i = 0; i < Tile::MI; i += 2)
                store_bf16_pair(dst + (int64_t)n * a.ld, Tile::row_off(wave, i), m_end, n < n_end, packed[i], packed[i + 1]);
        };
        if (ragged || __any(mine)) column(std::true_type{});
        else column(std::false_type{});
    }
    if (t0 + cols.width >= Ntok) {                // the last tile: zeros up to the next multiple of 64 rows
        constexpr int VPR = Tile::BM / 8;
        for (int q = threadIdx.x + n_end * VPR; q < ((Ntok + 63) / 64 * 64 - t0) * VPR; q += Tile::NT)
            if (q % VPR * 8 < m_end) *reinterpret_cast<u32x4*>(dst + (int64_t)(q / VPR) * a.ld + q % VPR * 8) = u32x4{0u, 0u, 0u, 0u};
    }
}

// One launch of the backward pass over the vocabulary chunks: the two products of the PREVIOUS
// chunk (d_W and dHidden, from that chunk's dz) and the dz tiles of the NEXT chunk (into the other
// buffer) share the grid, longest tiles first.  Tile counts of the separate products rarely fill the
// 256 compute units a whole number of times; as parts of one launch the short dz tiles fill what the
// products leave idle.  dHidden has only rows/256 x Hd/256 tiles, each over the whole chunk: where that
// is too few, its contraction is cut into dh_splits parts that accumulate into slabs of their own (the
// finish kernel adds them in order).  Each part starts at a multiple of 8 workgroups, so a workgroup's
// XCD is its part-local id modulo 8.  n_live (device, may be NULL): the number of live rows, when rows
// were gathered.
struct BwdStepArgs {
    // d_W columns of the previous chunk: dW[k, vp + v] = sum_t dZ[t, v] H[t, k]
    Operand dw_z, dw_h;              // K_COLS both
    bf16_t* d_W;                     // d_W + vp
    int64_t ld_w;
    // dHidden accumulator: acc[t, k] (+)= sum_v W[k, vp + v] dZ[t, v]
    Operand dh_w, dh_z;              // K_ROWS both; dh_z.count is replaced by the live count
    const bf16_t* dh_tail;           // W's columns from vp + dh_K to V, padded to [Hd][64] with zeros (may be NULL)
    int dh_K, dh_accumulate, dh_splits;
    float* dh_acc;                   // [dh_splits, + 1 with a tail][N][Hd]
    int dh_first;                    // dHidden's tiles are the longer ones
    DzArgs dz;
    int have_products, have_dz;
    int N;                           // token rows (upper bound of the live count)
    int group_m;
    const int* n_live;
};

template <template <int, int> class TileT>
ULORL_TILE_KERNEL((TileT<K_ROWS, K_ROWS>::NT), (TileT<K_ROWS, K_ROWS>::WAVES_PER_SIMD))
void lmhead_bwd_step_kernel(const BwdStepArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    using TileDw = TileT<K_COLS, K_COLS>;
    using TileDh = TileT<K_ROWS, K_ROWS>;
    using TileDz = TileT<K_COLS, K_ROWS>;
    constexpr int B = TileDw::BM;
    int rows = a.N;
    if (a.n_live != nullptr) rows = min(rows, *a.n_live);
    int bid = (int)blockIdx.x;
    int tm, tn;
    if (a.have_products) {
        const int nk = (a.dw_h.count + B - 1) / B, nv = (a.dw_z.count + B - 1) / B;
        const int nt = (rows + B - 1) / B, nh = (a.dh_w.count + B - 1) / B;
        const int g_dw = (int)tile_grid(nk, nv);
        const int g_dh1 = rows > 0 ? (int)tile_grid(nt, nh) : 0;
        const int g_dh = g_dh1 * (a.dh_splits + (a.dh_tail != nullptr ? 1 : 0));
        if (bid < g_dw + g_dh) {
            const int dh_bid = a.dh_first ? bid : bid - g_dw;
            if (dh_bid >= 0 && dh_bid < g_dh) {
                if (!tile_coords(dh_bid % g_dh1, nt, nh, a.group_m, tn, tm)) return;
                const int split = dh_bid / g_dh1;
                const bool tail = split == a.dh_splits;           // W's last columns, once, into a slab of their own
                const int per = (a.dh_K / kTileK + a.dh_splits - 1) / a.dh_splits * kTileK;
                const int k0 = tail ? a.dh_K : split * per, K = tail ? kTileK : min(per, a.dh_K - k0);
                const bool add = a.dh_accumulate && !tail;
                if (K <= 0 && add) return;
                TileDh T;
                T.init(lds_raw);
                Operand w = a.dh_w, z = a.dh_z;
                w.p = tail ? a.dh_tail : w.p + k0;
                w.ld = tail ? kTileK : w.ld;
                z.p += k0;
                z.count = rows;
                const ColumnTile c = TileDh::columns(rows, tn);
                if (K > 0) T.run(w, tm * B, z, c, K);
                else T.clear();
                float* acc = a.dh_acc + (int64_t)split * a.N * a.dh_w.count;
                if (add) store_tile_f32<true>(T, acc, a.dh_w.count, a.dh_w.count, rows, tm * B, c.first, true);
                else store_tile_f32<false>(T, acc, a.dh_w.count, a.dh_w.count, rows, tm * B, c.first, true);
                return;
            }
            if (!tile_coords(a.dh_first ? bid - g_dh : bid, nk, nv, a.group_m, tn, tm)) return;
            TileDw T;
            T.init(lds_raw);
            if (rows > 0) T.run(a.dw_z, tm * B, a.dw_h, TileDw::columns(a.dw_h.count, tn), (rows + 63) / 64 * 64);
            else T.clear();                       // no live row: the product is zero
            const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
            const int n_end = a.dw_h.count - tn * B, m_end = a.dw_z.count - tm * B;
#pragma unroll
            for (int j = 0; j < TileDw::NJ; ++j) {
                if (j >= T.blocks()) continue;
                const int n = T.col_off(wave, j) + (lane & 15);
                bf16_t* column = a.d_W + (int64_t)(tn * B + n) * a.ld_w + tm * B;
                auto packed = [&](int i) {
                    return u32x2{pack_bf16x2(T.acc[i][j][0], T.acc[i][j][1]), pack_bf16x2(T.acc[i][j][2], T.acc[i][j][3])};
                };
#pragma unroll
                for (int i = 0; i < TileDw::MI; i += 2)
                    store_bf16_pair(column, TileDw::row_off(wave, i), m_end, n < n_end, packed(i), packed(i + 1));
            }
            return;
        }
        bid -= g_dw + g_dh;
    }
    if (a.have_dz && rows > 0) lmhead_dz_block<TileDz>(bid, a.dz, rows, a.group_m, lds_raw);
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
static_assert(tile_edge(0) == TileLarge<K_ROWS, K_ROWS>::BM && tile_edge(1) == TileSmall<K_ROWS, K_ROWS>::BM, "the plan's tiles");

LmheadLayout layout_of(int64_t N, int64_t Hd, int64_t V, int32_t R, int32_t vocab_chunk, int tile)
{
    return lmhead_layout(N, Hd, V, vocab_chunk, tile, workspace_layout(N, 0, R).total);
}

int32_t check_lmhead(const void* hidden, const void* W, int64_t N, int64_t Hd, int64_t V, int32_t chunk)
{
    if (!hidden || !W) return ULORL_ERR_NULL;
    // N, the chunk width and V become leading dimensions of GEMM operands (see kMaxLeadingDim)
    if (N <= 0 || N > kMaxLeadingDim - 256 || V <= 0 || V > kMaxColsLeadingDim || Hd <= 0 || Hd > (1 << 20)) return ULORL_ERR_SHAPE;
    if (Hd % 8 != 0 || V % 8 != 0) return ULORL_ERR_SHAPE;     // 16-byte rows of hidden and W
    if (chunk <= 0 || chunk % 64 != 0 || chunk > kMaxLeadingDim - 256) return ULORL_ERR_SHAPE;
    if (((uintptr_t)hidden & 15u) != 0 || ((uintptr_t)W & 15u) != 0) return ULORL_ERR_ALIGN;
    return ULORL_OK;
}

// Raises the kernel's dynamic-LDS limit once per kernel and process (the runtime call is not a
// stream operation; keeping it out of later launches also keeps it out of stream captures that
// follow a warm-up call).
bool allow_lds_for(const void* kernel, size_t bytes)
{
    static std::mutex mu;
    static std::unordered_map<const void*, size_t> allowed;
    std::lock_guard<std::mutex> lock(mu);
    auto it = allowed.find(kernel);
    if (it != allowed.end() && it->second >= bytes) return true;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess) return false;
    allowed[kernel] = bytes;
    return true;
}

template <class Kernel>
bool allow_lds(Kernel k, size_t bytes)
{
    return allow_lds_for(reinterpret_cast<const void*>(k), bytes);
}

void launch_copy_rows_padded(const bf16_t* src, int64_t ld_src, int64_t rows, int64_t cols, bf16_t* dst, int64_t dst_cols,
                             hipStream_t st, const int* row_map = nullptr, const int* n_rows = nullptr)
{
    const int64_t nvec = round_up64(rows) * (dst_cols / 8);
    hipLaunchKernelGGL(copy_rows_padded_kernel, dim3((unsigned)((nvec + 255) / 256)), dim3(256), 0, st, src, ld_src, (int)cols,
                       row_map, n_rows, rows, dst, dst_cols);
}

template <class Tile>
bool launch_gemm(const GemmArgs& g, int group_m, hipStream_t st)
{
    auto kern = gemm_tn_kernel<Tile>;
    if (!allow_lds(kern, Tile::LDS_BYTES)) return false;
    dim3 grid(tile_grid((g.a.count + Tile::BN - 1) / Tile::BN, (g.b.count + Tile::BM - 1) / Tile::BM));
    hipLaunchKernelGGL(kern, grid, dim3(Tile::NT), Tile::LDS_BYTES, st, g, group_m);
    return true;
}

template <template <int, int> class TileT>
bool launch_stats(const Operand& W, const Operand& H, int K, const int32_t* token_ids, const LmheadLayout& L, StatQuad* partial,
                  int group_m, hipStream_t st)
{
    using Tile = TileT<K_COLS, K_ROWS>;
    auto kern = lmhead_stats_kernel<Tile>;
    if (!allow_lds(kern, Tile::LDS_BYTES)) return false;
    dim3 grid(tile_grid((H.count + Tile::BN - 1) / Tile::BN, L.splits));
    hipLaunchKernelGGL(kern, grid, dim3(Tile::NT), Tile::LDS_BYTES, st, W, H, K, token_ids, L.v_per_split, L.splits, partial, group_m);
    return true;
}

template <template <int, int> class TileT>
bool launch_bwd_step(const BwdStepArgs& a, hipStream_t st)
{
    using Tile = TileT<K_COLS, K_COLS>;
    auto kern = lmhead_bwd_step_kernel<TileT>;
    constexpr size_t lds = Tile::LDS_BYTES + Tile::BN * sizeof(DzTerm);
    if (!allow_lds(kern, lds)) return false;
    // the largest grid the live count allows; workgroups beyond the actual tiles return at once
    constexpr int B = Tile::BM;
    unsigned grid = 0;
    if (a.have_products) {
        grid += tile_grid((a.dw_h.count + B - 1) / B, (a.dw_z.count + B - 1) / B);
        grid += tile_grid((a.N + B - 1) / B, (a.dh_w.count + B - 1) / B) * (unsigned)(a.dh_splits + (a.dh_tail != nullptr ? 1 : 0));
    }
    if (a.have_dz) grid += tile_grid((a.dz.cw + B - 1) / B, (a.N + B - 1) / B);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(Tile::NT), lds, st, a);
    return true;
}

// W as the products read it: itself, or a copy padded with zeros to multiples of 64 (pad).
Operand weight_operand(const bf16_t* W, int64_t Hd, int64_t V, const LmheadLayout& L, char* ws, bool pad, hipStream_t st)
{
    if (!pad) return Operand{W, V, (int)V};
    bf16_t* wp = (bf16_t*)(ws + L.wp);
    launch_copy_rows_padded(W, V, Hd, V, wp, L.v64, st);
    return Operand{wp, L.v64, (int)V};
}

}  // namespace

extern "C" {

int32_t ulorl_gemm_tn_bf16(const void* A, int64_t lda, const void* B, int64_t ldb, int64_t M, int64_t N, int64_t K,
                           float* C, int64_t ldc, const ulorl_launch* launch, void* hip_stream)
{
    if (!A || !B || !C) return ULORL_ERR_NULL;
    LaunchOpts opts;
    const int32_t lrc = resolve_launch(launch, &opts);
    if (lrc != ULORL_OK) return lrc;
    if (M <= 0 || N <= 0 || K <= 0 || M > 0x7fffffffLL || N > 0x7fffffffLL || K > 0x7fffffffLL) return ULORL_ERR_SHAPE;
    if (K % 8 != 0 || lda % 8 != 0 || ldb % 8 != 0 || lda < K || ldb < K || ldc < N) return ULORL_ERR_SHAPE;
    if (lda > kMaxLeadingDim || ldb > kMaxLeadingDim) return ULORL_ERR_SHAPE;
    if (((uintptr_t)A & 15u) != 0 || ((uintptr_t)B & 15u) != 0) return ULORL_ERR_ALIGN;
    GemmArgs g;
    g.a = Operand{(const bf16_t*)A, lda, (int)M};
    g.b = Operand{(const bf16_t*)B, ldb, (int)N};
    g.K = (int)K;
    g.C = C;
    g.ldc = ldc;
    g.wide = (((uintptr_t)C & 15u) == 0 && ldc % 4 == 0) ? 1 : 0;
    hipStream_t st = (hipStream_t)hip_stream;
    const bool ok = K % kTileK != 0      ? launch_gemm<TileRagged>(g, opts.gemm_group_m, st)
                    : opts.gemm_tile == 1 ? launch_gemm<TileSmall<K_ROWS, K_ROWS>>(g, opts.gemm_group_m, st)
                                          : launch_gemm<TileLarge<K_ROWS, K_ROWS>>(g, opts.gemm_group_m, st);
    if (!ok) return ULORL_ERR_HIP;
    return hipGetLastError() == hipSuccess ? ULORL_OK : ULORL_ERR_HIP;
}

size_t ulorl_lmhead_workspace_bytes(int64_t N, int64_t Hd, int64_t V, int32_t R, int32_t vocab_chunk)
{
    if (N <= 0 || N > 0x7fffffffLL || Hd <= 0 || V <= 0 || V > kMaxColsLeadingDim || R <= 0 || vocab_chunk <= 0 || vocab_chunk % 64 != 0) return 0;
    return layout_of(N, Hd, V, R, vocab_chunk, 0).total;      // the same for every tile shape
}

int32_t ulorl_lmhead_token_loss_fwd(const void* hidden, const void* W, int64_t N, int64_t Hd, int64_t V,
                                    int32_t vocab_chunk, const int32_t* token_ids, const int32_t* cu_seqlens,
                                    int32_t R, const int32_t* segment_ids, const float* old_logp,
                                    const float* advantages, const ulorl_params* p, float* loss, float* logp,
                                    float* entropy, float* lse, float* gcoef, uint8_t* mpt_mask, float* ratio,
                                    int32_t* segment_out, float* resp_entropy, uint8_t* resp_gate, int64_t* counters,
                                    const ulorl_segment_stats* seg_stats, void* workspace, size_t workspace_bytes,
                                    const ulorl_launch* launch, void* hip_stream)
{
    int32_t rc = check_lmhead(hidden, W, N, Hd, V, vocab_chunk);
    if (rc != ULORL_OK) return rc;
    if (!token_ids || !logp || !entropy || !lse) return ULORL_ERR_NULL;
    LaunchOpts opts;
    rc = resolve_launch(launch, &opts);
    if (rc != ULORL_OK) return rc;
    const bool stats_only = advantages == nullptr;      // lse, logp and entropy only (recording old log-probs)
    SegStatsArgs seg;
    seg.K = 0;
    if (!stats_only) {
        rc = check_objective_args(cu_seqlens, R, old_logp, p, loss, gcoef);
        if (rc != ULORL_OK) return rc;
        rc = resolve_segment_stats(seg_stats, N, &seg);
        if (rc != ULORL_OK) return rc;
    } else if (R <= 0) {
        R = 1;      // only sizes the workspace layout
    }
    const int tile = forward_tile(opts.gemm_tile, N, Hd, V);
    const LmheadLayout L = layout_of(N, Hd, V, R, vocab_chunk, tile);
    if (!workspace || ((uintptr_t)workspace & 255u) != 0 || workspace_bytes < L.total) return ULORL_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)hip_stream;
    char* ws = (char*)workspace;
    StatQuad* partial = (StatQuad*)(ws + L.partial);

    const Operand Wop = weight_operand((const bf16_t*)W, Hd, V, L, ws, L.pad_k, st);
    Operand Hop = {(const bf16_t*)hidden, Hd, (int)N};
    if (L.pad_k) {
        bf16_t* hp = (bf16_t*)(ws + L.hp);
        launch_copy_rows_padded((const bf16_t*)hidden, Hd, N, Hd, hp, L.hd64, st);
        Hop = Operand{hp, L.hd64, (int)N};
    }
    const bool ok = tile == 1
                        ? launch_stats<TileSmall>(Wop, Hop, (int)L.hd64, token_ids, L, partial, opts.gemm_group_m, st)
                        : launch_stats<TileLarge>(Wop, Hop, (int)L.hd64, token_ids, L, partial, opts.gemm_group_m, st);
    if (!ok) return ULORL_ERR_HIP;
    const int lanes = L.splits > 64 ? 32 : 8;
    hipLaunchKernelGGL(lanes == 32 ? lmhead_stats_merge_kernel<32> : lmhead_stats_merge_kernel<8>, dim3((unsigned)((N * lanes + 255) / 256)),
                       dim3(256), 0, st, partial, L.splits, (int)N, (int)V, token_ids, lse, logp, entropy);
    if (hipGetLastError() != hipSuccess) return ULORL_ERR_HIP;
    if (stats_only) return ULORL_OK;

    const WorkspaceLayout wl = workspace_layout(N, 0, R);
    const TokenArgs a = make_token_args(N, V, token_ids, cu_seqlens, R, segment_ids, old_logp, advantages, p, logp,
                                        entropy, lse, gcoef, mpt_mask, ratio, segment_out, resp_entropy, resp_gate,
                                        loss, counters, ws + L.token_ws, wl, seg);
    launch_token_epilogue(a, wl, st);
    return hipGetLastError() == hipSuccess ? ULORL_OK : ULORL_ERR_HIP;
}

int32_t ulorl_lmhead_token_loss_bwd(const void* hidden, const void* W, int64_t N, int64_t Hd, int64_t V,
                                    int32_t vocab_chunk, const int32_t* token_ids, const float* lse,
                                    const float* gcoef, float grad_out, void* d_hidden, void* d_W, void* workspace,
                                    size_t workspace_bytes, const ulorl_launch* launch, void* hip_stream)
{
    int32_t rc = check_lmhead(hidden, W, N, Hd, V, vocab_chunk);
    if (rc != ULORL_OK) return rc;
    LaunchOpts opts;
    rc = resolve_launch(launch, &opts);
    if (rc != ULORL_OK) return rc;
    if (!token_ids || !lse || !gcoef || !d_hidden || !d_W) return ULORL_ERR_NULL;
    if (((uintptr_t)d_hidden & 15u) != 0 || ((uintptr_t)d_W & 15u) != 0) return ULORL_ERR_ALIGN;
    const int tile = backward_tile(opts.gemm_tile, N, Hd, V);
    const LmheadLayout L = layout_of(N, Hd, V, 1, vocab_chunk, tile);
    if (!k_rows_fit(tile_edge(tile), L.v64, L.chunk)) return ULORL_ERR_SHAPE;     // W as an operand of the dHidden product
    if (!workspace || ((uintptr_t)workspace & 255u) != 0 || workspace_bytes < L.total) return ULORL_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)hip_stream;
    char* ws = (char*)workspace;
    float* dHacc = (float*)(ws + L.dhacc);
    bf16_t* hc = (bf16_t*)(ws + L.rows);
    const bf16_t* H = (const bf16_t*)hidden;
    const Operand Wop = weight_operand((const bf16_t*)W, Hd, V, L, ws, L.pad_k || L.pad_v, st);
    const int64_t v_whole = L.tail_v ? V / kTileK * kTileK : L.v64;      // columns that whole K tiles of the dHidden product cover
    bf16_t* w_tail = nullptr;
    if (L.tail_v) {
        w_tail = (bf16_t*)(ws + L.tail);
        launch_copy_rows_padded((const bf16_t*)W + v_whole, V, Hd, V - v_whole, w_tail, kTileK, st);
    }

    // Live rows (those with a non-zero coefficient): positions in order and gathered hidden rows.
    // ULORL_LAUNCH_DENSE_ROWS runs every row through the products instead.
    Operand Hop = {hc, L.hd64, (int)N};
    const int* row_map = nullptr;
    const int* pos = nullptr;
    const int* n_live = nullptr;
    if (!opts.dense_rows) {
        int* posw = (int*)(ws + L.pos);
        int* mapw = (int*)(ws + L.row_map);
        int* cntw = (int*)(ws + L.block_count);
        int* nlw = (int*)(ws + L.n_live);
        const int nblk = (int)((N + kLiveBlock - 1) / kLiveBlock);
        if (N <= kLiveRecountRows) {
            hipLaunchKernelGGL(live_rows_kernel, dim3((unsigned)nblk), dim3(kLiveBlock), 0, st, gcoef, lse, token_ids, grad_out, N,
                               (int32_t)V, posw, mapw, nlw);
        } else {
            hipLaunchKernelGGL(live_count_kernel, dim3((unsigned)nblk), dim3(kLiveBlock), 0, st, gcoef, lse, token_ids, grad_out,
                               N, (int32_t)V, cntw);
            hipLaunchKernelGGL(live_scan_kernel, dim3(1), dim3(kLiveBlock), 0, st, cntw, nblk, nlw);
            hipLaunchKernelGGL(live_fill_kernel, dim3((unsigned)nblk), dim3(kLiveBlock), 0, st, gcoef, lse, token_ids, grad_out, N,
                               (int32_t)V, (const int*)cntw, posw, mapw);
        }
        launch_copy_rows_padded(H, Hd, N, Hd, hc, L.hd64, st, mapw, nlw);
        row_map = mapw; pos = posw; n_live = nlw;
    } else if (L.pad_k || N % 64 != 0) {
        launch_copy_rows_padded(H, Hd, N, Hd, hc, L.hd64, st);
    } else {
        Hop.p = H;
    }
    if (hipGetLastError() != hipSuccess) return ULORL_ERR_HIP;

    // Chunk pipeline: launch c holds the dz tiles of chunk c and the two products of chunk c - 1.
    const int64_t n_chunks = (V + L.chunk - 1) / L.chunk;
    auto width = [&](int64_t c) { return (int)(V - c * L.chunk < L.chunk ? V - c * L.chunk : L.chunk); };
    for (int64_t c = 0; c <= n_chunks; ++c) {
        BwdStepArgs a;
        memset(&a, 0, sizeof(a));
        a.N = (int)N;
        a.group_m = opts.gemm_group_m;
        a.n_live = n_live;
        a.dh_splits = 1;
        if (c >= 1) {
            const int64_t vp = (c - 1) * L.chunk;
            const int cwp = width(c - 1);
            const bf16_t* dZ = (const bf16_t*)(ws + L.dz[(c - 1) & 1]);
            a.have_products = 1;
            a.dw_z = Operand{dZ, L.chunk, cwp};
            a.dw_h = Operand{Hop.p, L.hd64, (int)Hd};
            a.d_W = (bf16_t*)d_W + vp;
            a.ld_w = V;
            a.dh_w = Operand{Wop.p + vp, Wop.ld, (int)Hd};
            a.dh_z = Operand{dZ, L.chunk, (int)N};
            a.dh_K = (int)(vp + L.chunk < v_whole ? L.chunk : v_whole - vp);
            a.dh_tail = c == n_chunks ? w_tail : nullptr;
            a.dh_accumulate = c > 1;
            a.dh_splits = L.dh_splits;
            a.dh_acc = dHacc;
            a.dh_first = a.dh_K / L.dh_splits > N;      // contraction lengths of the two products' tiles
        }
        if (c < n_chunks) {
            a.have_dz = 1;
            a.dz.W = Wop; a.dz.H = Hop; a.dz.K = (int)L.hd64; a.dz.vc0 = (int)(c * L.chunk);
            a.dz.cw = (int)round_up64(width(c));         // dz of the padding columns is written as zero
            a.dz.token_ids = token_ids; a.dz.lse = lse; a.dz.gcoef = gcoef; a.dz.grad_out = grad_out;
            a.dz.dZ = (bf16_t*)(ws + L.dz[c & 1]); a.dz.ld = L.chunk;
            a.dz.row_map = row_map;
        }
        const bool ok = tile == 1 ? launch_bwd_step<TileSmall>(a, st) : launch_bwd_step<TileLarge>(a, st);
        if (!ok || hipGetLastError() != hipSuccess) return ULORL_ERR_HIP;
    }
    const int64_t nh = N * Hd;
    hipLaunchKernelGGL(dhidden_finish_kernel, dim3((unsigned)((nh / 8 + 255) / 256)), dim3(256), 0, st, (const float*)dHacc, L.dh_slabs, pos,
                       N, (int)Hd, (bf16_t*)d_hidden);
    return hipGetLastError() == hipSuccess ? ULORL_OK : ULORL_ERR_HIP;
}

}  // extern "C"
