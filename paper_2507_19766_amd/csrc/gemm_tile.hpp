// Block tiles of a bf16 MFMA product for gfx950, used by every product of the lm_head variant:
//     acc[m, n] = sum_k A[m, k] * B[n, k]        (fp32 accumulation, v_mfma_f32_16x16x32_bf16)
//
// An operand may lie in memory either way:
//   K_ROWS   one row per m (or n), k contiguous:   element (m, k) at base[m * ld + k]
//   K_COLS   one row per k, m (or n) contiguous:   element (m, k) at base[k * ld + m]
// so that no operand has to be transposed through memory first: a K_COLS fragment is transposed on
// its way from LDS to registers (ds_read_b64_tr_b16).
//
// Result layout: block (i, j) of a wave is a 16 x 16 piece of the tile; in it lane L holds column
// n = L % 16 and the four consecutive rows m = 4 (L / 16) + r.  Results are therefore written with m
// contiguous, and a reduction over m is mostly lane-local.
#ifndef ULORL_GEMM_TILE_HPP
#define ULORL_GEMM_TILE_HPP

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm_limits.hpp"
#include "gemm_loop.hpp"

namespace ulorl_detail {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x32 __attribute__((ext_vector_type(32)));
typedef uint16_t bf16_t;  // raw storage

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    f32x2 x = {lo, hi};
    bf16x2 b = __builtin_convertvector(x, bf16x2);  // round to nearest even
    return __builtin_bit_cast(uint32_t, b);
}

enum { K_ROWS = 0, K_COLS = 1 };

// One operand of a product: `count` rows (columns) of the result, its memory layout is the kernel's
// template argument.
struct Operand {
    const bf16_t* p;
    int64_t ld;
    int count;
};

constexpr int kHalf = 128;                       // rows (columns) of one half tile: the unit of copying
constexpr int kHalfElems = kHalf * kTileK;       // 16 KB
// Word 3 of a raw (unstructured, stride 0) buffer descriptor on gfx9-family parts: 32-bit data format.
constexpr int kRawBufferFlags = 0x00020000;
// s_waitcnt immediates: at most n vector memory operations (LDS operations) still outstanding.
#define ULORL_WAIT_VMEM(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (7 << 4) | (15 << 8) | (((n) >> 4) << 14))
#define ULORL_WAIT_LDS(n) __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | ((n) << 8) | (3 << 14))

// A workgroup barrier without the waits of __syncthreads (copies to LDS stay in flight across it);
// nothing is moved over it by the compiler.
__device__ __forceinline__ void bare_barrier()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// One operand of a block tile: the global -> LDS copies of its half tiles and the reads of MFMA
// fragments.  NW waves copy; a wave's fragments are 16-row blocks that start at row `wave_row` of a
// half.
//
// LDS images of a half tile (16 KB), both written by buffer_load_dwordx4 ... lds, which deposits lane
// L's 16 bytes at base + 16 L, so the images are unpadded and bank conflicts are avoided by
// permuting the 16-byte vectors of a row (each lane fetches the vector that belongs in its slot):
//   K_ROWS   128 rows of 64 k (128 B); vector v of row r in slot v ^ ((r / 2) mod 8).  A ds_read_b128 is
//            served 16 rows at a time, which then fall in 16 different 16-byte columns.
//   K_COLS   64 rows (k) of 128 m (256 B); vector v of row k in slot v ^ (4 (k mod 4) + 2 ((k / 8) mod 2)).
//            A ds_read_b64_tr_b16 takes 32 bytes of rows k .. k+3 for each 16 lanes; 32 lanes then cover
//            the 256-byte bank line once.
//
// With HALVES == 2 (the large tile) the copies and reads themselves stand in gemm_loop.hpp; what issues them here serves one half.
template <int LAYOUT, int NW, int HALVES>
struct TileOperand {
    static constexpr int BLOCKS = 4;             // 16-row fragments of a wave
    static constexpr int J = 16 / NW;            // copy instructions per wave and half tile
    static constexpr int NV = HALVES == 2 && LAYOUT == K_ROWS ? 1 : LAYOUT == K_ROWS ? J : HALVES;
    static constexpr int NR = LAYOUT == K_ROWS ? 2 : BLOCKS;
    const char* src;          // this wave's rows of the K tile at the copy cursor (uniform)
    int64_t step;             // bytes from one K tile to the next
    int64_t row_step;         // K_COLS, and K_ROWS of the large tile: bytes from copy instruction j to j + 1
    int soff;                 // K_ROWS: byte offset of the copy cursor along k
    uint32_t extent;
    uint32_t voff[NV];        // this lane's byte offset
    int roff[NR];             // this lane's LDS read offset, in bytes inside a half
    bf16_t* lds;              // [stage][half]
    int64_t ld;
    int count;                // rows (columns) of this tile
    int wave;

    // first: first row (column) of the tile, `most` of them at most; the copy cursor is at k = 0.  K_ROWS rows past the last
    // lie outside the buffer and arrive as zeros, without memory traffic; K_COLS columns past it repeat earlier ones (their
    // results are ignored).
    __device__ __forceinline__ void set_tile(const Operand& op, int first, int64_t K, int wave_, int most = HALVES * kHalf)
    {
        wave = wave_;
        ld = op.ld;
        count = min(most, op.count - first);
        if constexpr (LAYOUT == K_ROWS) {
            src = reinterpret_cast<const char*>(op.p + (int64_t)first * ld);
            soff = 0;
            row_step = (int64_t)NW * 8 * ld * 2;
            const uint64_t ext = ((uint64_t)(count - 1) * (uint64_t)ld + (uint64_t)K) * 2;
            extent = (uint32_t)min(ext, (uint64_t)0xffffffffu);
        } else {
            src = reinterpret_cast<const char*>(op.p + (int64_t)(wave * 4) * ld + first);
            step = (int64_t)kTileK * ld * 2;
            row_step = (int64_t)NW * 4 * ld * 2;
            // rows of k reached from src: 4 (each copy instruction has its own base) or, with the large tile's offsets, 48 more
            const uint64_t ext = ((uint64_t)(HALVES == 2 ? 51 : 3) * (uint64_t)ld + (uint64_t)count) * 2;
            extent = (uint32_t)min(ext, (uint64_t)0xffffffffu);
        }
    }
    __device__ __forceinline__ void set_copies(int lane)
    {
        if constexpr (LAYOUT == K_ROWS) {
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                const int row = (j * NW + wave) * 8 + lane / 8;
                const int vec = (lane % 8) ^ ((row >> 1) & 7);
                voff[j] = (uint32_t)(((int64_t)row * ld + vec * 8) * 2);
            }
        } else {
            const int k = wave * 4 + lane / 16;
            const int vec = (lane % 16) ^ (((k & 3) << 2) | (((k >> 3) & 1) << 1));
#pragma unroll
            for (int h = 0; h < HALVES; ++h) {
                const int col = min(h * kHalf + vec * 8, count - 8);     // counts are multiples of 8
                voff[h] = (uint32_t)(((int64_t)(lane / 16) * ld + col) * 2);
            }
        }
    }
    __device__ __forceinline__ void set_reads(bf16_t* lds_, int wave_row, int lane)
    {
        lds = lds_;
        if constexpr (LAYOUT == K_ROWS) {
            const int row = wave_row + (lane & 15);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) roff[ks] = row * 128 + (((ks * 4 + (lane >> 4)) ^ ((row >> 1) & 7)) * 16);
        } else {
            const int k = 8 * (lane >> 4) + ((lane & 15) >> 2);
            const int swz = ((k & 3) << 2) | (((k >> 3) & 1) << 1);
#pragma unroll
            for (int b = 0; b < BLOCKS; ++b) {
                const int slot = ((wave_row / 8 + b * 2) ^ swz) + ((lane & 3) >> 1);
                roff[b] = k * 256 + slot * 16 + (lane & 1) * 8;
            }
        }
    }

    // This wave's share of the K tile at the cursor, into stage s; one of its J instructions.
    __device__ __forceinline__ void copy_part(int j, int s) const
    {
        static_assert(HALVES == 1, "the large tile's copies are in gemm_loop.hpp");
        bf16_t* dst = lds + s * kHalfElems;
        if constexpr (LAYOUT == K_ROWS) {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(src), 0, (int)extent, kRawBufferFlags);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(dst + (j * NW + wave) * 512), 16,
                                                     voff[j], soff, 0, 0);
        } else {
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(src + j * row_step), 0, (int)extent, kRawBufferFlags);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(dst + (j * NW + wave) * 512), 16,
                                                     voff[0], 0, 0, 0);
        }
    }
    __device__ __forceinline__ void copy(int s) const
    {
#pragma unroll
        for (int j = 0; j < J; ++j) copy_part(j, s);
    }
    __device__ __forceinline__ void advance()
    {
        if constexpr (LAYOUT == K_ROWS) soff += kTileK * 2;
        else src += step;
    }

    // The fragments of stage s: f[ks][b], lane L: row 16 b + L % 16, k = 32 ks + 8 (L / 16) ..+7.
    // K_COLS fragments have arrived on return; K_ROWS ones are waited for by the caller (or their use).
    // The compiler's builtin for the transposing read is taken for a possible LDS write and gets a wait
    // for ALL copies in flight put before it; here the reads are issued and waited for in one block.
    __device__ __forceinline__ void read(int s, bf16x8 (&f)[2][BLOCKS]) const
    {
        static_assert(HALVES == 1, "the large tile's reads are in gemm_loop.hpp");
        bf16_t* half = lds + s * kHalfElems;
        if constexpr (LAYOUT == K_ROWS) {
            const char* base = reinterpret_cast<const char*>(half);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int b = 0; b < BLOCKS; ++b)
                    f[ks][b] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(base + roff[ks] + b * 16 * 128));
        } else {
            const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) bf16_t*)half;
            u32x2 r[4 * BLOCKS];          // [ks][block][low / high four k]
            asm volatile(
                "ds_read_b64_tr_b16 %0, %16\n\t"
                "ds_read_b64_tr_b16 %1, %16 offset:1024\n\t"
                "ds_read_b64_tr_b16 %2, %17\n\t"
                "ds_read_b64_tr_b16 %3, %17 offset:1024\n\t"
                "ds_read_b64_tr_b16 %4, %18\n\t"
                "ds_read_b64_tr_b16 %5, %18 offset:1024\n\t"
                "ds_read_b64_tr_b16 %6, %19\n\t"
                "ds_read_b64_tr_b16 %7, %19 offset:1024\n\t"
                "ds_read_b64_tr_b16 %8, %16 offset:8192\n\t"
                "ds_read_b64_tr_b16 %9, %16 offset:9216\n\t"
                "ds_read_b64_tr_b16 %10, %17 offset:8192\n\t"
                "ds_read_b64_tr_b16 %11, %17 offset:9216\n\t"
                "ds_read_b64_tr_b16 %12, %18 offset:8192\n\t"
                "ds_read_b64_tr_b16 %13, %18 offset:9216\n\t"
                "ds_read_b64_tr_b16 %14, %19 offset:8192\n\t"
                "ds_read_b64_tr_b16 %15, %19 offset:9216\n\t"
                "s_waitcnt lgkmcnt(0)"
                : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7]),
                "=&v"(r[8]), "=&v"(r[9]), "=&v"(r[10]), "=&v"(r[11]), "=&v"(r[12]), "=&v"(r[13]), "=&v"(r[14]), "=&v"(r[15])
                : "v"(base + roff[0]), "v"(base + roff[1]), "v"(base + roff[2]), "v"(base + roff[3])
                : "memory");
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int b = 0; b < BLOCKS; ++b) f[ks][b] = join(r[(ks * BLOCKS + b) * 2], r[(ks * BLOCKS + b) * 2 + 1]);
        }
    }

    static __device__ __forceinline__ bf16x8 join(u32x2 lo, u32x2 hi)
    {
        return __builtin_bit_cast(bf16x8, u32x4{lo[0], lo[1], hi[0], hi[1]});
    }
};

// Columns [first, first + width) of the result.
struct ColumnTile {
    int first, width;
};

// ---------------------------------------------------------------------------------------------
// 256 x 256 tile, four waves (gemm_loop.hpp)
// ---------------------------------------------------------------------------------------------
// Wave (wm, wn) owns the 64-row pieces at rows 128 h + 64 wm, h = 0, 1, and the columns 64 wn ..+63 of half 0 and
// 16 j1 wn ..+16 j1 - 1 of half 1, where j1 = 1..4 is a quarter of the width of half 1: with B K_ROWS the tile may be 160,
// 192, 224 or 256 columns wide, or up to 128 (half 1 is then run as one of 160 and has empty columns only).  The tiles of a product share its columns evenly, in units of 32 (columns()), so
// that a last tile of a few columns does not cost a whole one: the parts that multiply half 1 leave after j1 of four blocks.
//
// begin() issues the first copies, finish() does the rest: a kernel that walks several tiles begins the next one
// before it works on the results of the last.
template <int LA, int LB>
struct TileLarge {
    static constexpr int BM = 256, BN = 256, NW = 4, NT = 256;
    static constexpr int WAVES_PER_SIMD = 1;
    static constexpr int MI = 8, NJ = 8;                       // 16 x 16 blocks of a wave
    static constexpr int WAVES_M = 2;
    static constexpr size_t LDS_BYTES = 8 * (size_t)kHalfElems * sizeof(bf16_t);

    TileOperand<LA, NW, 2> a;
    TileOperand<LB, NW, 2> b;
    f32x4 acc[MI][NJ];
    uint32_t lds_base;
    uint32_t y_shift;         // K_ROWS B: bytes from a half 0 read address to that of half 1
    int wave, j1, kt;

    static __device__ __forceinline__ int row_off(int wave, int i) { return (i >> 2) * 128 + (wave >> 1) * 64 + (i & 3) * 16; }
    __device__ __forceinline__ int col_off(int wave, int j) const
    {
        return j < 4 ? (wave & 1) * 64 + j * 16 : 128 + (wave & 1) * 16 * j1 + (j - 4) * 16;
    }
    static __device__ __forceinline__ int wave_m(int wave) { return wave >> 1; }
    __device__ __forceinline__ int blocks() const { return 4 + j1; }          // column blocks that hold results

    // Tile t of ceil(count / 256).
    static __device__ __forceinline__ ColumnTile columns(int count, int t)
    {
        if constexpr (LB == K_COLS) return ColumnTile{t * BN, BN};
        const int tiles = (count + BN - 1) / BN, units = (count + 31) / 32;
        const int each = units / tiles, more = units - each * tiles;
        return ColumnTile{32 * (t * each + min(t, more)), 32 * (each + (t < more ? 1 : 0))};
    }

    __device__ __forceinline__ void init(unsigned char* lds)
    {
        wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;
    }
    // A lane's addresses are formed anew for each of the two blocks of assembly: kept over the main loop they are
    // spilled, and their reloads wait for the copies in flight.
    static __device__ __forceinline__ int fresh_lane()
    {
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        return lane;
    }
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        j1 = 4;
    }
    // K a positive multiple of 64, or 0: nothing is copied but zeros, and finish() may not follow.  No wave may still read from LDS.
    __device__ __forceinline__ void begin(const Operand& A, int m0, const Operand& B, ColumnTile c, int K)
    {
        const int lane = fresh_lane();
        a.set_tile(A, m0, K, wave);
        b.set_tile(B, c.first, K, wave, c.width);
        a.set_copies(lane);
        b.set_copies(lane);
        const int width = min(c.width, B.count - c.first);
        j1 = LB == K_COLS ? (width > kHalf ? 4 : 1) : max((width + 31) / 32 - 4, 1);
        y_shift = (uint32_t)((wave & 1) * (16 * j1 - 64) * 128);
        kt = K / kTileK;
        const uint64_t pa = (uint64_t)(uintptr_t)a.src, pb = (uint64_t)(uintptr_t)b.src;
#define UL_POINTERS [pa] "s"(pa), [pb] "s"(pb)
        if constexpr (LA == K_ROWS && LB == K_ROWS)
            asm volatile(UL_BEGIN(ROWS, ROWS) : : UL_IN, UL_POINTERS, UL_IN_COPY_ROWS_A, UL_IN_COPY_ROWS_B : UL_CLOBBERS);
        else if constexpr (LA == K_COLS && LB == K_ROWS)
            asm volatile(UL_BEGIN(COLS, ROWS) : : UL_IN, UL_POINTERS, UL_IN_COPY_COLS_A, UL_IN_COPY_ROWS_B : UL_CLOBBERS);
        else
            asm volatile(UL_BEGIN(COLS, COLS) : : UL_IN, UL_POINTERS, UL_IN_COPY_COLS_A, UL_IN_COPY_COLS_B : UL_CLOBBERS);
    }
    // acc = the product over K.  On return no wave reads from LDS any more.
    __device__ __forceinline__ void finish()
    {
        static_assert(LA == K_COLS || LB == K_ROWS, "not written out");
        const int lane = fresh_lane();
        a.set_copies(lane);
        b.set_copies(lane);
        a.set_reads(nullptr, (wave >> 1) * 64, lane);
        b.set_reads(nullptr, (wave & 1) * 64, lane);
        uint64_t pa, pb;
        cursors(pa, pb);
        f32x32 f0, f1, f2, f3;
#define UL_FRAGMENTS "=&{v[128:159]}"(f0), "=&{v[160:191]}"(f1), "=&{v[192:223]}"(f2), "=&{v[224:255]}"(f3)
#define UL_MAIN_IN UL_IN, UL_POINTERS, [j1] "s"(j1)
        if constexpr (LA == K_ROWS && LB == K_ROWS)
            asm volatile(UL_MAIN(ROWS, ROWS) : UL_BLOCKS(UL_OUT) UL_FRAGMENTS
                         : UL_MAIN_IN, UL_IN_COPY_ROWS_A, UL_IN_COPY_ROWS_B, UL_IN_READ_ROWS_A, UL_IN_READ_ROWS_B : UL_CLOBBERS);
        else if constexpr (LA == K_COLS && LB == K_ROWS)
            asm volatile(UL_MAIN(COLS, ROWS) : UL_BLOCKS(UL_OUT) UL_FRAGMENTS
                         : UL_MAIN_IN, UL_IN_COPY_COLS_A, UL_IN_COPY_ROWS_B, UL_IN_READ_COLS_A, UL_IN_READ_ROWS_B : UL_CLOBBERS);
        else
            asm volatile(UL_MAIN(COLS, COLS) : UL_BLOCKS(UL_OUT) UL_FRAGMENTS
                         : UL_MAIN_IN, UL_IN_COPY_COLS_A, UL_IN_COPY_COLS_B, UL_IN_READ_COLS_A, UL_IN_READ_COLS_B : UL_CLOBBERS);
    }
    // The same with the caller's 32 running values given to the block, which leaves them alone, in registers of their own: the
    // compiler would keep some of them in scratch memory around it, and a reload waits for every copy in flight.  Others of the
    // statistics kernel's values are still there (22 registers spilled, 56 bytes a lane), and some of their reloads stand
    // in the work on a tile's results, behind the next tile's first copies.
    __device__ __forceinline__ void finish_keep(float (&m)[NJ], float (&S)[NJ], float (&C)[NJ], float (&T)[NJ])
    {
        const int lane = fresh_lane();
        a.set_copies(lane);
        b.set_copies(lane);
        a.set_reads(nullptr, (wave >> 1) * 64, lane);
        b.set_reads(nullptr, (wave & 1) * 64, lane);
        uint64_t pa, pb;
        cursors(pa, pb);
        f32x32 f0, f1, f2, f3;
        asm volatile(UL_MAIN(COLS, ROWS) : UL_BLOCKS(UL_OUT) UL_FRAGMENTS
                     : UL_MAIN_IN, UL_IN_COPY_COLS_A, UL_IN_COPY_ROWS_B, UL_IN_READ_COLS_A, UL_IN_READ_ROWS_B,
                       UL_KEPT(m, 96, 97, 98, 99, 100, 101, 102, 103), UL_KEPT(S, 104, 105, 106, 107, 108, 109, 110, 111),
                       UL_KEPT(C, 112, 113, 114, 115, 116, 117, 118, 119), UL_KEPT(T, 120, 121, 122, 123, 124, 125, 126, 127)
                     : UL_CLOBBERS);
    }
    // x = block (I, J) of the result, taken when it is needed.
    template <int I, int J>
    __device__ __forceinline__ void take(float (&x)[4]) const
    {
        UL_BLOCKS(UL_TAKE)
    }
    // Value p (4 i + r; -1: none, the result is then anything) of this lane in column block J.
    template <int J>
    __device__ __forceinline__ float pick(int p) const
    {
        float z = 0.0f, t;
        UL_COLUMNS(UL_PICK)
        return z;
    }
    // Where begin() left the copy cursors, B's one K tile further (a K_ROWS operand's offsets count from k = 0).
    __device__ __forceinline__ void cursors(uint64_t& pa, uint64_t& pb) const
    {
        pa = (uint64_t)(uintptr_t)a.src + (LA == K_COLS ? a.step : 0);
        pb = (uint64_t)(uintptr_t)b.src + (LB == K_COLS ? 2 * b.step : 0);
    }
    __device__ __forceinline__ void run(const Operand& A, int m0, const Operand& B, ColumnTile c, int K)
    {
        begin(A, m0, B, c, K);
        finish();
    }
};

// ---------------------------------------------------------------------------------------------
// 128 x 128 tile, four waves; two workgroups share a compute unit and cover each other's waits
// ---------------------------------------------------------------------------------------------
template <int LA, int LB>
struct TileSmall {
    static constexpr int BM = 128, BN = 128, NW = 4, NT = 256;
    static constexpr int WAVES_PER_SIMD = 2;
    static constexpr int MI = 4, NJ = 4;
    static constexpr int WAVES_M = 2;
    static constexpr size_t LDS_BYTES = 4 * (size_t)kHalfElems * sizeof(bf16_t);

    TileOperand<LA, NW, 1> a;
    TileOperand<LB, NW, 1> b;
    f32x4 acc[MI][NJ];
    int wave;

    static __device__ __forceinline__ int row_off(int wave, int i) { return (wave >> 1) * 64 + i * 16; }
    static __device__ __forceinline__ int col_off(int wave, int j) { return (wave & 1) * 64 + j * 16; }
    static __device__ __forceinline__ int wave_m(int wave) { return wave >> 1; }
    static __device__ __forceinline__ int blocks() { return NJ; }
    static __device__ __forceinline__ ColumnTile columns(int, int t) { return ColumnTile{t * BN, BN}; }

    __device__ __forceinline__ void init(unsigned char* lds)
    {
        wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        a.set_reads(reinterpret_cast<bf16_t*>(lds), (wave >> 1) * 64, threadIdx.x & 63);
        b.set_reads(reinterpret_cast<bf16_t*>(lds) + 2 * kHalfElems, (wave & 1) * 64, threadIdx.x & 63);
    }
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    __device__ __forceinline__ void copy_tile(int s)
    {
        a.copy(s);
        b.copy(s);
        a.advance();
        b.advance();
    }
    template <int I, int J>
    __device__ __forceinline__ void take(float (&x)[4]) const
    {
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = acc[I][J][r];
    }
    template <int J>
    __device__ __forceinline__ float pick(int p) const
    {
        float z = 0.0f;
        if (__any(p >= 0)) {
#pragma unroll
            for (int n = 0; n < 4 * MI; ++n) z = p == n ? acc[n / 4][J][n % 4] : z;
        }
        return z;
    }
    // The two workgroups of a compute unit cover each other's start: nothing is begun early.
    const Operand* next_a;
    const Operand* next_b;
    int next_m, next_n, next_k;
    __device__ __forceinline__ void begin(const Operand& A, int m0, const Operand& B, ColumnTile c, int K)
    {
        next_a = &A; next_b = &B; next_m = m0; next_n = c.first; next_k = K;
    }
    __device__ __forceinline__ void finish_keep(float (&m)[NJ], float (&S)[NJ], float (&C)[NJ], float (&T)[NJ]) { finish(); }
    __device__ __forceinline__ void finish() { run(*next_a, next_m, *next_b, ColumnTile{next_n, BN}, next_k); }
    // Tile k is in stage k & 1.  It is read once this wave's share has landed (the eight copies of tile
    // k + 1 may be outstanding) and everybody has passed a barrier; after the second barrier every wave
    // has its fragments in registers and tile k + 2 may overwrite the stage.
    __device__ __forceinline__ void run(const Operand& A, int m0, const Operand& B, ColumnTile c, int K)
    {
        clear();
        const int KT = K / kTileK;
        a.set_tile(A, m0, K, wave);
        b.set_tile(B, c.first, K, wave);
        a.set_copies(threadIdx.x & 63);
        b.set_copies(threadIdx.x & 63);
        copy_tile(0);
        if (KT > 1) copy_tile(1);
        for (int k = 0; k < KT; ++k) {
            if (k + 1 < KT) ULORL_WAIT_VMEM(8);
            else ULORL_WAIT_VMEM(0);
            bare_barrier();
            bf16x8 fa[2][4], fb[2][4];
            a.read(k & 1, fa);
            b.read(k & 1, fb);
            ULORL_WAIT_LDS(0);
            bare_barrier();
            if (k + 2 < KT) copy_tile(k & 1);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[ks][i], fb[ks][j], acc[i][j], 0, 0, 0);
        }
        bare_barrier();
    }
};

// ---------------------------------------------------------------------------------------------
// 128 x 128 tile for a contraction that is no multiple of 64 (both operands K_ROWS): copies through
// registers, with zeros past K
// ---------------------------------------------------------------------------------------------
struct TileRagged {
    static constexpr int BM = 128, BN = 128, NW = 4, NT = 256;
    static constexpr int WAVES_PER_SIMD = 2;
    static constexpr int MI = 4, NJ = 4;
    static constexpr int WAVES_M = 2;
    static constexpr int PITCH = kTileK + 8;                   // elements; the pad spreads rows over banks
    static constexpr size_t LDS_BYTES = 2 * (size_t)128 * PITCH * sizeof(bf16_t);

    f32x4 acc[MI][NJ];
    bf16_t* lds;

    static __device__ __forceinline__ int row_off(int wave, int i) { return (wave >> 1) * 64 + i * 16; }
    static __device__ __forceinline__ int col_off(int wave, int j) { return (wave & 1) * 64 + j * 16; }

    __device__ __forceinline__ void init(unsigned char* p) { lds = reinterpret_cast<bf16_t*>(p); }
    static __device__ __forceinline__ int blocks() { return NJ; }
    static __device__ __forceinline__ ColumnTile columns(int, int t) { return ColumnTile{t * BN, BN}; }
    __device__ __forceinline__ void run(const Operand& A, int m0, const Operand& B, ColumnTile c, int K)
    {
        const int n0 = c.first;
        const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        bf16_t* sA = lds;
        bf16_t* sB = lds + 128 * PITCH;
        for (int k0 = 0; k0 < K; k0 += kTileK) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int idx = tid + q * NT, row = idx / 8, kv = (idx % 8) * 8;
                u32x4 xa = {0u, 0u, 0u, 0u}, xb = {0u, 0u, 0u, 0u};
                if (k0 + kv < K) {                             // K is a multiple of 8
                    xa = *reinterpret_cast<const u32x4*>(A.p + (int64_t)min(m0 + row, A.count - 1) * A.ld + k0 + kv);
                    xb = *reinterpret_cast<const u32x4*>(B.p + (int64_t)min(n0 + row, B.count - 1) * B.ld + k0 + kv);
                }
                *reinterpret_cast<u32x4*>(sA + row * PITCH + kv) = xa;
                *reinterpret_cast<u32x4*>(sB + row * PITCH + kv) = xb;
            }
            __syncthreads();
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                bf16x8 fa[MI], fb[NJ];
                const int kk = ks * 32 + 8 * (lane >> 4);
#pragma unroll
                for (int i = 0; i < MI; ++i)
                    fa[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(sA + (row_off(wave, i) + (lane & 15)) * PITCH + kk));
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    fb[j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(sB + (col_off(wave, j) + (lane & 15)) * PITCH + kk));
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < NJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
            }
            __syncthreads();
        }
    }
};

// Workgroup -> tile mapping.  The hardware deals consecutive workgroup ids round-robin to the 8
// XCDs, each with its own L2.  Ids are first regrouped so that every XCD owns one contiguous
// range of logical tile numbers, and logical numbers walk the tile grid in blocks of group_m
// (default 4) tiles along M by all tiles along N (column-major inside the block): the 32
// workgroups resident on an XCD then cover about 4 x 8 tiles and share their A and B slices
// through that XCD's L2.
constexpr int kXcds = 8;

// bid: the workgroup's id within its kernel, or within its part of a launch that several products
// share (a part starts at a multiple of 8 workgroups, so bid % 8 is still the XCD).
__device__ __forceinline__ bool tile_coords(int bid, int num_m, int num_n, int group_m, int& tile_m, int& tile_n)
{
    const int total = num_m * num_n;
    const int per_xcd = (total + kXcds - 1) / kXcds;
    const int logical = (bid % kXcds) * per_xcd + bid / kXcds;
    if (bid / kXcds >= per_xcd || logical >= total) return false;
    const int group_size = group_m * num_n;
    const int group = logical / group_size;
    const int first_m = group * group_m;
    const int gm = min(group_m, num_m - first_m);
    const int in_group = logical % group_size;
    tile_m = first_m + in_group % gm;
    tile_n = in_group / gm;
    return true;
}

__host__ __device__ inline unsigned tile_grid(int num_m, int num_n)
{
    const int total = num_m * num_n;
    return (unsigned)(((total + kXcds - 1) / kXcds) * kXcds);
}

}  // namespace ulorl_detail

#endif
