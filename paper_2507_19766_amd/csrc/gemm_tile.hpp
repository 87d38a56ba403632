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

namespace ulorl_detail {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t bf16_t;  // raw storage

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    f32x2 x = {lo, hi};
    bf16x2 b = __builtin_convertvector(x, bf16x2);  // round to nearest even
    return __builtin_bit_cast(uint32_t, b);
}
__device__ __forceinline__ bf16_t to_bf16(float x) { return (bf16_t)(pack_bf16x2(x, 0.0f) & 0xffffu); }

enum { K_ROWS = 0, K_COLS = 1 };

// One operand of a product: `count` rows (columns) of the result, its memory layout is the kernel's
// template argument.
struct Operand {
    const bf16_t* p;
    int64_t ld;
    int count;
};

constexpr int kTileK = 64;                       // contraction depth of one LDS stage
constexpr int kHalf = 128;                       // rows (columns) of one half tile: the unit of copying
constexpr int kHalfElems = kHalf * kTileK;       // 16 KB
// Word 3 of a raw (unstructured, stride 0) buffer descriptor on gfx9-family parts: 32-bit data format.
constexpr int kRawBufferFlags = 0x00020000;
// Operands are addressed by 32-bit byte offsets: K_ROWS from a tile's first row (up to 256 rows of ld elements), K_COLS from the
// first of four rows.  With at most kMaxLeadingDim elements either stays below 2^31 bytes; larger ones are
// checked by the caller (k_rows_fit, kMaxColsLeadingDim).
constexpr int64_t kMaxLeadingDim = 1 << 22;
constexpr int64_t kMaxColsLeadingDim = 1 << 29;
inline bool k_rows_fit(int64_t tile_rows, int64_t ld, int64_t K) { return ((tile_rows - 1) * ld + K) * 2 <= 0xffffffffLL; }

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
template <int LAYOUT, int NW, int HALVES, int BLOCKS>
struct TileOperand {
    static constexpr int J = 16 / NW;            // copy instructions per wave and half tile
    static constexpr int NV = LAYOUT == K_ROWS ? HALVES * J : HALVES;
    static constexpr int NR = LAYOUT == K_ROWS ? 2 : BLOCKS;
    const char* src;          // this wave's rows of the K tile at the copy cursor (uniform)
    int64_t step;             // bytes from one K tile to the next
    int64_t row_step;         // K_COLS: bytes from copy instruction j to j + 1
    int soff;                 // K_ROWS: byte offset of the copy cursor along k
    uint32_t extent;
    uint32_t voff[NV];        // this lane's byte offset
    int roff[NR];             // this lane's LDS read offset, in bytes inside a half
    bf16_t* lds;              // [stage][half]
    int wave;

    // first: first row (column) of the tile; the copy cursor is at k = 0.  Rows past op.count are
    // taken from the last one (their results are ignored).
    __device__ __forceinline__ void set_tile(const Operand& op, int first, int64_t K)
    {
        const int lane = threadIdx.x & 63;
        if constexpr (LAYOUT == K_ROWS) {
            src = reinterpret_cast<const char*>(op.p + (int64_t)first * op.ld);
            soff = 0;
            const int rows = min(HALVES * kHalf, op.count - first);
            const uint64_t ext = ((uint64_t)(rows - 1) * (uint64_t)op.ld + (uint64_t)K) * 2;
            extent = (uint32_t)min(ext, (uint64_t)0xffffffffu);
#pragma unroll
            for (int h = 0; h < HALVES; ++h)
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const int row = (j * NW + wave) * 8 + lane / 8;
                    const int vec = (lane % 8) ^ ((row >> 1) & 7);
                    const int r = min(h * kHalf + row, rows - 1);
                    voff[h * J + j] = (uint32_t)(((int64_t)r * op.ld + vec * 8) * 2);
                }
        } else {
            const int cols = min(HALVES * kHalf, op.count - first);
            src = reinterpret_cast<const char*>(op.p + (int64_t)(wave * 4) * op.ld + first);
            step = (int64_t)kTileK * op.ld * 2;
            row_step = (int64_t)NW * 4 * op.ld * 2;
            const uint64_t ext = ((uint64_t)3 * (uint64_t)op.ld + (uint64_t)cols) * 2;
            extent = (uint32_t)min(ext, (uint64_t)0xffffffffu);
            const int k = wave * 4 + lane / 16;
            const int vec = (lane % 16) ^ (((k & 3) << 2) | (((k >> 3) & 1) << 1));
#pragma unroll
            for (int h = 0; h < HALVES; ++h) {
                const int col = min(h * kHalf + vec * 8, cols - 8);      // counts are multiples of 8
                voff[h] = (uint32_t)(((int64_t)(lane / 16) * op.ld + col) * 2);
            }
        }
    }

    __device__ __forceinline__ void set_reads(bf16_t* lds_, int wave_, int wave_row)
    {
        lds = lds_;
        wave = wave_;
        const int lane = threadIdx.x & 63;
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

    // This wave's share of half h of the K tile `back` tiles before the cursor, into stage s; one of its J instructions.
    __device__ __forceinline__ void copy_part(int j, int h, int s, int back = 0) const
    {
        bf16_t* dst = lds + (s * HALVES + h) * kHalfElems;
        if constexpr (LAYOUT == K_ROWS) {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(src), 0, (int)extent, kRawBufferFlags);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(dst + (j * NW + wave) * 512), 16,
                                                     voff[h * J + j], soff - back * kTileK * 2, 0, 0);
        } else {
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(src + j * row_step - back * step), 0, (int)extent, kRawBufferFlags);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(dst + (j * NW + wave) * 512), 16,
                                                     voff[h], 0, 0, 0);
        }
    }
    __device__ __forceinline__ void copy(int h, int s, int back = 0) const
    {
#pragma unroll
        for (int j = 0; j < J; ++j) copy_part(j, h, s, back);
    }
    __device__ __forceinline__ void advance()
    {
        if constexpr (LAYOUT == K_ROWS) soff += kTileK * 2;
        else src += step;
    }

    // The fragments of half h in stage s: f[ks][b], lane L: row 16 b + L % 16, k = 32 ks + 8 (L / 16) ..+7.
    // K_COLS fragments have arrived on return; K_ROWS ones are waited for by the caller (or their use).
    // The compiler's builtin for the transposing read is taken for a possible LDS write and gets a wait
    // for ALL copies in flight put before it; here the reads are issued and waited for in one block.
    __device__ __forceinline__ void read(int h, int s, bf16x8 (&f)[2][BLOCKS]) const
    {
        bf16_t* half = lds + (s * HALVES + h) * kHalfElems;
        if constexpr (LAYOUT == K_ROWS) {
            const char* base = reinterpret_cast<const char*>(half);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int b = 0; b < BLOCKS; ++b)
                    f[ks][b] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(base + roff[ks] + b * 16 * 128));
        } else {
            const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) bf16_t*)half;
            static_assert(BLOCKS == 2 || BLOCKS == 4, "fragment reads are written out");
            u32x2 r[4 * BLOCKS];          // [ks][block][low / high four k]
            if constexpr (BLOCKS == 4) {
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
            } else {
                asm volatile(
                "ds_read_b64_tr_b16 %0, %8\n\t"
                "ds_read_b64_tr_b16 %1, %8 offset:1024\n\t"
                "ds_read_b64_tr_b16 %2, %9\n\t"
                "ds_read_b64_tr_b16 %3, %9 offset:1024\n\t"
                "ds_read_b64_tr_b16 %4, %8 offset:8192\n\t"
                "ds_read_b64_tr_b16 %5, %8 offset:9216\n\t"
                "ds_read_b64_tr_b16 %6, %9 offset:8192\n\t"
                "ds_read_b64_tr_b16 %7, %9 offset:9216\n\t"
                    "s_waitcnt lgkmcnt(0)"
                    : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
                    : "v"(base + roff[0]), "v"(base + roff[1])
                    : "memory");
            }
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

// ---------------------------------------------------------------------------------------------
// 256 x 256 tile, eight waves in two groups of four that take turns
// ---------------------------------------------------------------------------------------------
// A wave alternates read phases (fragments LDS -> registers) and multiply phases (16 MFMAs), with a
// barrier after each; its share of a copy global -> LDS is issued in one of the two, see below.  The second group runs one phase behind the
// first, and each SIMD holds one wave of each group: while one multiplies, the other reads, so the
// matrix pipe always has a wave with its operands in registers.  (With all eight waves in step, as
// before, every wave waited for its fragments at the same time.)
//
// Wave (wm, wn), wm = group, owns the four 64 x 32 pieces at rows 128 h + 64 wm, columns 128 g + 32 wn;
// per K tile it multiplies them in the order (0,0) (0,1) (1,0) (1,1):
//     phase   reads                 copies (tile k + 2)     multiplies
//     1       A half 0              B half 0                (0,0)
//     2       B half 1              A half 0                (0,1)
//     3       A half 1              B half 1                (1,0)
//     4       B half 0 of k + 1     A half 1                (1,1)
// Count barriers as time slots; in slot s group 0 runs segment s of its sequence [read, multiply, read,
// ...] and group 1 segment s - 1.
//   * A half may be overwritten by a copy issued one read phase after the phase that read it: group 0
//     issues it in slot s + 2, group 1 finished its reads (waited for before its barrier) in slot s + 1.
//   * A half is read in the read phase after one that ended with a wait for it: each wave waits for its
//     own share and then passes the barrier; group 1's wait lies in slot s + 1, the first read in s + 2.
//     Copies complete in order, and six halves (twelve instructions of a wave) are issued after the one
//     the next phase needs: so every read phase ends with "at most 12 outstanding" -- ten where the
//     phase's own copy is issued after that wait, in the multiply phase (one slot later: also safe).
// Both LDS stages are in flight all the time: a copy has six phase pairs (about 3000 clocks) to land.
//
// Where the copy goes: the read phase is the longer of the two (four waves take 32 KB out of LDS in about the
// 256 clocks that 16 MFMAs last), and a copy instruction holds up the reads behind it.  With both operands
// K_ROWS it is issued right after the reads and overlaps them; a K_COLS read returns only when its data
// is there, so the copy goes between the MFMAs instead, its two instructions apart.  Products of
// 8192 x 32768 x 2048, TFLOP/s, copy before the reads / after them / between the MFMAs: both K_ROWS 1493 /
// 1570 / 1539 (contraction 8192, strided: 1461 / 1557 / 1513), A K_COLS 1425 / 1395 / 1434, both K_COLS
// 1365 / 1363 / 1412.  (Copies out of L2 only would be 3 to 8 % faster still, no copies at all 22 %.)
//
// Against 1240 / 1340 for the eight-waves-in-step loop it replaces at 2048 x 8192 x 32768 / 32768 x 2048 x 8192
// (hipBLASLt: 1550 / 1570 on the same card).  Raising the multiplying wave's priority (s_setprio) made it
// 3 % slower.
template <int LA, int LB>
struct TileLarge {
    static constexpr int BM = 256, BN = 256, NW = 8, NT = 512;
    static constexpr int WAVES_PER_SIMD = 2;
    static constexpr int MI = 8, NJ = 4;                       // 16 x 16 blocks of a wave
    static constexpr int WAVES_M = 2;
    static constexpr bool kCopyAfterReads = LA == K_ROWS && LB == K_ROWS;
    static constexpr int kSteady = kCopyAfterReads ? 12 : 10;  // copy instructions outstanding at the end of a read phase
    static constexpr size_t LDS_BYTES = 8 * (size_t)kHalfElems * sizeof(bf16_t);

    TileOperand<LA, NW, 2, 4> a;
    TileOperand<LB, NW, 2, 2> b;
    f32x4 acc[MI][NJ];
    bf16x8 fa[2][4], fb[2][2][2];
    int wm;

    static __device__ __forceinline__ int row_off(int wave, int i) { return (i >> 2) * 128 + (wave >> 2) * 64 + (i & 3) * 16; }
    static __device__ __forceinline__ int col_off(int wave, int j) { return (j >> 1) * 128 + (wave & 3) * 32 + (j & 1) * 16; }
    static __device__ __forceinline__ int wave_m(int wave) { return wave >> 2; }

    __device__ __forceinline__ void init(unsigned char* lds)
    {
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        wm = wave >> 2;
        a.set_reads(reinterpret_cast<bf16_t*>(lds), wave, (wave >> 2) * 64);
        b.set_reads(reinterpret_cast<bf16_t*>(lds) + 4 * kHalfElems, wave, (wave & 3) * 32);
    }
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    // 16 MFMAs; `copy(j)` issues instruction j (0, 1) of a copy between them.
    template <int H, int G, class Copy>
    __device__ __forceinline__ void multiply(Copy copy)
    {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[H * 4 + i][G * 2 + j] =
                        __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[ks][i], fb[G][ks][j], acc[H * 4 + i][G * 2 + j], 0, 0, 0);
                if (ks == 0 && i == 1) copy(0);
                if (ks == 1 && i == 0) copy(1);
            }
        bare_barrier();
    }
    template <int H, int G>
    __device__ __forceinline__ void multiply()
    {
        multiply<H, G>([](int) {});
    }
    // End of a read phase: the fragments are in registers, and at most VM of this wave's copies are outstanding.
    template <int VM>
    __device__ __forceinline__ void read_done()
    {
        ULORL_WAIT_LDS(0);
        if constexpr (VM >= 0) ULORL_WAIT_VMEM(VM);
        bare_barrier();
    }
    // One K tile out of stage s.  COPY: the copies of tile k + 2 go along; NEXT: there is a tile k + 1.
    template <bool COPY, bool NEXT, int W1, int W2, int W3, int W4>
    __device__ __forceinline__ void tile(int s)
    {
        a.read(0, s, fa);
        phase<0, 0, COPY, W1>(b, 0, s);
        b.read(1, s, fb[1]);
        phase<0, 1, COPY, W2>(a, 0, s);
        a.read(1, s, fa);
        phase<1, 0, COPY, W3>(b, 1, s);
        if constexpr (NEXT) b.read(0, s ^ 1, fb[0]);
        phase<1, 1, COPY, W4>(a, 1, s);
        if constexpr (COPY) {
            a.advance();
            b.advance();
        }
    }
    // The rest of a phase whose reads have been issued: the copy of half h of operand op, the waits, the MFMAs.
    template <int H, int G, bool COPY, int W, class Op>
    __device__ __forceinline__ void phase(const Op& op, int h, int s)
    {
        if constexpr (COPY && kCopyAfterReads) {
            __builtin_amdgcn_sched_barrier(0);
            op.copy(h, s);
        }
        read_done<W>();
        multiply<H, G>([&](int j) {
            if constexpr (COPY && !kCopyAfterReads) {
                __builtin_amdgcn_sched_barrier(0);
                op.copy_part(j, h, s);
                __builtin_amdgcn_sched_barrier(0);
            }
        });
    }
    __device__ __forceinline__ void copy_tile(int s)
    {
        b.copy(0, s);
        a.copy(0, s);
        b.copy(1, s);
        a.copy(1, s);
        a.advance();
        b.advance();
    }
    // First copies and the first read; the second group falls one phase behind.
    template <int W0, int W1>
    __device__ __forceinline__ void start()
    {
        ULORL_WAIT_VMEM(W0);               // half 0 of B has landed (this wave's share) ...
        bare_barrier();                    // ... and everybody's
        if (wm == 1) bare_barrier();
        b.read(0, 0, fb[0]);
        read_done<W1>();                   // half 0 of A
        bare_barrier();                    // the multiply phase that would follow
    }
    // A tile with no column beyond the first 128: only half 0 of B exists, two phases per K tile,
    //     phase   reads                   copies                     multiplies
    //     1       B half 0, A half 0      A half 1 of k + 1          (0,0)
    //     2       A half 1                B, A halves 0 of k + 2     (1,0)
    // and by the same count of slots as above: what phase 1 reads was waited for at the end of phase 2 before
    // (three halves are issued after it: six instructions), what phase 2 reads at the end of phase 1
    // (likewise), and every copy goes where the phase before it read.
    // It takes about three quarters of a whole tile's time (three quarters of the copies, the same start and
    // store).  Backward call, 2048 x 151936, whole / half last tile: 300 rows 819 / 800 us, 520 1145 / 1105,
    // 777 1513 / 1489, 2100 3327 / 3234.
    static __device__ __forceinline__ bool half_tile(const Operand& B, int n0) { return B.count - n0 <= kHalf; }
    template <bool COPY1, bool COPY2, int W1, int W2>
    __device__ __forceinline__ void tile_half(int s)
    {
        if constexpr (COPY1) a.copy(1, s ^ 1, 1);
        b.read(0, s, fb[0]);
        a.read(0, s, fa);
        read_done<W1>();
        multiply<0, 0>();
        if constexpr (COPY2) {
            b.copy(0, s);
            a.copy(0, s);
            a.advance();
            b.advance();
        }
        a.read(1, s, fa);
        read_done<W2>();
        multiply<1, 0>();
    }
    __device__ __forceinline__ void run_half(int KT)
    {
        b.copy(0, 0);
        a.copy(0, 0);
        a.copy(1, 0);
        a.advance();
        b.advance();
        if (KT > 1) {
            b.copy(0, 1);
            a.copy(0, 1);
            a.advance();
            b.advance();
            ULORL_WAIT_VMEM(6);
        } else {
            ULORL_WAIT_VMEM(2);
        }
        bare_barrier();
        if (wm == 1) bare_barrier();
        int k = 0;
        for (; k + 2 < KT; ++k) tile_half<true, true, 6, 6>(k & 1);
        if (KT > 1) {
            tile_half<true, false, 6, 2>(k & 1);
            ++k;
        }
        tile_half<false, false, 0, -1>(k & 1);
        if (wm == 0) bare_barrier();
    }
    // acc = the product over K (a positive multiple of 64).  On return every wave is past its last LDS read.
    __device__ __forceinline__ void run(const Operand& A, int m0, const Operand& B, int n0, int K)
    {
        clear();
        const int KT = K / kTileK;
        a.set_tile(A, m0, K);
        b.set_tile(B, n0, K);
        if (half_tile(B, n0)) {
            run_half(KT);
            return;
        }
        copy_tile(0);
        if (KT > 1) {
            copy_tile(1);
            start<14, 12>();
            int k = 0;
            for (; k + 2 < KT; ++k) tile<true, true, kSteady, kSteady, kSteady, kSteady>(k & 1);
            tile<false, true, 10, 8, 6, 4>(k & 1);
            ++k;
            tile<false, false, 2, 0, -1, -1>(k & 1);
        } else {
            start<6, 4>();
            tile<false, false, 2, 0, -1, -1>(0);
        }
        if (wm == 0) bare_barrier();       // the groups are in step again
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

    TileOperand<LA, NW, 1, 4> a;
    TileOperand<LB, NW, 1, 4> b;
    f32x4 acc[MI][NJ];

    static __device__ __forceinline__ int row_off(int wave, int i) { return (wave >> 1) * 64 + i * 16; }
    static __device__ __forceinline__ int col_off(int wave, int j) { return (wave & 1) * 64 + j * 16; }
    static __device__ __forceinline__ int wave_m(int wave) { return wave >> 1; }
    static __device__ __forceinline__ bool half_tile(const Operand&, int) { return false; }

    __device__ __forceinline__ void init(unsigned char* lds)
    {
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        a.set_reads(reinterpret_cast<bf16_t*>(lds), wave, (wave >> 1) * 64);
        b.set_reads(reinterpret_cast<bf16_t*>(lds) + 2 * kHalfElems, wave, (wave & 1) * 64);
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
        a.copy(0, s);
        b.copy(0, s);
        a.advance();
        b.advance();
    }
    // Tile k is in stage k & 1.  It is read once this wave's share has landed (the eight copies of tile
    // k + 1 may be outstanding) and everybody has passed a barrier; after the second barrier every wave
    // has its fragments in registers and tile k + 2 may overwrite the stage.
    __device__ __forceinline__ void run(const Operand& A, int m0, const Operand& B, int n0, int K)
    {
        clear();
        const int KT = K / kTileK;
        a.set_tile(A, m0, K);
        b.set_tile(B, n0, K);
        copy_tile(0);
        if (KT > 1) copy_tile(1);
        for (int k = 0; k < KT; ++k) {
            if (k + 1 < KT) ULORL_WAIT_VMEM(8);
            else ULORL_WAIT_VMEM(0);
            bare_barrier();
            bf16x8 fa[2][4], fb[2][4];
            a.read(0, k & 1, fa);
            b.read(0, k & 1, fb);
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
    __device__ __forceinline__ void run(const Operand& A, int m0, const Operand& B, int n0, int K)
    {
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
