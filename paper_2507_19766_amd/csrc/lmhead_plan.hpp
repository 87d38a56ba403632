// How a call of the lm_head variant is carried out: which tile its products take, into how many parts they are cut, and where
// everything lies in the workspace.  No device code: the tests compile it by itself.
#ifndef ULORL_LMHEAD_PLAN_HPP
#define ULORL_LMHEAD_PLAN_HPP

#include <stddef.h>
#include <stdint.h>

#include "gemm_limits.hpp"

namespace ulorl_detail {

// Partial statistics of token t over one slice of the vocabulary: (max, sum, weighted sum,
// chosen logit or kEmpty).
struct StatQuad {
    float m, S, T, zy;
};

constexpr int kLiveBlock = 1024;                  // rows of a workgroup that looks for live ones

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline int64_t round_up64(int64_t x) { return (x + 63) / 64 * 64; }

constexpr int kComputeUnits = 256;

// ulorl_launch.gemm_tile: 0 = by shape, 1 = TileSmall (gemm_tile.hpp).
//
// Forward: what either tile's launch costs, in us, from a sweep of 64 to 4096 rows, hidden sizes of 512 to 2048 and
// vocabularies of 4096 to 151936 (both tiles at 96 shapes; the choice costs 0.3 % on average, 9 % at most 2 shapes, against
// the better of the two; "more than 256 rows and hidden size" cost 7.7 %).  A round of large tiles takes 8 us to start and
// to finish and 17 per 1024 of the hidden size, a little less when they are narrow; small tiles 1.5 us and 15.5 per 1024 for
// two on every compute unit, 9.3 for one.  us, large / small: 512 x 2048 x 4096 46 / 28, 512 x 2048 x 32008 64 / 75, 2048 x 2048 x
// 5000 53 / 63, 512 x 1024 x 20000 37 / 33, 128 x 1024 x 151936 85 / 77, 256 x 2048 x 151936 159 / 220, 4096 x 1024 x 4096 39 / 41.
// The large tile adds 48 rows of W to a lane's 32-bit offset (kMaxLargeColsLeadingDim).
inline int forward_tile(int asked, int64_t N, int64_t Hd, int64_t V)
{
    if (asked == 1 || Hd <= 256 || V > kMaxLargeColsLeadingDim) return 1;
    const int64_t ttiles = (N + 255) / 256, width = (N + 31) / 32 * 32 / ttiles;
    const double depth = Hd / 1024.0, narrow = 0.4 + 0.6 * (width > 160 ? (double)width : 160.0) / 256;
    const int64_t large = ttiles * ((V + 255) / 256), small = ((N + 127) / 128) * ((V + 127) / 128);
    const int64_t last = small % (2 * kComputeUnits);
    const double cost_large = (double)((large + kComputeUnits - 1) / kComputeUnits) * (8.0 + 17.0 * depth * narrow);
    const double cost_small = (double)(small / (2 * kComputeUnits)) * (1.5 + 15.5 * depth) +
                              (last == 0 ? 0.0 : last <= kComputeUnits ? 1.5 + 9.3 * depth : 1.5 + 15.5 * depth);
    return cost_small <= cost_large ? 1 : 0;
}
// Backward: small tiles where large ones would be mostly padding, too few for the chip, too short a contraction to pay for their
// start and their store, or a d_W of few tiles that contract over many rows.  us, large / small, rows x hidden x columns:
// 64 x 2048 x 151936 556 / 458, 512 x 512 x 151936 526 / 382, 777 x 512 534 / 557; 200 x 2048 x 20000 113 / 101, 256 x 2048 x 50000
// 276 / 256, 400 x 1024 x 100000 445 / 389, 300 x 2048 x 20000 112 / 116; few tiles: 1024 x 2048 x 4096 91 / 79, 2048 x 2048 x
// 4096 124 / 124, 2048 x 1024 x 4096 84 / 74, 1500 x 1024 x 5640 89 / 97, 4096 x 512 x 5000 126 / 102; 20000 x 512 x 4096 507 / 373, x 8192 645 / 662.
inline int backward_tile(int asked, int64_t N, int64_t Hd, int64_t V)
{
    const int64_t vtiles = (V + 255) / 256, dz_tiles = vtiles * ((N + 255) / 256), dw_tiles = vtiles * ((Hd + 255) / 256);
    const bool shallow = Hd <= 256 || N * Hd <= 3 * (1 << 17) || (Hd >= 1024 && N * Hd <= 1 << 19);
    return asked == 1 || shallow || dz_tiles < 112 || dw_tiles < 64 || dz_tiles + dw_tiles < 224 ? 1 : 0;
}

constexpr int tile_edge(int tile) { return tile == 1 ? 128 : 256; }

// Workspace of one call.  The forward and the backward call lay the same bytes out differently.
struct LmheadLayout {
    size_t total;
    size_t wp;                                                            // both calls
    size_t hp, token_ws, partial;                                         // forward
    size_t dz[2], dhacc, tail, rows, pos, row_map, block_count, n_live;   // backward
    int64_t hd64, v64;   // padded hidden size and vocabulary
    bool pad_k;          // the products read copies of hidden and W with zeros up to hd64 (Hd no multiple of 64)
    // V no multiple of 64: the dHidden product, which contracts over the vocabulary, reads a copy of W with zeros up to
    // v64 (pad_v) or takes W's last columns from a small copy of theirs, into an accumulator of their own (tail_v).
    // The first moves 4 V Hd bytes, the second 8 N Hd.  Backward, 1000 columns: 20000 x 2048 570 / 650 us, x 5120 905 / 1110;
    // 50264 columns: 150 x 128 96 / 93, 100008 columns: 3000 x 1024 1860 / 1725.
    bool pad_v, tail_v;
    int64_t chunk;       // vocabulary columns per backward launch, a multiple of 64 (leading dimension of dZ)
    int dh_splits, dh_slabs;
    int splits;
    int v_per_split;
};

// Vocabulary slices of the forward statistics: a workgroup takes one tile of tokens and one slice.  Rounds
// of the chip's tile slots times tiles per slice (plus about a third of a tile per workgroup for its
// start and its merge) is what the launch costs; at least 8 slices, so that the workgroups of an XCD
// (tile_coords) form a block of 4 token tiles by 8 slices and share both operands in its L2.
inline int stats_splits(int64_t N, int64_t V, int edge, int slots, int most)
{
    const int ttiles = (int)((N + edge - 1) / edge), vtiles = (int)((V + edge - 1) / edge);
    const int lo = vtiles < 8 ? vtiles : 8, hi = vtiles < most ? vtiles : most;
    int best = lo;
    double best_cost = (double)(((int64_t)ttiles * lo + slots - 1) / slots) * ((double)((vtiles + lo - 1) / lo) + 0.35);
    for (int rounds = 1; rounds <= 8; ++rounds) {           // the most slices that fit that many rounds
        int s = rounds * slots / ttiles;
        if (s < lo) continue;
        if (s > hi) s = hi;
        const double cost = (double)rounds * ((double)((vtiles + s - 1) / s) + 0.35);
        if (cost < best_cost - 1e-9) {
            best = s;
            best_cost = cost;
        }
        if (s == hi) break;
    }
    return best;
}

// token_ws: bytes of the token loss's own workspace.
inline LmheadLayout lmhead_layout(int64_t N, int64_t Hd, int64_t V, int32_t vocab_chunk, int fwd_tile, size_t token_ws)
{
    LmheadLayout L;
    L.hd64 = round_up64(Hd);
    L.v64 = round_up64(V);
    L.pad_k = L.hd64 != Hd;
    L.pad_v = L.v64 != V && (L.pad_k || V < 2 * N);
    L.tail_v = L.v64 != V && !L.pad_v;
    const int64_t n64 = round_up64(N);
    const size_t padded_w = (size_t)L.hd64 * (size_t)L.v64 * 2;
    const size_t count_blocks = (size_t)((N + kLiveBlock - 1) / kLiveBlock) * sizeof(int);
    const size_t slice = (size_t)N * sizeof(StatQuad), slab = (size_t)N * Hd * 4, column = (size_t)n64 * 2;
    size_t off;
    auto place = [&](size_t bytes) {
        const size_t at = off;
        off = align_up(off + bytes, 256);
        return at;
    };
    auto larger = [](size_t x, size_t y) { return x > y ? x : y; };
    auto smaller = [](size_t x, size_t y) { return x < y ? x : y; };
    auto forward = [&](size_t slices) {
        off = 0;
        L.wp = place(L.pad_k ? padded_w : 0);
        L.hp = place(L.pad_k ? (size_t)n64 * L.hd64 * 2 : 0);
        L.token_ws = place(token_ws);
        L.partial = place(slices * slice);
        return off;
    };
    // The dZ chunks in front: 5.55 ms where they began at any multiple of 256 bytes 5.88 (20000 x 128 x 151936).
    auto backward = [&](size_t dz_bytes, int buffers, size_t slab_bytes) {
        off = 0;
        L.wp = place(L.pad_k || L.pad_v ? padded_w : 0);
        L.dz[0] = place(dz_bytes);
        L.dz[1] = buffers == 2 ? place(dz_bytes) : L.dz[0];
        L.dhacc = place(slab_bytes);
        L.tail = place(L.v64 != V && !L.pad_k ? (size_t)Hd * kTileK * 2 : 0);
        L.rows = place((size_t)n64 * L.hd64 * 2);
        L.pos = place((size_t)N * sizeof(int));
        L.row_map = place((size_t)n64 * sizeof(int));
        L.block_count = place(count_blocks);
        L.n_live = place(sizeof(int));
        return off;
    };

    // What more room than the least is used for.  Statistics: 8 to 128 slices (up to 512 where
    // the room is there all the same).  dHidden (see BwdStepArgs): enough tiles for
    // every compute unit, at most 8 parts.  dZ: vocab_chunk columns, or what a buffer of 64 to 256 MB (as W and
    // hidden are larger) holds: with few rows a chunk of 8192 columns is too little work for 256 compute
    // units.  777 x 2048 x 151936: 20 steps of 8192 columns 3.3 ms, all columns in one chunk 1.4 ms.  With 16384 rows
    // and more the width does not matter (8192, 16384, 32768: +-0.5 %).
    const int tail_slab = L.tail_v ? 1 : 0;
    const int64_t weights = (V + N) * Hd;                        // half the bytes of hidden and W
    const size_t budget = weights < ((int64_t)64 << 20) ? (size_t)64 << 20 : weights > ((int64_t)256 << 20) ? (size_t)256 << 20 : (size_t)weights;
    const int64_t least = vocab_chunk < L.v64 ? vocab_chunk : L.v64;
    const size_t dz_least = align_up(column * least, 256), dz_all = align_up(column * L.v64, 256);
    constexpr size_t kTileRound = (size_t)kComputeUnits * 256 * 256 * 4;
    const size_t slabs_most = larger(slab, smaller(8 * slab, kTileRound)) + tail_slab * slab;

    // What a call asks for grows with N, R and vocab_chunk, so that a workspace sized for the largest batch serves the
    // smaller ones, and has a bound that vocab_chunk sets: the larger of 16 KB a column beyond the least, and twice hidden
    // and W, four dZ chunks, one dHidden accumulator, 16 statistics a row and the token loss.
    const size_t need = larger(forward(8), backward(dz_least, 2, (1 + tail_slab) * slab));
    const size_t dz_most = dz_all <= budget ? larger(2 * dz_least, dz_all) : 2 * larger(dz_least, budget);
    const size_t use = larger(forward(128), backward(dz_most, 1, slabs_most));
    off = 0;
    if (L.pad_k) place(padded_w);
    place((size_t)V * Hd * 2);
    place((size_t)Hd * n64 * 2);
    for (int b = 0; b < 2; ++b) {
        place((size_t)N * vocab_chunk * 2);
        place((size_t)vocab_chunk * n64 * 2);
    }
    place(slab);
    place(16 * slice);
    place(token_ws);
    place((size_t)N * Hd * 2);
    place((size_t)N * sizeof(int));
    place((size_t)n64 * sizeof(int));
    place(count_blocks);
    place(sizeof(int));
    L.total = larger(need, smaller(use, larger(off, need + (size_t)vocab_chunk * 16384)));

    const size_t room_slices = (L.total - forward(0)) / slice;
    const int edge = tile_edge(fwd_tile);
    const int64_t vtiles = (V + edge - 1) / edge;
    const int64_t slices = stats_splits(N, V, edge, fwd_tile == 1 ? 2 * kComputeUnits : kComputeUnits, (int)smaller(room_slices, 512));
    const int64_t per_split = (vtiles + slices - 1) / slices;
    L.v_per_split = (int)(per_split * edge);
    L.splits = (int)((vtiles + per_split - 1) / per_split);

    // Every column in one dZ buffer if that and half of the accumulators fit, else up to a quarter of the room for the accumulators.
    const size_t room = L.total - backward(0, 1, 0);
    auto slabs = [&](int64_t n) { return align_up((size_t)(n + tail_slab) * slab, 256); };
    int64_t dh_splits = kComputeUnits / (((N + 255) / 256) * ((Hd + 255) / 256));
    dh_splits = dh_splits > 8 ? 8 : dh_splits < 1 ? 1 : dh_splits;
    int64_t chunk = L.v64;
    int64_t fitting = dh_splits;                 // accumulators beside a dZ of all columns
    while (fitting > 0 && slabs(fitting) + dz_all > room) --fitting;
    // With few of them a handful of workgroups contract over all columns: 1500 x 512 x 50000, two of eight, 858 us; in three chunks 320.
    if (chunk <= kMaxLeadingDim - 256 && fitting > 0 && 2 * fitting >= dh_splits) {
        dh_splits = fitting;
    } else {
        while (dh_splits > 1 && (slabs(dh_splits) + 2 * dz_least > room || slabs(dh_splits) > room / 4)) --dh_splits;
        const size_t half = (room - slabs(dh_splits)) / 2 / 256 * 256;
        chunk = (int64_t)(smaller(budget, half) / column / 64 * 64);
        if (chunk >= 256) chunk = chunk / 256 * 256;
        if (chunk < vocab_chunk) chunk = vocab_chunk;
        if (chunk > kMaxLeadingDim - 256) chunk = (kMaxLeadingDim - 256) / 64 * 64;      // at least vocab_chunk: see check_lmhead
        if (chunk > L.v64) chunk = L.v64;
    }
    if (dh_splits > chunk / 1024) dh_splits = chunk / 1024;      // no part shorter than 16 K tiles
    if (dh_splits < 1) dh_splits = 1;
    L.chunk = chunk;
    L.dh_splits = (int)dh_splits;
    L.dh_slabs = L.dh_splits + tail_slab;
    forward(L.splits);
    // two dz buffers: one chunk's products read theirs while the next chunk's dz is written
    backward(column * chunk, chunk < V ? 2 : 1, (size_t)L.dh_slabs * slab);
    return L;
}

}  // namespace ulorl_detail

#endif
