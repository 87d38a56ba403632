// What the block tiles of gemm_tile.hpp can address; no device code.
#ifndef ULORL_GEMM_LIMITS_HPP
#define ULORL_GEMM_LIMITS_HPP

#include <stdint.h>

namespace ulorl_detail {

constexpr int kTileK = 64;                       // contraction depth of one LDS stage
// Operands are addressed by 32-bit byte offsets: K_ROWS from a tile's first row (up to 256 rows of ld elements), K_COLS from the
// first of four rows (small tile) or of 52 (large tile).  With at most kMaxLeadingDim elements any stays below 2^31 bytes;
// larger ones are checked by the caller (k_rows_fit, kMaxColsLeadingDim, kMaxLargeColsLeadingDim).
constexpr int64_t kMaxLeadingDim = 1 << 22;
constexpr int64_t kMaxColsLeadingDim = 1 << 29;
constexpr int64_t kMaxLargeColsLeadingDim = 1 << 25;
inline bool k_rows_fit(int64_t tile_rows, int64_t ld, int64_t K) { return ((tile_rows - 1) * ld + K) * 2 <= 0xffffffffLL; }

}  // namespace ulorl_detail

#endif
