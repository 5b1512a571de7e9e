// Which form of a kernel a call takes, where that depends on sizes and on the pattern's shape (host
// only, plain C++). Each rule gives the times, in us, on both sides of its line.
#pragma once

#include <cstdint>

namespace abilu_rules {

// Chunked application on chunks that are chains: sixteen lanes per chunk (k_fwd_chain, k_bwd_chain) or a
// quad per chunk. The sixteen lanes hold sixteen rows at a time, so on shorter chunks most of them repeat
// the last row: below five rows (FP64: seven, and ten with three blocks a side) the quad is faster, unless
// the chunks are so few that the idle lanes cost nothing. One and three sweeps each way, quad / sixteen:
//   500,000 line-ordered quads, FP32   1 row 177 / 563 (3 sweeps), 4 rows 164 / 167, 5 rows 177 / 146
//                               FP64   1 row 279 / 1,153, 5 rows 286 / 300, 6 rows 279 / 274, 8 rows 260 / 254
//   500,000 hexahedra (three a side)   FP32 4 rows 200 / 240, 5 rows 219 / 213
//                                      FP64 8 rows 345 / 408, 10 rows 387 / 367
//   120,000 quads   FP32 5 rows 50 / 50, 6 rows 54 / 45   FP64 6 rows 77 / 82, 8 rows 84 / 75
//    10,057 quads   FP32 2 rows (5,029 chunks) 28 / 27, 3 rows 30 / 26   FP64 2 rows 30 / 35, 3 rows 33 / 27
//    64,000 hexahedra   FP64 6 rows (10,667 chunks) 71 / 72, 8 rows (8,000 chunks) 84 / 56
inline bool chain_apply(int rows_per_chunk, int64_t nchunks, int side, bool f64) {
    const int rows = !f64 ? 5 : side <= 2 ? 7 : 10;
    return rows_per_chunk >= rows || (rows_per_chunk >= 3 && nchunks <= 8192);
}

}  // namespace abilu_rules
