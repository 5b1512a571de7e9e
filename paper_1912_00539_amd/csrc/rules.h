// Which form of a kernel a call takes, where that depends on sizes and on the pattern's shape (host
// only, plain C++). Each rule gives the times, in us, on both sides of its line.
#pragma once

#include <cstdint>

namespace abilu_rules {

// Application sweeps two at a time: rows of at most three blocks a side (a row of c blocks reads c^2 more:
// on the nine-point grid's rows of four that is more than the sweep saves), from three sweeps on, where
// most neighbours are near enough to be read again out of an L2 (`local`; `near` is the narrower distance).
// In single precision, where nearly every row has three blocks a side, the second reading and the longer
// records weigh as much as the sweep saved once the rows of an XCD and their neighbours' pass its L2.
// Three sweeps each way, single / pairs, hexahedra in planes of k x k cells:
//   FP32   64,000 cells k = 40 21.7 / 16.4, k = 120 (72,000) 22.7 / 21.3; 200,000 cells k = 100 48.8 / 49.0;
//          700,000 cells k = 20 156 / 149, k = 40 158 / 156, k = 50 157 / 157, k = 70 158 / 166, k = 100 160 / 177,
//          k = 120 161 / 186
//   FP64   700,000 cells k = 20 284 / 230, k = 70 290 / 257, k = 120 298 / 276
//   600,000 triangles in random order within 2,000 and 16,000 cells (up to three a side, 1.5 on average)
//          FP32 108 / 80 and 114 / 80, FP64 173 / 125 and 175 / 127
// `local` ends where quads lose (neighbours d rows away, 700,000 cells, FP32): d = 4,000 113 / 95,
// 12,000 114 / 107, 16,000 111 / 110 (150,000 cells 26.6 / 27.9); in FP64 there 207 / 175.
inline bool sweep_pairs(int nsweeps, int side, bool local, bool near, int64_t n, int64_t lower_blocks, bool f64) {
    if (nsweeps < 3 || side > 3 || !local) return false;
    return f64 || near || n <= 131072 || 2 * lower_blocks <= 5 * n;
}

// Launches of the backward sweeps 2 .. nsweeps, alone or two at a time. The first runs descending, behind the
// ascending forward sweeps, and each then opposite to the one before, so that it starts on the rows touched
// last; the Arnoldi SpMV behind an application runs opposite to its last launch.
inline int backward_launches(int nsweeps, bool pairs) { return nsweeps < 2 ? 0 : pairs ? nsweeps / 2 : nsweeps - 1; }
inline bool backward_descends(int launch) { return launch % 2 == 0; }
inline bool apply_ends_descending(int nsweeps, bool pairs) {
    const int launches = backward_launches(nsweeps, pairs);
    return launches > 0 && backward_descends(launches - 1);
}

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

// Chunked factor sweep on chains of rows with diagonal update sets: all rows at once and then the links
// (k_factor_chunk_far, k_factor_chunk_links) or whole rows, one after the other. The two launches write the
// diagonal blocks and the links' L twice and read them back, but no chain of loads runs through the rows.
// In double precision, and with three blocks a side, that pays almost always; in single precision with
// two where the chunks are long or few. One sweep, whole rows / two launches:
//   FP32, from A (with the initial inverses that whole rows need)
//     500,000 line-ordered quads   1 row 124 / 173, 2 rows 152 / 160, 4 rows 154 / 155,
//                                  5 rows 164 / 157, 6 rows 167 / 157, 8 rows 164 / 158, 64 rows 239 / 183
//     120,000 quads   1 row 34 / 47, 4 rows 37 / 39, 6 rows 41 / 42, 8 rows 42 / 40, 16 rows 57 / 46
//      10,057 quads   1 row 12 / 11, 4 rows 15 / 13
//   FP32, from the previous iterate
//     500,000 quads   1 row 195 / 261, 4 rows 231 / 254, 16 rows 241 / 259, 24 rows 272 / 264, 48 rows 254 / 260, 64 rows 293 / 275
//     120,000 quads   4 rows 47 / 54, 8 rows 51 / 54, 10 rows (12,000 chunks) 56 / 56, 12 rows 59 / 58, 16 rows 67 / 60
//      10,057 quads   1 row 14 / 18, 3 rows 16 / 18, 4 rows 18 / 18, 8 rows 28 / 21
//     500,000 hexahedra (three a side)   1 row 313 / 329, 2 rows 330 / 323, 16 rows 348 / 322
//   FP64, 500,000 quads   from A 1 row 233 / 208; from the previous iterate 1 row 365 / 376, 3 rows 374 / 369
inline bool chain_factor(int rows_per_chunk, int64_t nchunks, int side, bool f64, bool from_a) {
    const bool few = nchunks <= 12000;
    if (side > 2) return rows_per_chunk >= 2 || (f64 && from_a);
    if (f64) return from_a || rows_per_chunk >= 3;
    if (from_a) return rows_per_chunk >= 8 || few || (rows_per_chunk >= 5 && nchunks > 50000);
    return rows_per_chunk >= 24 || (rows_per_chunk >= 4 && few);
}

// The same in place, from A: few chunks all run side by side, and one sees little of the same sweep of
// another (ILU residual after it, by rows / by two launches: 629 chunks of line-ordered quads 3.44e-3 both,
// 1,000 chunks of hexahedra 1.0e-3 / 1.25e-3), while whole rows are bound by latency (629 chunks, FP32 44 / 24 us).
inline bool chain_factor_in_place(int64_t nchunks) { return nchunks <= 1024; }

// Synchronous factor sweep with a quad per block, or with a quad per row, on patterns whose rows do not fit
// the row-at-once form. With update sets off the diagonal the blocks win by up to half. With the diagonal
// ones alone only the diagonal blocks have pairs, and on large patterns with far neighbours a row's blocks,
// read together, pay for a row's serial chain. One sweep, rows / blocks:
//   from A, FP32   hexahedra in random order 396,800 cells (2.7 million blocks) 175 / 176, 550,000 (3.8) 240 / 254,
//                  700,000 306 / 335, shuffled within ten cells 400,000 152 / 141, 700,000 256 / 283;
//                  quads in random order 550,000 (2.7) 174 / 172, 800,000 (4.0) 251 / 265;
//                  shuffled within eight cells (near) 800,000 228 / 162
//   from A, FP64   700,000 hexahedra in random order 474 / 428, 800,000 quads 409 / 349
//   from the previous iterate, FP64   hexahedra in random order 150,000 157 / 158, 249,900 253 / 260,
//                  700,000 679 / 722; quads 250,000 189 / 191, 800,000 571 / 604; near 800,000 554 / 548
//   from the previous iterate, FP32   700,000 hexahedra 450 / 460, 550,000 359 / 362, shuffled within ten 426 / 414
inline bool sweep_by_blocks(int64_t n, int64_t blocks, int64_t lower_blocks, int64_t pairs, bool near, bool f64,
                            bool from_a) {
    if (pairs > lower_blocks || near || f64 == from_a) return true;
    return f64 ? n < 200000 : blocks < 3600000;
}

// Workgroups of the asynchronous first sweep from A that a compute unit takes at once, bounded (by LDS
// that the launch asks for and nobody uses) where rows are long and A is larger than the 256 MB cache that
// all XCDs share: each row in flight brings some 27 blocks and as many rows of others, and with four or more
// of these workgroups on every unit the rows push each other's blocks out. One sweep, as many as fit / three:
//   27-point rows   100,000 cells (333 MB) FP64 642 / 558, FP32 699 / 480; 294,000 FP64 1,885 / 1,602, FP32 2,064 / 1,376
//                    57,600 cells (186 MB) FP64 346 / 418, FP32 294 / 369
//   rows of 7       560,000 cells FP64 385 / 432, FP32 295 / 365
constexpr int CROWDED_LDS = 53000;   // bytes of 160 KB: three workgroups
inline bool crowded_sweep(int64_t n, int64_t blocks) { return blocks >= 18 * n && 128 * blocks > ((int64_t)256 << 20); }

// Launches of an application that FGMRES makes ahead of the status which decides on it. They cover the 6-8 us
// between the status being written and the next launch arriving; where the solve stops they were for
// nothing, which costs the more the longer a sweep takes. So two while a launch is shorter than that wait
// (60,000 rows of about eight blocks), one while it costs little beside an iteration, none beyond. A solve
// to 1e-10 (1e-2, two iterations or one), us, with none / one / two ahead:
//     48,000 rows, 191,380 blocks (triangles)   406 / 404 / 373 (165 / 157 / 152); FP64 432 / 417 / 399
//     24,000 rows, 168,000 blocks (nine-point)   572 / 537 / 526 (182 / 177 / 176)
//     40,000 rows, 199,000 blocks (quads, two sweeps)   438 / 428 / 419 (165 / 155 / 156)
//     60,000 rows, 299,000 blocks (quads, two sweeps)   493 / 477 / 465 (180 / 167 / 170)
//     80,000 rows, 399,000 blocks (quads)   490 / 473 / 462 (197 / 183 / 195)
//      8,000 rows, 195,112 blocks (27-point)   395 / 377 / 379 (217 / 213 / 220)
//     15,625 rows, 389,017 blocks (27-point)   443 / 427 / 421 (238 / 239 / 244)
//     57,600 rows, 1,475,944 blocks (27-point)   849 / 839 / 849 (497 / 505 / 516)
//    400,000 rows, 1,598,200 blocks (triangles)   1,365 / 1,349 / 1,379 (379 / 391 / 419)
//    230,000 rows, 1,600,000 blocks (nine-point)   1,876 / 1,829 / 1,839 (577 / 579 / 598)
//    400,000 rows, 2,800,000 blocks (nine-point)   2,971 / 2,907 / 2,944 (922 / 931 / 959)
//    700,000 rows, 2,797,600 blocks (triangles)   2,170 / 2,168 / 2,217 (591 / 621 / 666)
//    180,000 rows, 4,689,232 blocks (27-point)   2,294 / 2,316 / 2,355 (1,353 / 1,388 / 1,426)
inline int launches_ahead(int64_t n, int64_t blocks) {
    if (n <= 60000 && (blocks <= 150000 || blocks <= 8 * n)) return 2;
    return n <= 400000 && blocks <= 3000000 ? 1 : 0;
}

}  // namespace abilu_rules
