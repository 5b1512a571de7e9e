// Device bodies of the library's kernels, shared by the single-request kernels (one system per
// launch) and the batched serving kernels (one launch over the tiles of many systems). Every body
// takes its tile index `blk` explicitly; the arithmetic lives only here.
#pragma once

#include <type_traits>

#include "abilu_internal.h"

namespace abilu_k {

using namespace abilu;
using namespace abilu_dev;

constexpr int CH = 2;                        // factor sweep: blocks of a row loaded together
// Waves per SIMD the single-precision factor sweeps are compiled for (at most 102 VGPRs). The
// first sweep from A, which inverts a gathered A_jj for each of the two lower blocks in flight,
// would otherwise take 107 VGPRs and run 4 waves; it fits 5 without spilling. The FP64 sweeps
// keep the compiler's choice (at this budget they would spill).
template <typename T>
constexpr int sweep_waves() { return sizeof(T) == 4 ? 5 : 1; }
// apply sweeps: block rows per quad (FP32: two rows keep enough loads in flight; FP64 rows carry
// twice the bytes and run faster one per quad) and rows per workgroup
template <typename T>
constexpr int rpq() { return sizeof(T) == 8 ? 1 : 2; }
template <typename T>
constexpr int rows_per_wg2() { return rpq<T>() * ROWS_PER_WG; }
constexpr int MAX_RESTART = 256;
constexpr int SPMV_ROWS = WG / 8;            // SpMV: eight lanes per block row

// status slots (double[8] in the workspace header; the server copies them to the host)
enum { ST_EST = 0, ST_HN = 1, ST_BETA = 2, ST_NUM = 3, ST_GUARD = 4 };
// A single solve's status reaches the host through the pattern's pinned buffer: PIN_SLOTS slots of
// PIN_WORDS 8-byte words from word PIN_BASE on, taken in turn. The host fills a slot with
// PIN_EMPTY before it launches the kernel that will write it, and has the status when no word it
// needs is empty any more: no order between the words matters. Word 0 holds est (Arnoldi step) or
// beta, word 1 hn or ||b||, word 2 the flag word with bit 32 the second pass's guard. (PIN_EMPTY is a
// NaN whose payload no arithmetic gives; the kernel writes other NaNs as the default one.)
enum { PIN_BASE = 32, PIN_WORDS = 4, PIN_SLOTS = 4 };
constexpr unsigned long long PIN_EMPTY = 0x7ff4dead0badf00dull;
// misc slots (double[16])
enum { MI_NRM0 = 0, MI_NRM1 = 1, MI_TOL = 2, MI_DONE = 14, MI_GUARD = 15 };

template <typename T, typename S>
__device__ __forceinline__ void load_block_row(const S *base, int64_t pos, int r, T (&v)[4]) {
    load_row(base + pos * BB, r, v);
}

// t -= sum over the update set [p0, p1) of X_ik X_kj (this lane's row of the products).
// L_ik from XL at factor-layout positions (or from A at CSR positions when L_FROM_A),
// X_kj from XU likewise (or A when U_FROM_A).
template <typename T, bool L_FROM_A, bool U_FROM_A>
__device__ __forceinline__ void update_terms(int p0, int p1, int r, const int32_t *__restrict__ pik,
                                             const int32_t *__restrict__ pkj, const int32_t *__restrict__ sik,
                                             const int32_t *__restrict__ skj, const double *__restrict__ A,
                                             const T *XL, const T *XU, T (&t)[4]) {
    for (int q = p0; q < p1; ++q) {
        T l[4], u[4];
        if constexpr (L_FROM_A) load_block_row(A, pik[q], r, l);
        else load_block_row(XL, sik[q], r, l);
        if constexpr (U_FROM_A) load_block_row(A, pkj[q], r, u);
        else load_block_row(XU, skj[q], r, u);
        row_times_block_sub(l, u, t);
    }
}

// Sum over the 64 lanes, in every lane: within rows of 16 lanes by DPP (neighbour, pair, half row,
// row mirrored), then the four rows' sums by readlane. No LDS crossbar: six shuffles of a double
// through it take about four times as long, and a dot product kernel does one per vector and wave.
template <int CTRL>
__device__ __forceinline__ double add_dpp(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)(b & 0xffffffffll), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xF, 0xF, true);
    return v + __longlong_as_double(((long long)hi << 32) | (unsigned long long)(unsigned)lo);
}
__device__ __forceinline__ double wave_sum(double v) {
    v = add_dpp<0xB1>(v);    // quad_perm [1,0,3,2]
    v = add_dpp<0x4E>(v);    // quad_perm [2,3,0,1]
    v = add_dpp<0x141>(v);   // row_half_mirror
    v = add_dpp<0x140>(v);   // row_mirror
    const long long b = __double_as_longlong(v);
    const int lo = (int)(b & 0xffffffffll), hi = (int)(b >> 32);
    auto row = [&](int lane) {
        return __longlong_as_double(((long long)__builtin_amdgcn_readlane(hi, lane) << 32) |
                                    (unsigned long long)(unsigned)__builtin_amdgcn_readlane(lo, lane));
    };
    return (row(0) + row(16)) + (row(32) + row(48));
}

__device__ __forceinline__ bool skipped(const int *guard) { return guard && *guard == 0; }

// Values handed from one workgroup to another inside a launch (partial sums, counts): agent-scope
// accesses go past the L2 of the XCD to the memory all XCDs share, so no L2 write-back or
// invalidation is needed around them.
__device__ __forceinline__ void store_agent(double *p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double load_agent(const double *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// True in the last of `total` workgroups to get here; what the others stored with store_agent
// before is then visible to its load_agent. Each wave waits for its own stores, which have then
// reached the shared memory, before its workgroup counts itself done; the counts are cleared for
// the next launch. A __threadfence in every thread, which writes the whole L2 back, took 10 us over
// 64 workgroups against 2.4 us this way (a grid-wide count and wait, timed alone). GROUPED: more
// than DONE_SINGLE workgroups count in DONE_GROUPS groups and the last of each counts at the
// root, since additions to one address follow each other at about 15 ns (704 in a row: 10 us).
template <bool GROUPED>
__device__ __forceinline__ bool last_workgroup(int *done, int total, int id) {
    __shared__ int last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        auto count = [](int *c, int of) {
            if (of <= 1) return true;
            if (__hip_atomic_fetch_add(c, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != of - 1) return false;
            __hip_atomic_store(c, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return true;
        };
        bool is_last;
        if (GROUPED && total > DONE_SINGLE) {
            const int g = id % DONE_GROUPS;
            is_last = count(done + (1 + g) * DONE_STRIDE, (total - g + DONE_GROUPS - 1) / DONE_GROUPS) &&
                      count(done, DONE_GROUPS);
        } else {
            is_last = count(done, total);
        }
        last = is_last ? 1 : 0;
    }
    __syncthreads();
    return last != 0;
}

// Forward sweep on rows ib, ib + stride, ... (rpq<T>() rows per quad; rows >= n are skipped). The
// right-hand side is rs rhs, and the input vector ys yin where it is double (ys = rs when the input
// is the right-hand side itself, else 1): FGMRES hands over its basis vectors unnormalised.
template <typename T, typename YI, bool EMIT_Z>
__device__ __forceinline__ void fwd_rows(int ib, int stride, int n, const int32_t *__restrict__ lrow,
                                         const int32_t *__restrict__ lcol, const T *__restrict__ Lb,
                                         const double *__restrict__ rhs, const YI *yin, T *yout,
                                         const T *__restrict__ Dinv, T *__restrict__ zout, double rs, double ys) {
    constexpr int RPQ = rpq<T>();
    const int r = threadIdx.x & 3;
    if (ib >= n) return;
    int ii[RPQ], b0[RPQ], b1[RPQ];
    T acc[RPQ];
#pragma unroll
    for (int h = 0; h < RPQ; ++h) {
        ii[h] = ib + h * stride;
        const int i = min(ii[h], n - 1);
        b0[h] = lrow[i];
        b1[h] = (ii[h] < n) ? lrow[i + 1] : b0[h];
        acc[h] = (T)scaled(rhs[(int64_t)i * 4 + r], rs);
    }
    int cnt = 0;
#pragma unroll
    for (int h = 0; h < RPQ; ++h) cnt = max(cnt, b1[h] - b0[h]);
    for (int t0 = 0; t0 < cnt; t0 += 2) {
        int j[RPQ][2];
        T l[RPQ][2][4], yv[RPQ][2];
#pragma unroll
        for (int h = 0; h < RPQ; ++h)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int e = (b1[h] > b0[h]) ? min(b0[h] + t0 + u, b1[h] - 1) : 0;
                j[h][u] = lcol[e];
                load_row(Lb + (int64_t)e * BB, r, l[h][u]);
            }
#pragma unroll
        for (int h = 0; h < RPQ; ++h)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if constexpr (sizeof(YI) == 8) yv[h][u] = (T)scaled(yin[(int64_t)j[h][u] * 4 + r], ys);
                else yv[h][u] = (T)yin[(int64_t)j[h][u] * 4 + r];
            }
#pragma unroll
        for (int h = 0; h < RPQ; ++h)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                T yj[4];
                gather_vec(yv[h][u], yj);
                const T c = dot4(l[h][u][0], yj[0], l[h][u][1], yj[1], l[h][u][2], yj[2], l[h][u][3], yj[3]);
                acc[h] -= (b0[h] + t0 + u < b1[h]) ? c : T(0);
            }
    }
#pragma unroll
    for (int h = 0; h < RPQ; ++h) {
        if (ii[h] < n) {
            yout[(int64_t)ii[h] * 4 + r] = acc[h];
            if constexpr (EMIT_Z) {
                T dr[4], yi[4];
                load_row(Dinv + (int64_t)ii[h] * BB, r, dr);
                gather_vec(acc[h], yi);
                zout[(int64_t)ii[h] * 4 + r] = dot4(dr[0], yi[0], dr[1], yi[1], dr[2], yi[2], dr[3], yi[3]);
            }
        }
    }
}

template <typename T, typename YI, bool EMIT_Z>
__device__ __forceinline__ void fwd_body(int blk, int n, const int32_t *__restrict__ lrow, const int32_t *__restrict__ lcol,
                                            const T *__restrict__ Lb, const double *__restrict__ rhs, const YI *yin,
                                            T *yout, const T *__restrict__ Dinv, T *__restrict__ zout, double rs,
                                            double ys) {
    fwd_rows<T, YI, EMIT_Z>(blk * rows_per_wg2<T>() + (threadIdx.x >> 2), ROWS_PER_WG, n, lrow, lcol, Lb, rhs, yin, yout,
                            Dinv, zout, rs, ys);
}

// Backward sweep on rows ib, ib + stride, ... (rpq<T>() rows per quad). Without OFFDIAG, y is the
// right-hand side, taken times rs.
template <typename T, typename YI, typename ZO, bool OFFDIAG, bool DUAL>
__device__ __forceinline__ void bwd_rows(int ib, int stride, int n, const int32_t *__restrict__ urow,
                                         const int32_t *__restrict__ ucol, const T *__restrict__ Ub,
                                         const T *__restrict__ Dinv, const YI *__restrict__ y, const T *zin, ZO *zout,
                                         T *zout2, double rs = 1.0) {
    constexpr int RPQ = rpq<T>();
    const int r = threadIdx.x & 3;
    if (ib >= n) return;
    int ii[RPQ], b0[RPQ], b1[RPQ];
    T acc[RPQ];
#pragma unroll
    for (int h = 0; h < RPQ; ++h) {
        ii[h] = ib + h * stride;
        const int i = min(ii[h], n - 1);
        if constexpr (OFFDIAG) acc[h] = (T)y[(int64_t)i * 4 + r];
        else acc[h] = (T)scaled(y[(int64_t)i * 4 + r], rs);
        if constexpr (OFFDIAG) {
            b0[h] = urow[i];
            b1[h] = (ii[h] < n) ? urow[i + 1] : b0[h];
        }
    }
    if constexpr (OFFDIAG) {
        int cnt = 0;
#pragma unroll
        for (int h = 0; h < RPQ; ++h) cnt = max(cnt, b1[h] - b0[h]);
        for (int t0 = 0; t0 < cnt; t0 += 2) {
            int j[RPQ][2];
            T u4[RPQ][2][4], zv[RPQ][2];
#pragma unroll
            for (int h = 0; h < RPQ; ++h)
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int e = (b1[h] > b0[h]) ? min(b0[h] + t0 + u, b1[h] - 1) : 0;
                    j[h][u] = ucol[e];
                    load_row(Ub + (int64_t)e * BB, r, u4[h][u]);
                }
#pragma unroll
            for (int h = 0; h < RPQ; ++h)
#pragma unroll
                for (int u = 0; u < 2; ++u) zv[h][u] = zin[(int64_t)j[h][u] * 4 + r];
#pragma unroll
            for (int h = 0; h < RPQ; ++h)
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    T zj[4];
                    gather_vec(zv[h][u], zj);
                    const T c = dot4(u4[h][u][0], zj[0], u4[h][u][1], zj[1], u4[h][u][2], zj[2], u4[h][u][3], zj[3]);
                    acc[h] -= (b0[h] + t0 + u < b1[h]) ? c : T(0);
                }
        }
    }
#pragma unroll
    for (int h = 0; h < RPQ; ++h) {
        if (ii[h] < n) {
            T dr[4], a[4];
            load_row(Dinv + (int64_t)ii[h] * BB, r, dr);
            gather_vec(acc[h], a);
            const T z = dot4(dr[0], a[0], dr[1], a[1], dr[2], a[2], dr[3], a[3]);
            zout[(int64_t)ii[h] * 4 + r] = (ZO)z;
            if constexpr (DUAL) zout2[(int64_t)ii[h] * 4 + r] = z;
        }
    }
}

template <typename T, typename YI, typename ZO, bool OFFDIAG, bool DUAL>
__device__ __forceinline__ void bwd_body(int blk, int n, const int32_t *__restrict__ urow, const int32_t *__restrict__ ucol,
                                            const T *__restrict__ Ub, const T *__restrict__ Dinv,
                                            const YI *__restrict__ y, const T *zin, ZO *zout, T *zout2,
                                            double rs = 1.0) {
    bwd_rows<T, YI, ZO, OFFDIAG, DUAL>(blk * rows_per_wg2<T>() + (threadIdx.x >> 2), ROWS_PER_WG, n, urow, ucol, Ub, Dinv, y,
                                       zin, zout, zout2, rs);
}

// The tile of workgroup b of g (a multiple of 8) when each XCD takes one contiguous eighth of the
// tiles: workgroup b runs on XCD b mod 8.
__device__ __forceinline__ int xcd_tile(int b, int g) { return (b & 7) * (g >> 3) + (b >> 3); }
inline int xcd_grid(int tiles) { return (tiles + 7) / 8 * 8; }

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>)
template <int N, typename F>
__device__ __forceinline__ void unroll(F f) {
    if constexpr (N > 0) {
        unroll<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

// The indices of a row of a pair of sweeps: its first block b0 and its count, the columns j of its
// blocks, the first block c0 and the count nj of each row j, and their columns. A single system's
// pattern keeps all but b0 in a record of 32 bytes (rows of at most two blocks) or 64 (three), eight or
// sixteen per lane of the quad: the words j, then c0 with the count in its low two bits, then the columns
// of each row j, -1 where there is none. Every block and vector is asked for after one load, where the
// walk is two levels (four with the
// columns) deeper. The row's own blocks are asked for between first() and second(), so that the walk
// does not hold them up (server, which keeps no records: 57 us a sweep behind it, 52 so).
template <int CL, bool REC>
struct PairIndex {
    int b0, nl, j[CL], c0[CL], nj[CL], kk[CL][CL];
    __device__ __forceinline__ void first(int i, int r, const int32_t *__restrict__ row,
                                          const int32_t *__restrict__ col, const int32_t *__restrict__ rec) {
        b0 = row[i];
        if constexpr (REC) {
            constexpr int P = PAIR_REC<CL> / 4;   // words per lane
            int w[P];
            if constexpr (P == 2) {
                const int2 v = reinterpret_cast<const int2 *>(rec)[(int64_t)i * 4 + r];
                w[0] = v.x;
                w[1] = v.y;
            } else {
                const int4 v = reinterpret_cast<const int4 *>(rec)[(int64_t)i * 4 + r];
                w[0] = v.x;
                w[1] = v.y;
                w[2] = v.z;
                w[3] = v.w;
            }
            const auto word = [&](auto n) {
                constexpr int N = decltype(n)::value;
                return qb<N / P>(w[N % P]);
            };
            nl = 0;
            unroll<CL>([&](auto u) {
                constexpr int U = decltype(u)::value;
                j[U] = word(std::integral_constant<int, U>{});
                nl += j[U] >= 0;
                const unsigned cn = (unsigned)word(std::integral_constant<int, CL + U>{});
                c0[U] = (int)(cn >> 2);
                nj[U] = (int)(cn & 3);
                unroll<CL>([&](auto v) {
                    constexpr int V = decltype(v)::value;
                    kk[U][V] = word(std::integral_constant<int, 2 * CL + U * CL + V>{});
                });
            });
        } else {
            nl = row[i + 1] - b0;
#pragma unroll
            for (int u = 0; u < CL; ++u)
                if (u < nl) j[u] = col[b0 + u];
        }
    }
    __device__ __forceinline__ void second(const int32_t *__restrict__ row) {
        if constexpr (!REC) {
#pragma unroll
            for (int u = 0; u < CL; ++u) {
                if (u < nl) {
                    c0[u] = row[j[u]];
                    nj[u] = row[j[u] + 1] - c0[u];
                }
            }
        }
    }
};

// Two forward sweeps in one, for rows of at most CL strictly lower blocks: row i of the second sweep
// needs y_j of the first for its lower neighbours j, and forms each again from its own row,
// y_j = r_j - sum_k L_jk yin_k. Same operations on each element, so the bits of two synchronous
// sweeps; as an asynchronous iteration it is the schedule in which no read of the second sweep sees
// a value written in it.
// A small mesh spends a launch and a chain of loads on a sweep, here one launch for both; a large one
// reads L once instead of twice, if the neighbours' rows are still in the L2 of the same XCD, hence
// xcd_tile. Forward and backward together, three sweeps, us: 2,000 triangles 19 -> 11.5 (two launches
// for four); 61,952 FP64 21.2 -> 12.8; 180,000 FP32 29.8 -> 22.2; 500,000 line-ordered quads FP32
// 87.6 -> 73.0 (94.3 without xcd_tile); 4 million triangles FP32 608 -> 477. Of this the records gave,
// on kernels, 2,000 FP32 4 -> 3.1; 180,000 FP32 13.1 + 12.1 -> 12.1 + 10.1; 4 million 253 + 245 ->
// 251 + 227, and with three blocks a side 316 + 305 -> 272 + 233. Two rows per quad at once (95 registers) lose: 180,000 14.7 + 11.1, 4 million 272 + 221.
template <typename T, typename YI, bool EMIT_Z, int CL, bool REC>
__device__ __forceinline__ void fwd_pair_row(int i, int n, const int32_t *__restrict__ lrow,
                                             const int32_t *__restrict__ lcol, const int32_t *__restrict__ rec,
                                             const T *__restrict__ Lb,
                                             const double *__restrict__ rhs, const YI *__restrict__ yin,
                                             T *__restrict__ yout, const T *__restrict__ Dinv, T *__restrict__ zout,
                                             double rs, double ys) {
    const int r = threadIdx.x & 3;
    if (i >= n) return;
    T acc = (T)scaled(rhs[(int64_t)i * 4 + r], rs);
    PairIndex<CL, REC> X;
    X.first(i, r, lrow, lcol, rec);
    const auto &[b0, nl, j, c0, nj, kk] = X;
    T l[CL][4], yj[CL], m[CL][CL][4], yk[CL][CL];
#pragma unroll
    for (int u = 0; u < CL; ++u)
        if (u < nl) load_row(Lb + (int64_t)(b0 + u) * BB, r, l[u]);
    X.second(lrow);
#pragma unroll
    for (int u = 0; u < CL; ++u) {
        if (u < nl) {
            yj[u] = (T)scaled(rhs[(int64_t)j[u] * 4 + r], rs);
        }
    }
    T dr[4];
    if constexpr (EMIT_Z) load_row(Dinv + (int64_t)i * BB, r, dr);
#pragma unroll
    for (int u = 0; u < CL; ++u) {
        if (u < nl) {
#pragma unroll
            for (int v = 0; v < CL; ++v) {
                if (v < nj[u]) {
                    const int k = REC ? kk[u][v] : lcol[c0[u] + v];
                    load_row(Lb + (int64_t)(c0[u] + v) * BB, r, m[u][v]);
                    if constexpr (sizeof(YI) == 8) yk[u][v] = (T)scaled(yin[(int64_t)k * 4 + r], ys);
                    else yk[u][v] = (T)yin[(int64_t)k * 4 + r];
                }
            }
        }
    }
#pragma unroll
    for (int u = 0; u < CL; ++u) {
        if (u < nl) {
#pragma unroll
            for (int v = 0; v < CL; ++v) {
                if (v < nj[u]) {
                    T y[4];
                    gather_vec(yk[u][v], y);
                    yj[u] -= dot4(m[u][v][0], y[0], m[u][v][1], y[1], m[u][v][2], y[2], m[u][v][3], y[3]);
                }
            }
            T y[4];
            gather_vec(yj[u], y);
            acc -= dot4(l[u][0], y[0], l[u][1], y[1], l[u][2], y[2], l[u][3], y[3]);
        }
    }
    yout[(int64_t)i * 4 + r] = acc;
    if constexpr (EMIT_Z) {
        T y[4];
        gather_vec(acc, y);
        zout[(int64_t)i * 4 + r] = dot4(dr[0], y[0], dr[1], y[1], dr[2], y[2], dr[3], y[3]);
    }
}

// Two backward sweeps in one, likewise (rows of at most CU strictly upper blocks):
// z_j = D_j (y_j - sum_k U_jk zin_k) for the upper neighbours j, then z_i from them.
template <typename T, typename ZO, int CU, bool REC>
__device__ __forceinline__ void bwd_pair_row(int i, int n, const int32_t *__restrict__ urow,
                                             const int32_t *__restrict__ ucol, const int32_t *__restrict__ rec,
                                             const T *__restrict__ Ub, const T *__restrict__ Dinv,
                                             const T *__restrict__ y, const T *__restrict__ zin,
                                             ZO *__restrict__ zout) {
    const int r = threadIdx.x & 3;
    if (i >= n) return;
    T acc = y[(int64_t)i * 4 + r];
    PairIndex<CU, REC> X;
    X.first(i, r, urow, ucol, rec);
    const auto &[b0, nu, j, c0, nj, kk] = X;
    T l[CU][4], yj[CU], dj[CU][4], m[CU][CU][4], zk[CU][CU], dr[4];
#pragma unroll
    for (int u = 0; u < CU; ++u)
        if (u < nu) load_row(Ub + (int64_t)(b0 + u) * BB, r, l[u]);
    load_row(Dinv + (int64_t)i * BB, r, dr);
    X.second(urow);
#pragma unroll
    for (int u = 0; u < CU; ++u) {
        if (u < nu) {
            yj[u] = y[(int64_t)j[u] * 4 + r];
            load_row(Dinv + (int64_t)j[u] * BB, r, dj[u]);
        }
    }
#pragma unroll
    for (int u = 0; u < CU; ++u) {
        if (u < nu) {
#pragma unroll
            for (int v = 0; v < CU; ++v) {
                if (v < nj[u]) {
                    const int k = REC ? kk[u][v] : ucol[c0[u] + v];
                    load_row(Ub + (int64_t)(c0[u] + v) * BB, r, m[u][v]);
                    zk[u][v] = zin[(int64_t)k * 4 + r];
                }
            }
        }
    }
#pragma unroll
    for (int u = 0; u < CU; ++u) {
        if (u < nu) {
#pragma unroll
            for (int v = 0; v < CU; ++v) {
                if (v < nj[u]) {
                    T z[4];
                    gather_vec(zk[u][v], z);
                    yj[u] -= dot4(m[u][v][0], z[0], m[u][v][1], z[1], m[u][v][2], z[2], m[u][v][3], z[3]);
                }
            }
            T a[4], z[4];
            gather_vec(yj[u], a);
            const T zj = dot4(dj[u][0], a[0], dj[u][1], a[1], dj[u][2], a[2], dj[u][3], a[3]);
            gather_vec(zj, z);
            acc -= dot4(l[u][0], z[0], l[u][1], z[1], l[u][2], z[2], l[u][3], z[3]);
        }
    }
    T a[4];
    gather_vec(acc, a);
    zout[(int64_t)i * 4 + r] = (ZO)dot4(dr[0], a[0], dr[1], a[1], dr[2], a[2], dr[3], a[3]);
}

template <bool RESID>
__device__ __forceinline__ void spmv_body(int blk, int n, const int32_t *__restrict__ rowptr,
                                             const int32_t *__restrict__ colidx, const double *__restrict__ A,
                                             const double *__restrict__ x, double *__restrict__ y,
                                             const double *__restrict__ b) {
    // eight lanes per block row (SPMV_ROWS rows per workgroup): lane l takes row l / 2, columns
    // 2 (l % 2) and 2 (l % 2) + 1 of every block, so each load instruction covers whole 128-byte
    // FP64 blocks (a quad per row covers half of each block per instruction and reads each line
    // in two passes: 4-5% slower on the 4M-cell matrix)
    constexpr int SCH = 4;
    typedef double d2 __attribute__((ext_vector_type(2)));
    const int i = blk * SPMV_ROWS + (threadIdx.x >> 3);
    const int rr = (threadIdx.x >> 1) & 3, h = threadIdx.x & 1;
    if (i >= n) return;
    const int b0 = rowptr[i], b1 = rowptr[i + 1];
    double acc = 0.0;
    for (int e0 = b0; e0 < b1; e0 += SCH) {
        int j[SCH];
        d2 a[SCH], xv[SCH];
#pragma unroll
        for (int u = 0; u < SCH; ++u) {
            const int e = min(e0 + u, b1 - 1);
            j[u] = colidx[e];
            a[u] = *reinterpret_cast<const d2 *>(A + (int64_t)e * BB + rr * 4 + 2 * h);
        }
#pragma unroll
        for (int u = 0; u < SCH; ++u) xv[u] = *reinterpret_cast<const d2 *>(x + (int64_t)j[u] * 4 + 2 * h);
#pragma unroll
        for (int u = 0; u < SCH; ++u) {
            const double c = a[u].x * xv[u].x + a[u].y * xv[u].y;
            acc += (e0 + u < b1) ? c : 0.0;
        }
    }
    acc += __shfl_xor(acc, 1, 64);   // the row's other two columns, from the neighbouring lane
    if (h == 0) y[(int64_t)i * 4 + rr] = RESID ? b[(int64_t)i * 4 + rr] - acc : acc;
}

// partial[k nb + blk] = sum over the tile of V_k w for k < q, partial[q nb + blk] = that of w^2.
// The vectors are taken four at a time (16 or 32 loads in flight per lane): a system of a few hundred
// tiles leaves each compute unit one workgroup or two, which would otherwise wait for each vector
// in turn.
// VEC_E elements per lane (vec_e); sh: MAX_RESTART + 2 columns of LDS.
// Basis vector k lies at Basis{V0, V, ldv}(k): the first one may lie elsewhere (the right-hand side).
struct Basis {
    const double *V0, *V;
    int64_t ldv;
    __device__ __forceinline__ const double *operator()(int k) const { return k == 0 ? V0 : V + (int64_t)k * ldv; }
};
typedef double WaveSums[WG / 64];
template <int VEC_E>
__device__ __forceinline__ void mdot_body(int blk, int64_t len, const Basis &V, int q,
                                          const double *__restrict__ w, double *__restrict__ partial, int nb,
                                          WaveSums *sh) {
    const int64_t base = (int64_t)blk * (WG * VEC_E) + threadIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double wv[VEC_E];
    const bool full = base + (int64_t)(VEC_E - 1) * WG < len;
#pragma unroll
    for (int e = 0; e < VEC_E; ++e) {
        const int64_t t = base + (int64_t)e * WG;
        wv[e] = (full || t < len) ? w[t] : 0.0;
    }
    auto dots = [&](int k, auto count) {
        constexpr int C = decltype(count)::value;
        double v[C][VEC_E], s[C];
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int e = 0; e < VEC_E; ++e) {
                const int64_t t = base + (int64_t)e * WG;
                v[c][e] = (full || t < len) ? V(k + c)[t] : 0.0;
            }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            s[c] = 0.0;
#pragma unroll
            for (int e = 0; e < VEC_E; ++e) s[c] += v[c][e] * wv[e];
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            s[c] = wave_sum(s[c]);
            if (lane == 0) sh[k + c][wave] = s[c];
        }
    };
    int k = 0;
    for (; k + 4 <= q; k += 4) dots(k, std::integral_constant<int, 4>{});
    for (; k < q; ++k) dots(k, std::integral_constant<int, 1>{});
    double s = 0.0;
#pragma unroll
    for (int e = 0; e < VEC_E; ++e) s += wv[e] * wv[e];
    s = wave_sum(s);
    if (lane == 0) sh[q][wave] = s;
    __syncthreads();
    for (int c = threadIdx.x; c <= q; c += WG)
        store_agent(partial + (int64_t)c * nb + blk, ((sh[c][0] + sh[c][1]) + (sh[c][2] + sh[c][3])));
}

// w += alpha sum_k c[k] V_k over the tile (fresh: w was 0 and is not read); if partial:
// partial[blk] = sum of the new w^2
template <int VEC_E>
__device__ __forceinline__ void update_body(int blk, int64_t len, const Basis &V, int q,
                                               const double *__restrict__ c, double alpha, double *__restrict__ w,
                                               double *__restrict__ partial, const int *guard, bool fresh = false) {
    if (skipped(guard)) return;
    __shared__ double sh[WG / 64];
    const int64_t base = (int64_t)blk * (WG * VEC_E) + threadIdx.x;
    const bool full = base + (int64_t)(VEC_E - 1) * WG < len;
    double acc[VEC_E];
#pragma unroll
    for (int e = 0; e < VEC_E; ++e) {
        const int64_t t = base + (int64_t)e * WG;
        acc[e] = (!fresh && (full || t < len)) ? w[t] : 0.0;
    }
    auto add = [&](int k, auto count) {
        constexpr int C = decltype(count)::value;
        double v[C][VEC_E];
#pragma unroll
        for (int u = 0; u < C; ++u)
#pragma unroll
            for (int e = 0; e < VEC_E; ++e) {
                const int64_t t = base + (int64_t)e * WG;
                v[u][e] = (full || t < len) ? V(k + u)[t] : 0.0;
            }
#pragma unroll
        for (int u = 0; u < C; ++u) {
            const double ck = alpha * c[k + u];
#pragma unroll
            for (int e = 0; e < VEC_E; ++e) acc[e] += ck * v[u][e];
        }
    };
    int k = 0;
    for (; k + 4 <= q; k += 4) add(k, std::integral_constant<int, 4>{});
    for (; k < q; ++k) add(k, std::integral_constant<int, 1>{});
    double s = 0.0;
#pragma unroll
    for (int e = 0; e < VEC_E; ++e) {
        const int64_t t = base + (int64_t)e * WG;
        if (full || t < len) w[t] = acc[e];
        s += acc[e] * acc[e];
    }
    if (partial) {
        s = wave_sum(s);
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
        __syncthreads();
        if (threadIdx.x == 0) store_agent(partial + blk, (sh[0] + sh[1]) + (sh[2] + sh[3]));
    }
}

// The first Gram-Schmidt update and the second pass's dots in one pass over the basis:
// w -= sum_k c[k] V_k, then partial[k nb + blk] = sum over the tile of V_k w (new w), and that of
// w^2 at k = q. Bound by reading the basis once, where update and dots apart read it twice.
// QM >= q vectors of EB elements per lane stay in registers between the two uses (QM EB = 32
// doubles, 64 registers); QM = 0 takes any q and reads each vector again for its dot (the tile's
// second read mostly hits a cache). The sums run in the same order for every QM, so the choice
// does not change a bit. On 4 million cells, FGMRES(50), 8 vectors: update + dots apart 141 + 100 us.
template <int QM, int VEC_E>
__device__ __forceinline__ void update_dot_body(int blk, int64_t len, const Basis &V, int q,
                                                const double *__restrict__ c, double *__restrict__ w,
                                                double *__restrict__ partial, int nb, WaveSums *sh) {
    const int64_t base = (int64_t)blk * (WG * VEC_E) + threadIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool full = base + (int64_t)(VEC_E - 1) * WG < len;
    double sn = 0.0;
    if constexpr (QM > 0) {
        constexpr int EB = 32 / QM < VEC_E ? 32 / QM : VEC_E;
        double s[QM];
#pragma unroll
        for (int k = 0; k < QM; ++k) s[k] = 0.0;
#pragma unroll
        for (int e0 = 0; e0 < VEC_E; e0 += EB) {
            double v[QM][EB], acc[EB];
#pragma unroll
            for (int e = 0; e < EB; ++e) {
                const int64_t t = base + (int64_t)(e0 + e) * WG;
                acc[e] = (full || t < len) ? w[t] : 0.0;
            }
#pragma unroll
            for (int k = 0; k < QM; ++k)
                if (k < q) {
#pragma unroll
                    for (int e = 0; e < EB; ++e) {
                        const int64_t t = base + (int64_t)(e0 + e) * WG;
                        v[k][e] = (full || t < len) ? V(k)[t] : 0.0;
                    }
                }
#pragma unroll
            for (int k = 0; k < QM; ++k)
                if (k < q) {
                    const double ck = -c[k];
#pragma unroll
                    for (int e = 0; e < EB; ++e) acc[e] += ck * v[k][e];
                }
#pragma unroll
            for (int e = 0; e < EB; ++e) {
                const int64_t t = base + (int64_t)(e0 + e) * WG;
                if (full || t < len) w[t] = acc[e];
                sn += acc[e] * acc[e];
            }
#pragma unroll
            for (int k = 0; k < QM; ++k)
                if (k < q) {
#pragma unroll
                    for (int e = 0; e < EB; ++e) s[k] += v[k][e] * acc[e];
                }
        }
#pragma unroll
        for (int k = 0; k < QM; ++k)
            if (k < q) {
                s[k] = wave_sum(s[k]);
                if (lane == 0) sh[k][wave] = s[k];
            }
    } else {
        double acc[VEC_E];
#pragma unroll
        for (int e = 0; e < VEC_E; ++e) {
            const int64_t t = base + (int64_t)e * WG;
            acc[e] = (full || t < len) ? w[t] : 0.0;
        }
        for (int k = 0; k < q; ++k) {
            const double ck = -c[k];
#pragma unroll
            for (int e = 0; e < VEC_E; ++e) {
                const int64_t t = base + (int64_t)e * WG;
                acc[e] += ck * ((full || t < len) ? V(k)[t] : 0.0);
            }
        }
#pragma unroll
        for (int e = 0; e < VEC_E; ++e) {
            const int64_t t = base + (int64_t)e * WG;
            if (full || t < len) w[t] = acc[e];
            sn += acc[e] * acc[e];
        }
        for (int k = 0; k < q; ++k) {
            double s = 0.0;
#pragma unroll
            for (int e = 0; e < VEC_E; ++e) {
                const int64_t t = base + (int64_t)e * WG;
                s += ((full || t < len) ? V(k)[t] : 0.0) * acc[e];
            }
            s = wave_sum(s);
            if (lane == 0) sh[k][wave] = s;
        }
    }
    sn = wave_sum(sn);
    if (lane == 0) sh[q][wave] = sn;
    __syncthreads();
    for (int k = threadIdx.x; k <= q; k += WG)
        store_agent(partial + (int64_t)k * nb + blk, ((sh[k][0] + sh[k][1]) + (sh[k][2] + sh[k][3])));
}

// The register form for q vectors (0: any number).
inline int update_dot_form(int q) { return q <= 4 ? 4 : q <= 8 ? 8 : q <= 16 ? 16 : q <= 32 ? 32 : 0; }

// One column's sum by a whole workgroup; valid in lane 0 of the workgroup.
__device__ __forceinline__ double reduce_col(const double *__restrict__ pc, int nb) {
    __shared__ double sh[WG / 64];
    // eight independent partial sums keep eight loads in flight per lane (fixed order: entry b
    // goes to sum (b / WG) mod 8 while whole groups of 8 WG entries remain, the rest to sum 0)
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0, a4 = 0.0, a5 = 0.0, a6 = 0.0, a7 = 0.0;
    int b = threadIdx.x;
    for (; b + 7 * WG < nb; b += 8 * WG) {
        a0 += pc[b];
        a1 += pc[b + WG];
        a2 += pc[b + 2 * WG];
        a3 += pc[b + 3 * WG];
        a4 += pc[b + 4 * WG];
        a5 += pc[b + 5 * WG];
        a6 += pc[b + 6 * WG];
        a7 += pc[b + 7 * WG];
    }
    for (; b < nb; b += WG) a0 += pc[b];
    double s = ((a0 + a1) + (a2 + a3)) + ((a4 + a5) + (a6 + a7));
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

__device__ __forceinline__ void reduce_cols_body(int blk, const double *__restrict__ partial, int nb,
                                                    double *__restrict__ out, const int *guard) {
    if (skipped(guard)) return;
    const double s = reduce_col(partial + (int64_t)blk * nb, nb);
    if (threadIdx.x == 0) store_agent(out + blk, s);
}

// All `cols` column sums (nb <= FOLD_NB entries each, stored by other workgroups of this launch)
// by one workgroup, a wave per column: lane l of the wave adds the entries that lanes l, l + 64,
// l + 128 and l + 192 of reduce_col's workgroup would add, in the same order, so the sums have the
// same bits. out: LDS, valid for the whole workgroup on return.
constexpr int FOLD_NB = 512;
__device__ __forceinline__ void reduce_cols_fold(const double *partial, int nb, int cols, double *out) {
    constexpr int PER = FOLD_NB / WG;   // rounds of WG entries
    constexpr int CC = 3;               // columns whose loads a wave has in flight together
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int c0 = wave; c0 < cols; c0 += CC * (WG / 64)) {
        double v[CC][PER][WG / 64];
#pragma unroll
        for (int h = 0; h < CC; ++h) {
            const int c = c0 + h * (WG / 64);
#pragma unroll
            for (int r = 0; r < PER; ++r)
#pragma unroll
                for (int p = 0; p < WG / 64; ++p) {
                    const int b = r * WG + p * 64 + lane;
                    v[h][r][p] = c < cols && b < nb ? load_agent(partial + (int64_t)c * nb + b) : 0.0;
                }
        }
#pragma unroll
        for (int h = 0; h < CC; ++h) {
            const int c = c0 + h * (WG / 64);
            if (c < cols) {
                double s[WG / 64];
#pragma unroll
                for (int p = 0; p < WG / 64; ++p) {
                    s[p] = 0.0;
#pragma unroll
                    for (int r = 0; r < PER; ++r) s[p] += v[h][r][p];
                }
#pragma unroll
                for (int p = 0; p < WG / 64; ++p) s[p] = wave_sum(s[p]);
                if (lane == 0) out[c] = (s[0] + s[1]) + (s[2] + s[3]);
            }
        }
    }
    __syncthreads();
}

// Normalisation. The basis vectors stay as the Gram-Schmidt passes leave them, u_k; v_k = s_k u_k
// with s_k = 1 / ||u_k|| in vscale[k] (norms are at least 1e-162, a square root of a sum of squares,
// so s_k is finite; a zero norm leaves s_k = 1). The dots come as u_k . w and the coefficients are
// taken on u_k, each times s_k, and the preconditioner multiplies its input by s_k where it reads
// it. A pass that read u_k and wrote v_k took 40 us of 1,690 per iteration at 4 million cells.

// ---- steps on the small dense Hessenberg problem (column-major, ld = m + 1), run by one workgroup
// on the column sums `red` of the reduction before them (in LDS). Columns and rotations are taken one
// per lane; only the chain of rotations and the substitution are serial. What a step reads of earlier
// launches' results every workgroup loads before its reduction ends (StepIn): by the workgroup that
// turns out to be the last, no load is waited for between the sums and the status. (One lane taking
// everything from memory spent 8-12 us on six Arnoldi vectors. With the loads after the sums the
// Givens step's launch took 8.8 us at 10,000 cells and 5.8 at 180,000, with them before 7.4 and 4.9.)
enum { RS_BETA_START_ZERO = 0, RS_BETA_START_X, RS_BETA, RS_GS1, RS_GS2, RS_GIVENS, RS_NONE };

struct KPtrs {
    double *partials, *red, *H, *cs, *sn, *g, *coef, *misc, *status, *vscale;
    int *guard, *done;
    bool grouped;   // done has the counts of the groups too
    // a single solve only (host null in the server)
    unsigned long long *host = nullptr;   // the slot that this launch's status goes to
    const unsigned *flags = nullptr;
    double rtol = 0.0;
    bool single = false, last = false;    // last: no Arnoldi step follows this one
};

// Lane q has entry q of the vectors (q <= k < MAX_RESTART = WG).
static_assert(MAX_RESTART <= WG, "a lane per Arnoldi vector");
struct StepIn {
    double scale, h, cs, sn;      // of vector / rotation q
    double gk, nrm, tol, num;
    unsigned flags;
    int guard;
    template <int OP>
    __device__ __forceinline__ void load(const KPtrs &P, int k, int m) {
        const int q = threadIdx.x;
        if (OP == RS_GS1 || OP == RS_GS2) scale = q <= k ? P.vscale[q] : 0.0;
        if (OP == RS_GS2 || OP == RS_GIVENS) h = q <= k ? P.H[(int64_t)k * (m + 1) + q] : 0.0;
        if (OP == RS_GS2) nrm = P.misc[MI_NRM0];
        if (OP == RS_GIVENS) {
            cs = q < k ? P.cs[q] : 0.0;
            sn = q < k ? P.sn[q] : 0.0;
            guard = *P.guard;
            gk = P.g[k];
            nrm = P.misc[MI_NRM1];
            tol = P.misc[MI_TOL];
        }
        if (OP == RS_BETA) num = P.status[ST_NUM];
        if (P.host) flags = *P.flags;
    }
};

// Hand the status to the host (one lane): three writes through to its pinned memory.
__device__ __forceinline__ void publish(const KPtrs &P, double v0, double v1, unsigned flags, int guard) {
    if (!P.host) return;
    auto put = [&](int w, unsigned long long v) {
        __hip_atomic_store(P.host + w, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    };
    auto bits = [](double v) {
        return v == v ? (unsigned long long)__double_as_longlong(v) : 0x7ff8000000000000ull;
    };
    put(2, (unsigned long long)flags | (guard ? 1ull << 32 : 0ull));
    put(0, bits(v0));
    put(1, bits(v1));
}

__device__ __forceinline__ double lane_value(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
}

// Back substitution on the k x k upper triangle: coef = y, by columns (one workgroup). Up to 64
// unknowns stay in the lanes of one wave, and eight columns are loaded at a time (of eight
// unknowns: a launch of 4.2 us, and of 9.0 with a load and two barriers per column).
__device__ __forceinline__ void solve_body(int k, int m, const double *H, const double *g, double *coef) {
    if (k <= 64) {
        const int t = threadIdx.x;
        if (t >= 64) return;
        constexpr int E = 8;
        double y = t < k ? g[t] : 0.0;
        for (int q0 = k - 1; q0 >= 0; q0 -= E) {
            double h[E];
#pragma unroll
            for (int e = 0; e < E; ++e) h[e] = t <= q0 - e ? H[(int64_t)(q0 - e) * (m + 1) + t] : 0.0;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int q = q0 - e;
                if (q < 0) break;
                const double yq = lane_value(y, q) / lane_value(h[e], q);
                if (t < q) y -= h[e] * yq;
                else if (t == q) y = yq;
            }
        }
        if (t < k) coef[t] = y;
        return;
    }
    __shared__ double y[MAX_RESTART];
    for (int t = threadIdx.x; t < k; t += blockDim.x) y[t] = g[t];
    __syncthreads();
    for (int q = k - 1; q >= 0; --q) {
        const double *h = H + (int64_t)q * (m + 1);
        const double yq = y[q] / h[q];
        __syncthreads();
        for (int t = threadIdx.x; t <= q; t += blockDim.x) {
            if (t < q) y[t] -= h[t] * yq;
            else coef[q] = yq;
        }
        __syncthreads();
    }
}

__device__ __forceinline__ void beta_step(const KPtrs &P, const StepIn &I, int m, double r0, bool num, bool beta_slot,
                                          bool init_g) {
    const double beta = sqrt(r0);
    if (threadIdx.x == 0) {
        if (beta_slot) publish(P, beta, num ? beta : I.num, I.flags, 0);
        if (num) {
            P.status[ST_NUM] = beta;
            P.misc[MI_TOL] = P.rtol * (beta > 0 ? beta : 1.0);
        }
        if (beta_slot) P.status[ST_BETA] = beta;
        P.vscale[0] = beta != 0.0 ? 1.0 / beta : 1.0;
    }
    if (init_g)
        for (int q = threadIdx.x; q <= m + 1; q += blockDim.x) P.g[q] = q == 0 ? beta : 0.0;
}

// H(0:k,k) = v_k . w, coef those on u_k, nrm0 = ||w|| before the first pass
__device__ __forceinline__ void gs1_step(const KPtrs &P, const StepIn &I, int k, int m, const double *red) {
    const int q = threadIdx.x;
    if (q <= k) {
        const double h = I.scale * red[q];
        P.H[(int64_t)k * (m + 1) + q] = h;
        P.coef[q] = I.scale * h;
    }
    if (q == 0) P.misc[MI_NRM0] = sqrt(red[k + 1]);
}

// after the first update (red: the second pass's dots and ||w'||^2): a second pass if
// ||w'|| < ||w|| / sqrt(2); then H(0:k,k) += dots, coef likewise
__device__ __forceinline__ void gs2_step(const KPtrs &P, const StepIn &I, int k, int m, const double *red) {
    const int q = threadIdx.x;
    const double n1 = sqrt(red[k + 1]);
    const int again = n1 < 0.70710678118654752440 * I.nrm ? 1 : 0;
    if (q == 0) {
        P.misc[MI_NRM1] = n1;
        *P.guard = again;
    }
    if (!again || q > k) return;
    const double h = I.scale * red[q];
    P.H[(int64_t)k * (m + 1) + q] = I.h + h;
    P.coef[q] = I.scale * h;
}

// final norm, Givens rotations, residual estimate
__device__ __forceinline__ void givens_step(const KPtrs &P, const StepIn &I, int k, int m, const double *red) {
    __shared__ double lh[MAX_RESTART + 1], lc[MAX_RESTART], ls[MAX_RESTART], end[2];
    double *h = P.H + (int64_t)k * (m + 1);
    const int q = threadIdx.x;
    if (q <= k) lh[q] = I.h;
    if (q < k) {
        lc[q] = I.cs;
        ls[q] = I.sn;
    }
    __syncthreads();
    if (q == 0) {
        const double hn = I.guard ? sqrt(red[0]) : I.nrm;
        double a = lh[0];
        for (int e = 0; e < k; ++e) {
            const double b = lh[e + 1];
            lh[e] = lc[e] * a + ls[e] * b;
            a = -ls[e] * a + lc[e] * b;
        }
        const double rho = sqrt(a * a + hn * hn);
        const double c = rho > 0 ? a / rho : 1.0, sn = rho > 0 ? hn / rho : 0.0;
        const double est = fabs(-sn * I.gk);
        publish(P, est, hn, I.flags, I.guard);
        lh[k] = rho;
        P.cs[k] = c;
        P.sn[k] = sn;
        P.g[k + 1] = -sn * I.gk;
        P.g[k] = c * I.gk;
        P.vscale[k + 1] = hn != 0.0 ? 1.0 / hn : 1.0;
        P.status[ST_EST] = est;
        P.status[ST_HN] = hn;
        P.status[ST_GUARD] = (double)I.guard;
        end[0] = est;
        end[1] = hn;
    }
    __syncthreads();
    if (q <= k) h[q] = lh[q];
    if (q == 0) h[k + 1] = 0.0;
    // where the cycle ends, its least-squares solution (the host takes the same decision)
    if (P.single && (P.last || end[0] <= I.tol || end[1] == 0.0)) {
        __syncthreads();
        solve_body(k + 1, m, P.H, P.g, P.coef);
    }
}

// The step OP on the column sums red (whole workgroup; red readable by every lane).
template <int OP>
__device__ __forceinline__ void step_tail(const KPtrs &P, const StepIn &I, int k, int m, const double *red) {
    if constexpr (OP == RS_BETA_START_ZERO || OP == RS_BETA_START_X) {
        beta_step(P, I, m, red[0], true, OP == RS_BETA_START_ZERO, OP == RS_BETA_START_ZERO);
    }
    else if constexpr (OP == RS_BETA) beta_step(P, I, m, red[0], false, true, true);
    else if constexpr (OP == RS_GS1) gs1_step(P, I, k, m, red);
    else if constexpr (OP == RS_GS2) gs2_step(P, I, k, m, red);
    else if constexpr (OP == RS_GIVENS) givens_step(P, I, k, m, red);
}

// Column blk's sum, then step OP in the last of the `cols` workgroups to finish. The step runs also
// when the guard skipped the reduction (the Givens step needs it either way).
template <int OP>
__device__ __forceinline__ void reduce_step_body(int blk, int cols, const KPtrs &P, int nb, const int *guard, int k,
                                                 int m) {
    __shared__ double sred[MAX_RESTART + 2];
    StepIn in;
    in.load<OP>(P, k, m);
    reduce_cols_body(blk, P.partials, nb, P.red, guard);
    if (!last_workgroup<false>(P.done, cols, blk)) return;
    for (int c = threadIdx.x; c < cols; c += WG) sred[c] = load_agent(P.red + c);
    __syncthreads();
    step_tail<OP>(P, in, k, m, sred);
}

__device__ __forceinline__ void zero_body(int blk, int64_t len, double *v) {
    const int64_t tile = vec_tile(len), t0 = blk * tile, t1 = min(len, t0 + tile);
    for (int64_t t = t0 + threadIdx.x; t < t1; t += WG) v[t] = 0.0;
}

template <typename T, typename S, bool SRC_CSR, bool COPY>
__device__ __forceinline__ void factor_init_body(int blk, int n, int ZL, const int32_t *__restrict__ rowptr,
                                                    const int32_t *__restrict__ diag_pos,
                                                    const int32_t *__restrict__ lrow,
                                                    const int32_t *__restrict__ urow, const S *X0, T *Xout, T *D0,
                                                    unsigned *flags) {
    const int i = blk * ROWS_PER_WG + (threadIdx.x >> 2);
    const int r = threadIdx.x & 3;
    if (i >= n) return;
    if constexpr (COPY) {
        static_assert(SRC_CSR, "copy reads A");
        const int b0 = rowptr[i], d = diag_pos[i], b1 = rowptr[i + 1];
        const int lb = lrow[i], ub = urow[i];
        for (int e = b0; e < b1; ++e) {
            T v[4];
            load_row(X0 + (int64_t)e * BB, r, v);
            store_row(Xout + (int64_t)split_pos(e, i, b0, d, lb, ub, ZL, n) * BB, r, v);
        }
    }
    const int64_t dpos = SRC_CSR ? (int64_t)diag_pos[i] : (int64_t)ZL + i;
    T u[4], out[4];
    load_row(X0 + dpos * BB, r, u);
    bool ok = inv4_row(u, r, out);
    store_row(D0 + (int64_t)i * BB, r, out);
    if (!ok && r == 0) atomicOr(flags, ABILU_FLAG_MODIFIED);
}

// One sweep over block row i (a quad of 4 lanes). The strictly lower blocks are loaded in chunks
// of CHL (their A blocks and inverses fetched together) and computed and stored one at a time in
// ascending column order, so a block whose update set holds an earlier block of the row reads that
// block's value from this sweep when the sweep works in place (the strict Gauss-Seidel order within
// the row). This also keeps the first in-place sweep from A from reading the output buffer before
// this sweep has written it: there X_ik of the row is never taken from the initial guess.
// D_FROM_A (first sweep from the initial guess X0 = A): the inverses U_jj^{-1} = A_jj^{-1} the
// lower blocks need are formed here from A, in the same arithmetic as the initialisation kernel,
// so no separate pass writes and re-reads them. A row whose A_ii no other row inverts this way
// inverts it once itself, only to raise the flag the initialisation would raise when that inverse
// is replaced: with sym (structurally symmetric pattern) those are the rows without strictly upper
// blocks, otherwise every row checks its own.
template <typename T, bool L_FROM_A, bool U_FROM_A, int CHL = CH, bool D_FROM_A = false>
__device__ __forceinline__ void factor_sweep_row(int i,
    int n, int ZL, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
    const int32_t *__restrict__ diag_pos, const int32_t *__restrict__ lrow, const int32_t *__restrict__ urow,
    const int32_t *__restrict__ pair_ptr, const int32_t *__restrict__ pik, const int32_t *__restrict__ pkj,
    const int32_t *__restrict__ sik, const int32_t *__restrict__ skj, const double *__restrict__ A, const T *XL,
    const T *XU, const T *Dp, T *Xn, T *Dn, unsigned *flags, bool sym = false) {
    const int r = threadIdx.x & 3;
    if (i >= n) return;
    const int b0 = rowptr[i], b1 = rowptr[i + 1], d = diag_pos[i];
    const int lbase = lrow[i], ubase = urow[i];
    // update-set extents: lower blocks [pb0, pd), diagonal [pd, pd1), upper [pd1, pb1)
    const int pb0 = pair_ptr[b0], pd = pair_ptr[d], pd1 = pair_ptr[d + 1], pb1 = pair_ptr[b1];
    T *XnL = Xn + (int64_t)lbase * BB;
    T *XnU = Xn + ((int64_t)ZL + n + ubase) * BB;
    unsigned fl = 0;

    // strictly lower blocks: L_ij = (A_ij - sum) U_jj^{-1}
    for (int e0 = b0; e0 < d; e0 += CHL) {
        T t[CHL][4], dr[CHL][4];
        int j[CHL];
#pragma unroll
        for (int u = 0; u < CHL; ++u) {
            const int e = min(e0 + u, d - 1);
            load_row(A + (int64_t)e * BB, r, t[u]);
            j[u] = colidx[e];
        }
        if constexpr (D_FROM_A) {
#pragma unroll
            for (int u = 0; u < CHL; ++u) {
                T a[4];
                load_row(A + (int64_t)diag_pos[j[u]] * BB, r, a);
                if (!inv4_row(a, r, dr[u])) fl |= ABILU_FLAG_MODIFIED;
            }
        } else {
#pragma unroll
            for (int u = 0; u < CHL; ++u) load_row(Dp + (int64_t)j[u] * BB, r, dr[u]);
        }
#pragma unroll
        for (int u = 0; u < CHL; ++u) {
            if (e0 + u < d) {
                if (pd > pb0)
                    update_terms<T, L_FROM_A, U_FROM_A>(pair_ptr[e0 + u], pair_ptr[e0 + u + 1], r, pik, pkj, sik,
                                                        skj, A, XL, XU, t[u]);
                T x[4];
                row_times_block(t[u], dr[u], x);
                fl |= nonfinite4(x);
                store_row(XnL + (int64_t)(e0 + u - b0) * BB, r, x);
            }
        }
    }
    // diagonal block U_ii = A_ii - sum, and its inverse
    {
        T t[4];
        load_row(A + (int64_t)d * BB, r, t);
        if constexpr (D_FROM_A) {
            if ((!sym || d + 1 == b1) && !surely_invertible(t, r)) {
                T unused[4];
                if (!inv4_row(t, r, unused)) fl |= ABILU_FLAG_MODIFIED;
            }
        }
        update_terms<T, L_FROM_A, U_FROM_A>(pd, pd1, r, pik, pkj, sik, skj, A, XL, XU, t);
        fl |= nonfinite4(t);
        store_row(Xn + ((int64_t)ZL + i) * BB, r, t);
        T out[4];
        if (!inv4_row(t, r, out)) fl |= ABILU_FLAG_MODIFIED;
        store_row(Dn + (int64_t)i * BB, r, out);
    }
    // strictly upper blocks: U_ij = A_ij - sum
    for (int e0 = d + 1; e0 < b1; e0 += CH) {
        T t[CH][4];
#pragma unroll
        for (int u = 0; u < CH; ++u) load_row(A + (int64_t)min(e0 + u, b1 - 1) * BB, r, t[u]);
        if (pb1 > pd1) {
#pragma unroll
            for (int u = 0; u < CH; ++u)
                if (e0 + u < b1)
                    update_terms<T, L_FROM_A, U_FROM_A>(pair_ptr[e0 + u], pair_ptr[e0 + u + 1], r, pik, pkj, sik,
                                                        skj, A, XL, XU, t[u]);
        }
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            if (e0 + u < b1) {
                fl |= nonfinite4(t[u]);
                store_row(XnU + (int64_t)(e0 + u - d - 1) * BB, r, t[u]);
            }
        }
    }
    if (fl) atomicOr(flags, fl);
}

// One synchronous sweep over block g of the factor layout (any pattern): a quad per block instead of
// per row. A row's sweep takes its blocks, and their update pairs, one after the other; here a row of
// seven blocks is seven quads, and the layout's order (lower, diagonal, upper) keeps the quads of a
// wave alike, so that upper blocks run no inverses (in CSR order: 51 us where this takes 38). The same
// operations on each element. An XCD takes the same eighth of the rows of all three kinds, in slabs of
// about 1,024 rows, so that the blocks its pairs read are in its L2 (without: 41 us).
// Bound by the chain record -> pair -> blocks below about 100,000 cells, by the pairs' reads beyond.
// Triangles and quadrilaterals mixed, two sweeps, us: 2,500 cells FP64 29.6 -> 11; 30,523 FP64 49 -> 38,
// FP32 42 -> 27; 1,300,000 FP64 1,913 -> 1,723, FP32 1,378 -> 1,245.
struct BlockPattern {
    int n, ZL, Z;
    const int4 *brec;                // per block of the factor layout: CSR position, pair range, ldiag
    int slabs, tl, td, tu;           // of an eighth: slabs, and their tiles of lower, diagonal, upper blocks
    int grid() const { return 8 * slabs * (tl + td + tu); }
    // the block of workgroup b's quad q, or -1
    __device__ __forceinline__ int block(int b, int q) const {
        const int per = tl + td + tu, s = (b & 7) * slabs + (b >> 3) / per, w = (b >> 3) % per;
        int64_t g = q;
        int hi;
        if (w < tl) {
            g += ((int64_t)s * tl + w) * ROWS_PER_WG;
            hi = ZL;
        } else if (w < tl + td) {
            g += ZL + ((int64_t)s * td + (w - tl)) * ROWS_PER_WG;
            hi = ZL + n;
        } else {
            g += ZL + n + ((int64_t)s * tu + (w - tl - td)) * ROWS_PER_WG;
            hi = Z;
        }
        return g < hi ? (int)g : -1;
    }
    const int32_t *lcol, *ik, *kj;   // ik, kj: CSR positions (from A) or factor-layout ones
};
template <typename T, bool FROM_A>
__device__ __forceinline__ void factor_sweep_block(int g, const BlockPattern &P, const double *__restrict__ A,
                                                   const T *__restrict__ XP, const T *__restrict__ Dp,
                                                   T *__restrict__ Xn, T *__restrict__ Dn, unsigned *flags) {
    const int r = threadIdx.x & 3;
    if (g < 0) return;
    const int4 rec = P.brec[g];
    const bool lower = g < P.ZL, diag = !lower && g < P.ZL + P.n;
    const int p0 = rec.y, p1 = rec.z;
    T t[4], v[4];
    load_row(A + (int64_t)rec.x * BB, r, t);
    if (lower) {
        if constexpr (FROM_A) load_row(A + (int64_t)rec.w * BB, r, v);
        else load_row(Dp + (int64_t)P.lcol[g] * BB, r, v);
    }
    unsigned fl = 0;
    // the initial inverse of a diagonal block that no lower block uses raises its flag here
    if (FROM_A && diag && !surely_invertible(t, r)) {
        T unused[4];
        if (!inv4_row(t, r, unused)) fl |= ABILU_FLAG_MODIFIED;
    }
    for (int q = p0; q < p1; q += 2) {
        const int q1 = min(q + 1, p1 - 1);
        const int a0 = P.ik[q], c0 = P.kj[q], a1 = P.ik[q1], c1 = P.kj[q1];
        T l0[4], u0[4], l1[4], u1[4];
        if constexpr (FROM_A) {
            load_block_row(A, a0, r, l0);
            load_block_row(A, c0, r, u0);
            load_block_row(A, a1, r, l1);
            load_block_row(A, c1, r, u1);
        } else {
            load_block_row(XP, a0, r, l0);
            load_block_row(XP, c0, r, u0);
            load_block_row(XP, a1, r, l1);
            load_block_row(XP, c1, r, u1);
        }
        row_times_block_sub(l0, u0, t);
        if (q + 1 < p1) row_times_block_sub(l1, u1, t);
    }
    if (lower) {
        T D[4], x[4];
        if constexpr (FROM_A) {
            if (!inv4_row(v, r, D)) fl |= ABILU_FLAG_MODIFIED;
            row_times_block(t, D, x);
        } else {
            row_times_block(t, v, x);
        }
        fl |= nonfinite4(x);
        store_row(Xn + (int64_t)g * BB, r, x);
    } else {
        fl |= nonfinite4(t);
        store_row(Xn + (int64_t)g * BB, r, t);
        if (diag) {
            T out[4];
            if (!inv4_row(t, r, out)) fl |= ABILU_FLAG_MODIFIED;
            store_row(Dn + (int64_t)(g - P.ZL) * BB, r, out);
        }
    }
    if (fl) atomicOr(flags, fl);
}

// One sweep over block row i of a pattern whose update sets are those of the diagonal blocks alone:
// structurally symmetric and free of triples of mutual neighbours (P = ZL: a mesh of triangles or
// quads without corner links), with at most CL strictly lower and CU strictly upper blocks a row.
// Then pair u of the row is its lower block u with the block (k, i) of column k, entry lrow[i] + u of
// the pair lists, and U_ij = A_ij above the diagonal.
// Bound by latency in factor_sweep_row, whose chain of dependent loads is about twelve long (row
// pointers, columns, diagonal positions, pairs, blocks, the row's own L_ik read back, one block or
// pair after the other). Here the loads form three levels: row pointers; the row's blocks and index
// entries; the gathered blocks. The arithmetic on every block, and its order, is that of
// factor_sweep_row.
//   LSRC  where L_ik of the diagonal update comes from: A (first synchronous sweep), the previous
//         iterate XP, or this sweep (in place)
//   FROM_A  first sweep from X0 = A: U_kj and the inverses U_jj^{-1} come from A
enum { L_FROM_A0 = 0, L_FROM_PREV = 1, L_FROM_NEW = 2 };
struct FvPattern {
    int n, ZL;
    const int32_t *rowptr, *lrow, *urow, *lcol, *ldiag, *pkj, *skj;
};
template <typename T, int LSRC, bool FROM_A, int CL, int CU>
__device__ __forceinline__ void factor_sweep_fv_row(int i, const FvPattern &P, const double *__restrict__ A,
                                                    const T *XP, const T *Dp, T *Xn, T *Dn, unsigned *flags) {
    const int r = threadIdx.x & 3;
    if (i >= P.n) return;
    const int b0 = P.rowptr[i], b1 = P.rowptr[i + 1], lb = P.lrow[i], nl = P.lrow[i + 1] - lb, ub = P.urow[i];
    const int d = b0 + nl, nu = b1 - d - 1;
    // the row's blocks and index entries (unused slots read the diagonal block's)
    int jd[CL], jc[CL], pk[CL];
    using LV = typename std::conditional<FROM_A, double, T>::type;
    double aL[CL][4], aD[4], aU[CU][4];
    T xl[LSRC == L_FROM_PREV ? CL : 1][4];
#pragma unroll
    for (int u = 0; u < CL; ++u) {
        const int e = lb + min(u, max(nl - 1, 0));
        if constexpr (FROM_A) {
            const int q = P.ldiag[e], k = P.pkj[e];
            jd[u] = u < nl ? q : d;
            pk[u] = u < nl ? k : d;
        } else {
            const int q = P.lcol[e], k = P.skj[e];
            jc[u] = u < nl ? q : i;
            pk[u] = u < nl ? k : P.ZL + i;
        }
    }
#pragma unroll
    for (int u = 0; u < CL; ++u) load_row(A + (int64_t)(b0 + min(u, nl)) * BB, r, aL[u]);
    load_row(A + (int64_t)d * BB, r, aD);
    if constexpr (LSRC == L_FROM_PREV) {
#pragma unroll
        for (int u = 0; u < CL; ++u) load_row(XP + (int64_t)(u < nl ? lb + u : P.ZL + i) * BB, r, xl[u]);
    }
    // the gathered blocks: U_kk^{-1} (or A_kk, to be inverted) and U_ki
    LV dj[CL][4], uk[CL][4];
#pragma unroll
    for (int u = 0; u < CL; ++u) {
        if constexpr (FROM_A) {
            load_row(A + (int64_t)jd[u] * BB, r, dj[u]);
            load_row(A + (int64_t)pk[u] * BB, r, uk[u]);
        } else {
            load_row(Dp + (int64_t)jc[u] * BB, r, dj[u]);
            load_row(XP + (int64_t)pk[u] * BB, r, uk[u]);
        }
    }
#pragma unroll
    for (int w = 0; w < CU; ++w) load_row(A + (int64_t)(d + min(w + 1, nu)) * BB, r, aU[w]);
    unsigned fl = 0;
    T t[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) t[c] = (T)aD[c];
    // a row without upper blocks has its A_ii inverted by no other row: raise the flag here
    if (FROM_A && nu == 0 && !surely_invertible(t, r)) {
        T unused[4];
        if (!inv4_row(t, r, unused)) fl |= ABILU_FLAG_MODIFIED;
    }
#pragma unroll
    for (int u = 0; u < CL; ++u) {
        if (u < nl) {
            T a[4], D[4], v[4], x[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                a[c] = (T)aL[u][c];
                D[c] = (T)dj[u][c];
                v[c] = (T)uk[u][c];
            }
            if constexpr (FROM_A) {
                T Di[4];
                if (!inv4_row(D, r, Di)) fl |= ABILU_FLAG_MODIFIED;
                row_times_block(a, Di, x);
            } else {
                row_times_block(a, D, x);
            }
            fl |= nonfinite4(x);
            store_row(Xn + (int64_t)(lb + u) * BB, r, x);
            if constexpr (LSRC == L_FROM_A0) row_times_block_sub(a, v, t);
            else if constexpr (LSRC == L_FROM_PREV) row_times_block_sub(xl[u], v, t);
            else row_times_block_sub(x, v, t);
        }
    }
    fl |= nonfinite4(t);
    store_row(Xn + ((int64_t)P.ZL + i) * BB, r, t);
    T out[4];
    if (!inv4_row(t, r, out)) fl |= ABILU_FLAG_MODIFIED;
    store_row(Dn + (int64_t)i * BB, r, out);
#pragma unroll
    for (int w = 0; w < CU; ++w) {
        if (w < nu) {
            T v[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = (T)aU[w][c];
            fl |= nonfinite4(v);
            store_row(Xn + ((int64_t)P.ZL + P.n + ub + w) * BB, r, v);
        }
    }
    if (fl) atomicOr(flags, fl);
}

// t -= sum over the update set [p0, p1) of X_ik X_kj for a row of a chunk (chunked sweeps).
// X_ik is a block of this row and comes from Xn (this sweep). X_kj lies in the strictly upper part
// of row k < i: rows of the chunk (factor-layout position >= ubound) come from Xn, earlier rows
// from XO, or from A at CSR positions when OUT_FROM_A (the first sweep from X0 = A). PAIR2 takes
// the pairs two at a time (clamped index loads, then the four block rows) so that a row's chain of
// dependent loads is short, at the cost of registers; either way the products are subtracted in
// the list's order, so both forms give the same values.
template <typename T, bool OUT_FROM_A>
__device__ __forceinline__ void load_u_chunk(int q, int sp, int ubound, int r, const int32_t *__restrict__ pkj,
                                             const double *__restrict__ A, const T *Xn, const T *XO, T (&u)[4]) {
    if (sp >= ubound) load_block_row(Xn, sp, r, u);
    else if constexpr (OUT_FROM_A) load_block_row(A, pkj[q], r, u);
    else load_block_row(XO, sp, r, u);
}

template <typename T, bool OUT_FROM_A, bool PAIR2>
__device__ __forceinline__ void update_terms_chunk(int p0, int p1, int r, int ubound, const int32_t *__restrict__ pkj,
                                                   const int32_t *__restrict__ sik, const int32_t *__restrict__ skj,
                                                   const double *__restrict__ A, const T *Xn, const T *XO,
                                                   T (&t)[4]) {
    if constexpr (PAIR2) {
        for (int q0 = p0; q0 < p1; q0 += 2) {
            const int qb = min(q0 + 1, p1 - 1);
            const int sa = sik[q0], sb = sik[qb];
            const int ka = skj[q0], kb = skj[qb];
            T la[4], lb[4], ua[4], ub[4];
            load_block_row(Xn, sa, r, la);
            load_block_row(Xn, sb, r, lb);
            load_u_chunk<T, OUT_FROM_A>(q0, ka, ubound, r, pkj, A, Xn, XO, ua);
            load_u_chunk<T, OUT_FROM_A>(qb, kb, ubound, r, pkj, A, Xn, XO, ub);
            row_times_block_sub(la, ua, t);
            if (q0 + 1 < p1) row_times_block_sub(lb, ub, t);
        }
    } else {
        for (int q = p0; q < p1; ++q) {
            T l[4], u[4];
            load_block_row(Xn, sik[q], r, l);
            load_u_chunk<T, OUT_FROM_A>(q, skj[q], ubound, r, pkj, A, Xn, XO, u);
            row_times_block_sub(l, u, t);
        }
    }
}

// One chunked sweep over block row i of the chunk starting at row c0: the blocks of the row in
// ascending column order, each stored before the next is computed (a Gauss-Seidel order within
// the row), reading the chunk's rows from this sweep (Xn, Dn) and earlier rows from XO, DO.
template <typename T, bool OUT_FROM_A, bool PAIR2>
__device__ __forceinline__ void factor_chunk_row(int i, int c0, int ubound,
    int n, int ZL, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
    const int32_t *__restrict__ diag_pos, const int32_t *__restrict__ lrow, const int32_t *__restrict__ urow,
    const int32_t *__restrict__ pair_ptr, const int32_t *__restrict__ pkj, const int32_t *__restrict__ sik,
    const int32_t *__restrict__ skj, const double *__restrict__ A, const T *XO, const T *DO, T *Xn, T *Dn,
    unsigned *flags) {
    const int r = threadIdx.x & 3;
    const int b0 = rowptr[i], b1 = rowptr[i + 1], d = diag_pos[i];
    T *XnL = Xn + (int64_t)lrow[i] * BB;
    T *XnU = Xn + ((int64_t)ZL + n + urow[i]) * BB;
    unsigned fl = 0;
    // strictly lower blocks: L_ij = (A_ij - sum) U_jj^{-1}, U_jj^{-1} of this sweep if j is in the
    // chunk. With PAIR2 and no update terms in the row's lower part the blocks are independent and
    // are computed two at a time; otherwise one at a time, each seeing the ones before it.
    if (PAIR2 && pair_ptr[d] == pair_ptr[b0]) {
        for (int e0 = b0; e0 < d; e0 += 2) {
            const int eb = min(e0 + 1, d - 1);
            T ta[4], tb[4], da[4], db[4];
            load_row(A + (int64_t)e0 * BB, r, ta);
            load_row(A + (int64_t)eb * BB, r, tb);
            const int ja = colidx[e0], jb = colidx[eb];
            load_row((ja >= c0 ? (const T *)Dn : DO) + (int64_t)ja * BB, r, da);
            load_row((jb >= c0 ? (const T *)Dn : DO) + (int64_t)jb * BB, r, db);
            T xa[4], xb[4];
            row_times_block(ta, da, xa);
            row_times_block(tb, db, xb);
            fl |= nonfinite4(xa);
            store_row(XnL + (int64_t)(e0 - b0) * BB, r, xa);
            if (e0 + 1 < d) {
                fl |= nonfinite4(xb);
                store_row(XnL + (int64_t)(e0 + 1 - b0) * BB, r, xb);
            }
        }
    } else {
        for (int e = b0; e < d; ++e) {
            T t[4], dr[4];
            load_row(A + (int64_t)e * BB, r, t);
            const int j = colidx[e];
            load_row((j >= c0 ? (const T *)Dn : DO) + (int64_t)j * BB, r, dr);
            update_terms_chunk<T, OUT_FROM_A, PAIR2>(pair_ptr[e], pair_ptr[e + 1], r, ubound, pkj, sik, skj, A, Xn, XO, t);
            T x[4];
            row_times_block(t, dr, x);
            fl |= nonfinite4(x);
            store_row(XnL + (int64_t)(e - b0) * BB, r, x);
        }
    }
    // diagonal block U_ii = A_ii - sum and its inverse
    {
        T t[4];
        load_row(A + (int64_t)d * BB, r, t);
        update_terms_chunk<T, OUT_FROM_A, PAIR2>(pair_ptr[d], pair_ptr[d + 1], r, ubound, pkj, sik, skj, A, Xn, XO, t);
        fl |= nonfinite4(t);
        store_row(Xn + ((int64_t)ZL + i) * BB, r, t);
        T out[4];
        if (!inv4_row_gathered(t, r, out)) fl |= ABILU_FLAG_MODIFIED;
        store_row(Dn + (int64_t)i * BB, r, out);
    }
    // strictly upper blocks: U_ij = A_ij - sum (independent of each other)
    for (int e0 = d + 1; e0 < b1; e0 += CH) {
        T t[CH][4];
#pragma unroll
        for (int u = 0; u < CH; ++u) load_row(A + (int64_t)min(e0 + u, b1 - 1) * BB, r, t[u]);
#pragma unroll
        for (int u = 0; u < CH; ++u)
            if (e0 + u < b1)
                update_terms_chunk<T, OUT_FROM_A, PAIR2>(pair_ptr[e0 + u], pair_ptr[e0 + u + 1], r, ubound, pkj, sik, skj,
                                                  A, Xn, XO, t[u]);
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            if (e0 + u < b1) {
                fl |= nonfinite4(t[u]);
                store_row(XnU + (int64_t)(e0 + u - d - 1) * BB, r, t[u]);
            }
        }
    }
    if (fl) atomicOr(flags, fl);
}

template <typename T, bool L_FROM_A, bool U_FROM_A, bool D_FROM_A = false>
__device__ __forceinline__ void factor_sweep_body(int blk,
    int n, int ZL, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
    const int32_t *__restrict__ diag_pos, const int32_t *__restrict__ lrow, const int32_t *__restrict__ urow,
    const int32_t *__restrict__ pair_ptr, const int32_t *__restrict__ pik, const int32_t *__restrict__ pkj,
    const int32_t *__restrict__ sik, const int32_t *__restrict__ skj, const double *__restrict__ A, const T *XL,
    const T *XU, const T *Dp, T *Xn, T *Dn, unsigned *flags, bool sym = false) {
    factor_sweep_row<T, L_FROM_A, U_FROM_A, CH, D_FROM_A>(blk * ROWS_PER_WG + (threadIdx.x >> 2), n, ZL, rowptr, colidx, diag_pos,
                                            lrow, urow, pair_ptr, pik, pkj, sik, skj, A, XL, XU, Dp, Xn, Dn, flags, sym);
}

// ------------------------------------------------------------------ per-row records of the
// quad-per-chunk runner (layout beside REC_INTS)

// Records are stored as REC_INTS / 4 planes of int4 (plane k holds fields 4k .. 4k + 3 of every
// record), each plane step-major: the record of row c * R + t at index t * nch + c. The quads of a
// wavefront run chunks c, c + 1, ... in lock step, so a load of one plane reads adjacent 16-byte
// pieces, and a sweep that needs only some fields reads only their planes.
__device__ __forceinline__ int4 rec_quad(const int32_t *__restrict__ rec, int R, int c, int nch, int t, int k) {
    return reinterpret_cast<const int4 *>(rec)[(int64_t)k * R * nch + (int64_t)t * nch + c];
}

__device__ __forceinline__ void load_rec(const int32_t *__restrict__ rec, int R, int c, int nch, int t, int4 (&rc)[6]) {
#pragma unroll
    for (int k = 0; k < 6; ++k) rc[k] = rec_quad(rec, R, c, nch, t, k);
}

template <int K>
__device__ __forceinline__ int rec_field(const int4 (&rc)[6]) {
    if constexpr ((K & 3) == 0) return rc[K >> 2].x;
    else if constexpr ((K & 3) == 1) return rc[K >> 2].y;
    else if constexpr ((K & 3) == 2) return rc[K >> 2].z;
    else return rc[K >> 2].w;
}

// v = rows[k] for a runtime k < N, as a masked blend of the bit patterns: the rows stay in
// registers (a chain of selects between the rows would be folded into a load at a computed offset,
// which forces the rows into scratch memory)
template <typename T, int N>
__device__ __forceinline__ void pick_row(const T (&rows)[N][4], int k, T (&v)[4]) {
    using U = typename std::conditional<sizeof(T) == 4, uint32_t, uint64_t>::type;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        U x = 0;
#pragma unroll
        for (int q = 0; q < N; ++q) x |= ((U)0 - (U)(k == q)) & __builtin_bit_cast(U, rows[q][c]);
        v[c] = __builtin_bit_cast(T, x);
    }
}

template <typename T>
__device__ __forceinline__ void copy_row(const T (&a)[4], T (&b)[4]) {
#pragma unroll
    for (int c = 0; c < 4; ++c) b[c] = a[c];
}

}  // namespace abilu_k
