// Pattern analysis on the device: validation, diagonal positions and the update sets
// K(i,j) = { k < min(i,j) : (i,k), (k,j) in S_B } of the block ILU(0) equations (Section 4.2,
// equation bilu), stored as CSR lists of block-position pairs ascending in k.
#include <algorithm>
#include <climits>
#include <cstring>
#include <new>

#include "setup_kernels.h"

namespace {

using namespace abilu_setup;

// also clears the words of k_pat_tri_counts, the one of k_pat_sym and the completion counts
__global__ void k_pat_rows(int n, int64_t Z, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
                           int32_t *__restrict__ diag_pos, unsigned *__restrict__ err, unsigned *__restrict__ more,
                           unsigned *__restrict__ unsym, int32_t *__restrict__ done) {
    if (blockIdx.x == 0) {
        if (threadIdx.x < 4) more[threadIdx.x] = 0;
        if (threadIdx.x == 0) *unsym = 0;
        for (int t = threadIdx.x; t < DONE_INTS; t += blockDim.x) done[t] = 0;
    }
    pat_rows_body(blockIdx.x, n, Z, rowptr, colidx, diag_pos, err);
}

__global__ __launch_bounds__(PAT_ROWS) void k_pat_count(int n, const int32_t *__restrict__ rowptr,
                                                         const int32_t *__restrict__ colidx,
                                                         const int32_t *__restrict__ diag_pos,
                                                         int64_t *__restrict__ cnt) {
    pat_count_body(blockIdx.x, n, rowptr, colidx, diag_pos, cnt);
}

__global__ __launch_bounds__(PAT_ROWS) void k_pat_fill(int n, int ZL, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
                           const int32_t *__restrict__ diag_pos, const int32_t *__restrict__ lrow,
                           const int32_t *__restrict__ urow, const int64_t *__restrict__ ptr,
                           int32_t *__restrict__ pik, int32_t *__restrict__ pkj, int32_t *__restrict__ sik,
                           int32_t *__restrict__ skj) {
    pat_fill_body(blockIdx.x, n, ZL, rowptr, colidx, diag_pos, lrow, urow, ptr, pik, pkj, sik, skj);
}

// also pat_side_body, and over a sample of 64 workgroups at most a tally of lower blocks: all of them, those
// farther than PAIR_NEAR rows and those farther than PAIR_NEAR3, in 21 bits each (TALLY_*; at most 64 of a
// row) of the 64-bit word at more + 2. One addition a workgroup: additions to one address follow each other
// at 15 ns, and three of every wave of 256 workgroups took 45 us.
constexpr int TALLY_FAR = 21, TALLY_FAR3 = 42, TALLY_ROW = 64;
constexpr unsigned long long TALLY_MASK = (1ull << 21) - 1;
__global__ __launch_bounds__(256) void k_pat_tri_counts(int n, const int32_t *__restrict__ rowptr,
                                                        const int32_t *__restrict__ colidx,
                                                        const int32_t *__restrict__ diag_pos, int64_t *__restrict__ nl,
                                                        int64_t *__restrict__ nu, unsigned *more) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    pat_tri_counts_body(blockIdx.x, n, rowptr, diag_pos, nl, nu);
    pat_side_body(i, n, rowptr, diag_pos, more);
    if (n <= PAIR_NEAR3 || blockIdx.x % (gridDim.x / 64 + 1) != 0) return;
    __shared__ unsigned long long sh[4];
    unsigned long long tally = 0;
    if (i < n) {
        const int b0 = rowptr[i], b1 = min(diag_pos[i], b0 + TALLY_ROW);
        for (int e = b0; e < b1; ++e) {
            const int away = i - colidx[e];
            tally += 1ull + ((unsigned long long)(away > PAIR_NEAR) << TALLY_FAR) +
                     ((unsigned long long)(away > PAIR_NEAR3) << TALLY_FAR3);
        }
    }
    for (int o = 32; o > 0; o >>= 1) tally += __shfl_xor(tally, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = tally;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd((unsigned long long *)(more + 2), (sh[0] + sh[1]) + (sh[2] + sh[3]));
}

__global__ void k_pat_tri_cols(int n, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
                               const int32_t *__restrict__ diag_pos, const int32_t *__restrict__ lrow,
                               const int32_t *__restrict__ urow, int32_t *__restrict__ lcol,
                               int32_t *__restrict__ ldiag, int32_t *__restrict__ ucol, int ZL, int ZU) {
    pat_tri_cols_body(blockIdx.x, n, rowptr, colidx, diag_pos, lrow, urow, lcol, ldiag, ucol);
    if (blockIdx.x == 0 && threadIdx.x == 0) {   // the padding entry behind each
        lcol[ZL] = 0;
        ldiag[ZL] = 0;
        ucol[ZU] = 0;
    }
}

__global__ void k_pat_sym(int n, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
                          const int32_t *__restrict__ diag_pos, unsigned *__restrict__ unsym) {
    pat_sym_body(blockIdx.x, n, rowptr, colidx, diag_pos, unsym);
}

template <int S>
__global__ void k_pat_pairs(int n, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colidx,
                            const int32_t *__restrict__ diag_pos, const int32_t *__restrict__ lrow,
                            const int32_t *__restrict__ urow, int32_t *__restrict__ lrec, int32_t *__restrict__ urec) {
    pat_pairs_body<S>(blockIdx.x, blockDim.x, threadIdx.x, n, rowptr, colidx, diag_pos, lrow, urow, lrec, urec);
}

// What a synchronous factor sweep needs of each block, in one load.
__global__ void k_pat_blocks(int n, int ZL, const int32_t *__restrict__ rowptr, const int32_t *__restrict__ diag_pos,
                             const int32_t *__restrict__ lrow, const int32_t *__restrict__ urow,
                             const int32_t *__restrict__ pair_ptr, const int32_t *__restrict__ ldiag,
                             int4 *__restrict__ brec) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int b0 = rowptr[i], d = diag_pos[i], b1 = rowptr[i + 1];
    for (int e = b0; e < b1; ++e) {
        const int g = (int)split_pos(e, i, b0, d, lrow[i], urow[i], ZL, n);
        brec[g] = make_int4(e, pair_ptr[e], pair_ptr[e + 1], e < d ? ldiag[g] : 0);
    }
}

// abilu_build_pattern's scratch kept as storage of records: where they start, and up to which size (beyond,
// an allocation of the records' own size holds a fifth to a third less memory).
constexpr size_t REC_AT = 256, KEEP_SCRATCH = (size_t)64 << 20;

// Device arrays of a pattern. Those of 2 MiB and more, which cost the runtime 12 us each to allocate and
// 12 to free, share one allocation; smaller ones come from its pool in under 1 us each.
constexpr size_t LARGE_INTS = (size_t)2 << 18;
struct Piece {
    int32_t **p;
    size_t ints;
};
hipError_t allocate(abilu_pattern *p, std::initializer_list<Piece> pieces) {
    const auto up = [](size_t ints) { return (ints + 63) / 64 * 64; };   // 256-byte boundaries
    size_t large = 0;
    for (const Piece &q : pieces) large += q.ints >= LARGE_INTS ? up(q.ints) : 0;
    const auto get = [&](size_t ints, int32_t **out) {
        if (p->nowned >= (int)(sizeof(p->owned) / sizeof(p->owned[0]))) return hipErrorOutOfMemory;
        const hipError_t e = hipMalloc(out, sizeof(int32_t) * ints);
        if (e == hipSuccess) p->owned[p->nowned++] = *out;
        return e;
    };
    int32_t *next = nullptr;
    if (large)
        if (const hipError_t e = get(large, &next); e != hipSuccess) return e;
    for (const Piece &q : pieces) {
        if (q.ints >= LARGE_INTS) {
            *q.p = next;
            next += up(q.ints);
        } else if (q.ints) {
            if (const hipError_t e = get(q.ints, q.p); e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

void free_pattern(abilu_pattern *p) {
    if (!p) return;
    for (int q = 0; q < p->nowned; ++q) (void)hipFree(p->owned[q]);
    abilu::free_chunks(p);
    if (p->pinned) (void)hipHostFree(p->pinned);
    delete p;
}

}  // namespace

namespace abilu {

// the four words of k_pat_tri_counts, behind the last pair offset (without rows, the last two lie in the
// scans' scratch behind it)
static unsigned *shape_words(void *scratch, int32_t n, int64_t Z) {
    return (unsigned *)(pat_scratch(scratch, n, Z).ptr64 + Z + 1);
}

// the word of k_pat_sym, beside the error word in the scratch's header
static unsigned *unsym_word(void *scratch) { return (unsigned *)scratch + 1; }

size_t pattern_scratch_bytes(int32_t n, int64_t Z) {
    const int64_t len = Z + n + 2;
    return 256 + sizeof(int64_t) * (size_t)(2 * len + scan_tiles(Z > n ? Z : n) + 1);
}

// Non-blocking stage 1a: validation and diagonal positions; the error word (nonzero: invalid
// pattern) is copied to h_err when the stream reaches it. Clears the completion counts `done`.
abilu_status pattern_validate_async(int32_t n, int64_t Z, const int32_t *rowptr, const int32_t *colidx,
                                    int32_t *diag_pos, int32_t *done, void *scratch, unsigned *h_err, hipStream_t s) {
    unsigned *err = (unsigned *)scratch;
    if (!hip_ok(hipMemsetAsync(err, 0, sizeof(unsigned), s), "pattern error clear")) return ABILU_EDEVICE;
    k_pat_rows<<<max(1, div_up(n, 256)), 256, 0, s>>>(n, Z, rowptr, colidx, diag_pos, err, shape_words(scratch, n, Z),
                                                      unsym_word(scratch), done);
    if (launch_status() != ABILU_OK) return ABILU_EDEVICE;
    if (!hip_ok(hipMemcpyAsync(h_err, err, sizeof(unsigned), hipMemcpyDeviceToHost, s), "pattern error readback"))
        return ABILU_EDEVICE;
    return ABILU_OK;
}

// Non-blocking stage 1b (valid patterns only): lower/upper row offsets and the update-set
// offsets (pair_ptr); h_sizes receives ZL, ZU, the number of pairs and the four words of
// k_pat_tri_counts. ptr64 in the scratch
// keeps the int64 pair offsets for pattern_fill.
abilu_status pattern_count_async(int32_t n, int64_t Z, const int32_t *rowptr, const int32_t *colidx,
                                 const int32_t *diag_pos, int32_t *lrow, int32_t *urow, int32_t *pair_ptr,
                                 void *scratch, int64_t *h_sizes, hipStream_t s) {
    const PatScratch S = pat_scratch(scratch, n, Z);
    int64_t *cnt = S.cnt, *ptr64 = S.ptr64, *tot = S.tot;
#define CK(x)                                              \
    do {                                                   \
        if (!hip_ok((x), #x)) return ABILU_EDEVICE;        \
    } while (0)
    if (n > 0) {
        k_pat_tri_counts<<<div_up(n, 256), 256, 0, s>>>(n, rowptr, colidx, diag_pos, cnt, cnt + (n + 1),
                                                        shape_words(scratch, n, Z));
        CK(hipGetLastError());
    }
    for (int part = 0; part < 2; ++part) {
        CK(scan_exclusive(n, cnt + (part == 0 ? 0 : (n + 1)), tot, ptr64, part == 0 ? lrow : urow, s));
        CK(hipMemcpyAsync(h_sizes + part, ptr64 + n, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    }
    if (n > 0) {
        k_pat_count<<<div_up(n, PAT_ROWS), PAT_ROWS, 0, s>>>(n, rowptr, colidx, diag_pos, cnt);
        CK(hipGetLastError());
    }
    CK(scan_exclusive(Z, cnt, tot, ptr64, pair_ptr, s));
    CK(hipMemcpyAsync(h_sizes + 2, ptr64 + Z, 3 * sizeof(int64_t), hipMemcpyDeviceToHost, s));
    return ABILU_OK;
#undef CK
}

bool pattern_sizes_ok(int32_t n, int64_t Z, const int64_t *sizes) {
    return sizes[0] >= 0 && sizes[1] >= 0 && sizes[0] + sizes[1] + n == Z && sizes[2] >= 0 &&
           sizes[2] <= (int64_t)INT_MAX;
}

// Blocking stage 1 (two stream syncs).
abilu_status pattern_count(int32_t n, int64_t Z, const int32_t *rowptr, const int32_t *colidx, int32_t *diag_pos,
                           int32_t *lrow, int32_t *urow, int32_t *pair_ptr, int32_t *done, void *scratch,
                           int64_t *h_pinned, hipStream_t s, int64_t *ZL, int64_t *ZU, int64_t *npairs, int32_t *side, bool *local,
                           bool *near) {
    abilu_status st = pattern_validate_async(n, Z, rowptr, colidx, diag_pos, done, scratch, (unsigned *)h_pinned, s);
    if (st != ABILU_OK) return st;
    if (!hip_ok(hipStreamSynchronize(s), "pattern validation sync")) return ABILU_EDEVICE;
    if (*(const unsigned *)h_pinned) return ABILU_EPATTERN;
    st = pattern_count_async(n, Z, rowptr, colidx, diag_pos, lrow, urow, pair_ptr, scratch, h_pinned, s);
    if (st != ABILU_OK) return st;
    if (!hip_ok(hipStreamSynchronize(s), "pattern count sync")) return ABILU_EDEVICE;
    *ZL = h_pinned[0];
    *ZU = h_pinned[1];
    *npairs = h_pinned[2];
    const unsigned *words = (const unsigned *)(h_pinned + 3);
    *side = side_class(words);
    const unsigned long long tally = (unsigned long long)h_pinned[4], all = tally & TALLY_MASK;
    *local = n <= PAIR_NEAR || 4 * ((tally >> TALLY_FAR) & TALLY_MASK) <= all;
    *near = n <= PAIR_NEAR3 || 4 * (tally >> TALLY_FAR3) <= all;
    return pattern_sizes_ok(n, Z, h_pinned) ? ABILU_OK : ABILU_EPATTERN;
}

// Columns of the lower/upper parts and the update-set lists (non-blocking; the scratch must
// still hold what pattern_count left there).
abilu_status pattern_fill(int32_t n, int64_t Z, int64_t ZL, int64_t ZU, int64_t npairs, const int32_t *rowptr,
                          const int32_t *colidx, const int32_t *diag_pos, const int32_t *lrow, const int32_t *urow,
                          int32_t *lcol, int32_t *ldiag, int32_t *ucol, int32_t *pik, int32_t *pkj, int32_t *sik,
                          int32_t *skj, const void *scratch, hipStream_t s) {
    const int64_t *ptr64 = pat_scratch(const_cast<void *>(scratch), n, Z).ptr64;
    k_pat_tri_cols<<<max(1, div_up(n, 256)), 256, 0, s>>>(n, rowptr, colidx, diag_pos, lrow, urow, lcol, ldiag, ucol,
                                                          (int)ZL, (int)ZU);
    if (launch_status() != ABILU_OK) return ABILU_EDEVICE;
    if (n > 0 && npairs > 0) {
        k_pat_fill<<<div_up(n, PAT_ROWS), PAT_ROWS, 0, s>>>(n, (int)ZL, rowptr, colidx, diag_pos, lrow, urow, ptr64, pik, pkj,
                                                   sik, skj);
        if (launch_status() != ABILU_OK) return ABILU_EDEVICE;
    }
    return ABILU_OK;
}

}  // namespace abilu

extern "C" abilu_status abilu_build_pattern(int32_t nbrows, const int32_t *d_rowptr,
                                            const int32_t *d_colidx, int32_t bs, void *stream,
                                            abilu_pattern **out) {
    using namespace abilu;
    if (!out) return ABILU_EINVAL;
    *out = nullptr;
    if (bs != 4 || nbrows < 0 || nbrows == INT32_MAX || !d_rowptr) return ABILU_EINVAL;   // N + 1 fits int32
    hipStream_t s = (hipStream_t)stream;
    const int n = nbrows;

    abilu_pattern *p = new (std::nothrow) abilu_pattern();
    if (!p) return ABILU_ENOMEM;
    void *scratch = nullptr;   // until the pattern keeps it
    size_t scratch_bytes = 0;
    // The scratch has served when the records are written: up to KEEP_SCRATCH the first of them that fit
    // take its place behind the header, instead of an allocation more (12 us, and 12 to free) and a free.
    auto keep_scratch = [&](size_t bytes) -> void * {
        if (!scratch || scratch_bytes > KEEP_SCRATCH || REC_AT + bytes > scratch_bytes) return nullptr;
        void *at = (char *)scratch + REC_AT;
        p->owned[p->nowned++] = scratch;
        scratch = nullptr;
        return at;
    };
    abilu_status st = ABILU_OK;
    int32_t ends[2] = {0, 0};
    int64_t ZL = 0, ZU = 0, npairs = 0;
#define CK(x)                                  \
    do {                                       \
        if (!hip_ok((x), #x)) {                \
            st = ABILU_EDEVICE;                \
            goto fail;                         \
        }                                      \
    } while (0)
#define CKA(x)                                 \
    do {                                       \
        if (!hip_ok((x), #x)) {                \
            st = ABILU_ENOMEM;                 \
            goto fail;                         \
        }                                      \
    } while (0)
    {
        CK(hipGetDevice(&p->device));
        p->n = n;
        CK(hipMemcpyAsync(&ends[0], d_rowptr, sizeof(int32_t), hipMemcpyDeviceToHost, s));
        CK(hipMemcpyAsync(&ends[1], d_rowptr + n, sizeof(int32_t), hipMemcpyDeviceToHost, s));
        CK(hipStreamSynchronize(s));
        if (ends[0] != 0 || ends[1] < n) { st = ABILU_EPATTERN; goto fail; }
        const int64_t Z = ends[1];
        if (Z > 0 && !d_colidx) { st = ABILU_EINVAL; goto fail; }
        p->nnzb = Z;
        CKA(hipHostMalloc((void **)&p->pinned, 64 * sizeof(double), hipHostMallocDefault));
        CK(hipHostGetDevicePointer((void **)&p->pinned_dev, p->pinned, 0));
        for (int q = 0; q < 64; ++q) p->pinned[q] = 0.0;
        const size_t lrow_ints = ((size_t)n + 1 + DONE_STRIDE - 1) / DONE_STRIDE * DONE_STRIDE;
        CKA(allocate(p, {{&p->rowptr, (size_t)n + 1}, {&p->colidx, (size_t)Z + 1}, {&p->diag_pos, (size_t)n + 1},
                         {&p->pair_ptr, (size_t)Z + 1}, {&p->lrow, lrow_ints + DONE_INTS}, {&p->urow, (size_t)n + 1}}));
        p->done = p->lrow + lrow_ints;
        scratch_bytes = pattern_scratch_bytes(n, Z);
        // room for the records of pairs of rows of two blocks a side, or of three where there are that many
        const size_t rec_room = REC_AT + (Z > 5 * (int64_t)n ? 128 : 64) * (size_t)n;
        if (rec_room <= KEEP_SCRATCH) scratch_bytes = std::max(scratch_bytes, rec_room);
        CKA(hipMalloc(&scratch, scratch_bytes));
        void *const work = scratch;
        unsigned *const unsym = unsym_word(scratch);
        CK(hipMemcpyAsync(p->rowptr, d_rowptr, sizeof(int32_t) * (n + 1), hipMemcpyDeviceToDevice, s));
        if (Z > 0) CK(hipMemcpyAsync(p->colidx, d_colidx, sizeof(int32_t) * Z, hipMemcpyDeviceToDevice, s));
        st = pattern_count(n, Z, p->rowptr, p->colidx, p->diag_pos, p->lrow, p->urow, p->pair_ptr, p->done, scratch,
                           (int64_t *)p->pinned, s, &ZL, &ZU, &npairs, &p->side, &p->local, &p->near);
        if (st != ABILU_OK) goto fail;
        p->nnzb_lower = ZL;
        p->nnzb_upper = ZU;
        p->npairs = npairs;
        p->local = p->local && pair_records_hold(n, ZL, ZU);
        const size_t np = (size_t)npairs + 1;
        const size_t recs = (!p->local || p->side > 3 ? 0 : p->side <= 2 ? PAIR_REC<2> : PAIR_REC<3>) * (size_t)n;
        // where both kinds of records are needed, the block form's in the allocation of the large arrays, if
        // there is one (else by itself while kernels run)
        const size_t both = recs && (npairs != ZL || p->side > 3) && np >= LARGE_INTS ? 4 * (size_t)Z : 0;
        CKA(allocate(p, {{&p->lcol, 2 * ((size_t)ZL + 1)}, {&p->ucol, (size_t)ZU + 1}, {&p->pik, np}, {&p->pkj, np},
                         {&p->sik, np}, {&p->skj, np}, {(int32_t **)&p->brec, both}}));
        if (recs) {
            if (int32_t *at = (int32_t *)keep_scratch(8 * recs)) {
                p->lrec = at;
                p->urec = at + recs;
            } else {
                CKA(allocate(p, {{&p->lrec, recs}, {&p->urec, recs}}));
            }
        }
        p->ldiag = p->lcol + (ZL + 1);
        st = pattern_fill(n, Z, ZL, ZU, npairs, p->rowptr, p->colidx, p->diag_pos, p->lrow, p->urow, p->lcol,
                          p->ldiag, p->ucol, p->pik, p->pkj, p->sik, p->skj, work, s);
        if (st != ABILU_OK) goto fail;
        // structural symmetry (the factor sweeps choose their form by it); the records of pairs and of
        // blocks, which need not wait for it, in the same wait of the host
        {
            auto blocks = [&]() -> abilu_status {
                if (!p->brec) p->brec = (int4 *)keep_scratch(16 * (size_t)Z);
                if (!p->brec && !hip_ok(allocate(p, {{(int32_t **)&p->brec, 4 * (size_t)Z}}), "block records"))
                    return ABILU_ENOMEM;
                k_pat_blocks<<<div_up(n, 256), 256, 0, s>>>(n, (int)ZL, p->rowptr, p->diag_pos, p->lrow, p->urow,
                                                            p->pair_ptr, p->ldiag, p->brec);
                return launch_status();
            };
            if (n > 0) {
                k_pat_sym<<<div_up(n, 256), 256, 0, s>>>(n, p->rowptr, p->colidx, p->diag_pos, unsym);
                CK(hipGetLastError());
            }
            CK(hipMemcpyAsync(p->pinned, unsym, sizeof(unsigned), hipMemcpyDeviceToHost, s));
            p->symmetric = true;   // until the host knows
            if (recs) {
                auto records = [&](auto size) {
                    k_pat_pairs<decltype(size)::value><<<div_up(2 * (int64_t)n, 256), 256, 0, s>>>(
                        n, p->rowptr, p->colidx, p->diag_pos, p->lrow, p->urow, p->lrec, p->urec);
                };
                if (p->side <= 2) records(std::integral_constant<int, 2>{});
                else records(std::integral_constant<int, 3>{});
                CK(hipGetLastError());
            }
            if (n > 0 && !p->fv() && (st = blocks()) != ABILU_OK) goto fail;
            CK(hipStreamSynchronize(s));
            p->symmetric = *(const unsigned *)p->pinned == 0;
            if (n > 0 && !p->fv() && !p->brec) {   // as many pairs as lower blocks, and not symmetric
                if ((st = blocks()) != ABILU_OK) goto fail;
                CK(hipStreamSynchronize(s));
            }
        }
    }
    (void)hipFree(scratch);
    *out = p;
    return ABILU_OK;
fail:
    (void)hipStreamSynchronize(s);
    (void)hipFree(scratch);
    free_pattern(p);
    return st;
#undef CK
#undef CKA
}

extern "C" abilu_status abilu_pattern_destroy(abilu_pattern *p) {
    free_pattern(p);
    return ABILU_OK;
}

extern "C" abilu_status abilu_pattern_info(const abilu_pattern *p, int32_t *nbrows, int64_t *nnzb,
                                           int64_t *npairs, int32_t *depth_D, int32_t *levels_lower,
                                           int32_t *levels_upper) {
    if (!p) return ABILU_EINVAL;
    if (nbrows) *nbrows = p->n;
    if (nnzb) *nnzb = p->nnzb;
    if (npairs) *npairs = p->npairs;
    if (depth_D) *depth_D = p->depth_D;
    if (levels_lower) *levels_lower = p->levels[0];
    if (levels_upper) *levels_upper = p->levels[1];
    return ABILU_OK;
}

extern "C" abilu_status abilu_pattern_export(const abilu_pattern *p, int32_t *d_diag_pos,
                                             int32_t *d_pair_ptr, int32_t *d_pik, int32_t *d_pkj,
                                             void *stream) {
    if (!p) return ABILU_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    hipError_t e = hipSuccess;
    if (d_diag_pos && p->n > 0)
        e = hipMemcpyAsync(d_diag_pos, p->diag_pos, sizeof(int32_t) * p->n, hipMemcpyDeviceToDevice, s);
    if (e == hipSuccess && d_pair_ptr)
        e = hipMemcpyAsync(d_pair_ptr, p->pair_ptr, sizeof(int32_t) * (p->nnzb + 1), hipMemcpyDeviceToDevice, s);
    if (e == hipSuccess && d_pik && p->npairs > 0)
        e = hipMemcpyAsync(d_pik, p->pik, sizeof(int32_t) * p->npairs, hipMemcpyDeviceToDevice, s);
    if (e == hipSuccess && d_pkj && p->npairs > 0)
        e = hipMemcpyAsync(d_pkj, p->pkj, sizeof(int32_t) * p->npairs, hipMemcpyDeviceToDevice, s);
    return abilu::hip_ok(e, "pattern export copy") ? ABILU_OK : ABILU_EDEVICE;
}
