// Host evaluation of the pattern analysis's index arithmetic near its limits, on sparse arrays (pages
// of anonymous memory that are never touched take no room). Prints one line; exit status 0 when all hold.
#include <sys/mman.h>
#include <unistd.h>

#include <cstdio>

#include "setup_kernels.h"

using namespace abilu_setup;

template <typename T>
static T *sparse(int64_t count) {
    void *p = mmap(nullptr, (size_t)count * sizeof(T), PROT_READ | PROT_WRITE,
                   MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (p == MAP_FAILED) {
        perror("mmap");
        _exit(2);
    }
    return (T *)p;
}

static int failures = 0;
static void expect(bool ok, const char *what) {
    if (!ok) {
        printf("FAILED: %s\n", what);
        ++failures;
    }
}

int main() {
    // a row of six blocks whose positions lie on either side of 2^30 and near 2^31
    for (int64_t first : {(int64_t)(1 << 30) - 3, (int64_t)INT32_MAX - 8}) {
        int32_t *colidx = sparse<int32_t>((int64_t)INT32_MAX + 1), rowptr[4] = {0, 0, (int32_t)first, (int32_t)first + 6};
        int32_t diag[3] = {0, 0, (int32_t)first + 1};
        const int32_t cols[6] = {1, 2, 9, 11, 40, 70};
        for (int q = 0; q < 6; ++q) colidx[first + q] = cols[q];
        for (int q = 0; q < 6; ++q) {
            expect(find_col(rowptr, colidx, 2, cols[q]) == first + q, "find_col");
            if (q > 1) expect(find_upper(rowptr, colidx, diag, 2, cols[q]) == first + q, "find_upper");
        }
        expect(find_col(rowptr, colidx, 2, 10) == -1, "find_col of an absent column");
        munmap(colidx, ((size_t)INT32_MAX + 1) * sizeof(int32_t));
    }

    // records of the last rows of a pattern of 2^30 + 100 rows: row i is coupled to i - 1 alone
    const int n = (1 << 30) + 100, i = n - 1, d = 1000;
    int32_t *rowptr = sparse<int32_t>((int64_t)n + 1), *diag = sparse<int32_t>(n), *lrow = sparse<int32_t>((int64_t)n + 1),
            *urow = sparse<int32_t>((int64_t)n + 1), colidx[1010] = {};
    int32_t *lrec = sparse<int32_t>((int64_t)n * PAIR_REC<2>), *urec = sparse<int32_t>((int64_t)n * PAIR_REC<2>);
    rowptr[i - 1] = d - 3;
    rowptr[i] = d - 1;
    rowptr[i + 1] = d + 1;
    diag[i - 1] = d - 2;
    diag[i] = d;
    colidx[d - 3] = i - 2;
    colidx[d - 2] = i - 1;
    colidx[d - 1] = i - 1;
    colidx[d] = i;
    lrow[i - 1] = 77;
    const int64_t t = 2 * (int64_t)i;
    for (int64_t q : {t, t + 1, t + 2})   // the row's two records, and a thread past the last row
        pat_pairs_body<2>((unsigned)(q / 256), 256, (unsigned)(q % 256), n, rowptr, colidx, diag, lrow, urow, lrec, urec);
    const int32_t *w = lrec + (int64_t)i * PAIR_REC<2>;
    expect(w[0] == i - 1 && w[1] == -1 && w[2] == (77 << 2 | 1) && w[4] == i - 2 && w[5] == -1, "lower record");
    w = urec + (int64_t)i * PAIR_REC<2>;
    expect(w[0] == -1 && w[1] == -1 && w[2] == 0, "upper record");

    // offsets that a record's 30 bits hold, and those for which the pattern keeps none
    const int64_t lim = (int64_t)1 << 30;
    expect(pair_records_hold(lim - 1, lim - 1, lim - 1), "records below the limit");
    expect(!pair_records_hold(lim, 0, 0) && !pair_records_hold(5, lim, 0) && !pair_records_hold(5, 0, lim), "records at the limit");
    if (!failures) printf("OK\n");
    return failures ? 1 : 0;
}
