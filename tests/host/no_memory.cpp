// A caller out of host memory: operator new fails once `failing` is set. An entry point then has to
// return ABILU_ENOMEM; an exception that left it would end this program. The arguments are not used
// before the allocation, and no device is needed.
#include <cstdio>
#include <cstdlib>
#include <new>

#include "abilu.h"

static bool failing = false;

void *operator new(std::size_t n) {
    void *p = failing ? nullptr : std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void *operator new(std::size_t n, const std::nothrow_t &) noexcept { return failing ? nullptr : std::malloc(n ? n : 1); }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

int main() {
    static int32_t rowptr[2] = {0, 1}, colidx[1] = {0};
    abilu_pattern *p = (abilu_pattern *)rowptr;
    failing = true;
    const abilu_status st = abilu_build_pattern(1, rowptr, colidx, 4, nullptr, &p);
    failing = false;
    if (st != ABILU_ENOMEM || p) {
        std::printf("status %d\n", (int)st);
        return 1;
    }
    std::printf("OK\n");
    return 0;
}
