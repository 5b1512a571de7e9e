// The dispatch rules at shapes measured on either side of their lines: "rule arguments -> 0 or 1" lines,
// compared with the measured choice by tests/test_rules.py.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "rules.h"

using namespace abilu_rules;

int main(int argc, char **argv) {
    auto a = [&](int q) { return q < argc ? std::atoll(argv[q]) : 0; };
    if (argc > 1 && !std::strcmp(argv[1], "chain_apply")) return chain_apply((int)a(2), a(3), (int)a(4), a(5) != 0);
    if (argc > 1 && !std::strcmp(argv[1], "chain_factor")) return chain_factor((int)a(2), a(3), (int)a(4), a(5) != 0, a(6) != 0);
    if (argc > 1 && !std::strcmp(argv[1], "sweep_pairs")) return sweep_pairs((int)a(2), (int)a(3), a(4) != 0, a(5) != 0, a(6), a(7), a(8) != 0);
    if (argc > 1 && !std::strcmp(argv[1], "crowded_sweep")) return crowded_sweep(a(2), a(3));
    if (argc > 1 && !std::strcmp(argv[1], "sweep_by_blocks")) return sweep_by_blocks(a(2), a(3), a(4), a(5), a(6) != 0, a(7) != 0, a(8) != 0);
    if (argc > 2 && !std::strcmp(argv[1], "launches_ahead")) return launches_ahead(a(2), a(3)) == a(4);
    if (argc > 1 && !std::strcmp(argv[1], "backward_descends")) return backward_descends((int)a(2));
    if (argc > 1 && !std::strcmp(argv[1], "apply_ends_descending")) return apply_ends_descending((int)a(2), a(3) != 0);
    return 2;
}
