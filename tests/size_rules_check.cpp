// Host check of the size rules that the kernels and the host side share, built with
// UndefinedBehaviorSanitizer by tests/test_size_rules.py. Prints "ok" and the checks made.
#include <cstdio>
#include <cstdlib>

#include "olive_internal.hpp"

using namespace olive;

static long n_checks = 0;
#define CHECK(c)                                                              \
    do {                                                                      \
        ++n_checks;                                                           \
        if (!(c)) {                                                           \
            std::printf("line %d: %s\n", __LINE__, #c);                       \
            std::exit(1);                                                     \
        }                                                                     \
    } while (0)

// Row tiles of a pass, up to a pass that takes every scored row as one chunk.
static void row_tiles() {
    for (int tile : {SIMPLE_BT, MFMA_BT, WIDE_BT})
        for (int64_t rows : {0, 1, tile - 1, tile, tile + 1, 8192, kOneChunk - 1, kOneChunk}) {
            const int64_t n = tiles_of(rows, tile);
            CHECK(n * tile >= rows && (n - 1) * tile < rows && n <= 0x7fffffff);
        }
}

int main() {
    row_tiles();
    std::printf("ok %ld checks\n", n_checks);
    return 0;
}
