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

static int splits(uint32_t n_tiles, int ksteps, int G, int64_t room) {
    uint64_t best = ~(uint64_t)0;
    for (int s = 1; s <= GEMM_PARTS; ++s) {
        const uint64_t k = gemm_split_key(s, n_tiles, ksteps, G, room);
        best = k < best ? k : best;
    }
    return (int)(best & 127);
}

// The reserved partial tiles hold every split that a workspace of max(tiles, 3 G) tiles
// allows, for the full product and for any smaller number of tiles in it.
static void product_splits() {
    for (int G : {64, 256, 304})
        for (int64_t ksteps : {4, 5, 16, 17, 63, 64, 65, 200, 782, 2374})
            for (int64_t tiles = 1; tiles <= 400; tiles += tiles < 40 ? 1 : 23) {
                const int64_t room = gemm_ws_tiles(tiles, ksteps, G);
                const int64_t all = tiles > 3 * G ? tiles : 3 * G;
                CHECK(room <= all);
                for (int64_t n = 1; n <= tiles; n += n < 40 ? 1 : 17) {
                    const int s = splits((uint32_t)n, (int)ksteps, G, room);
                    CHECK(s == splits((uint32_t)n, (int)ksteps, G, all));
                    CHECK((s - 1) * n <= room && (s - 1) * ((ksteps + s - 1) / s) < ksteps);
                }
            }
}

int main() {
    row_tiles();
    product_splits();
    std::printf("ok %ld checks\n", n_checks);
    return 0;
}
