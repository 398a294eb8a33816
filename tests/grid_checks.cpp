// Host checks of the launch and strip arithmetic in maps.hpp (compiled for the
// host alone, by test_grid_arithmetic.py).  Prints what fails; exit code 1 then.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "maps.hpp"

using namespace trimap;

static int failures = 0;

#define CHECK(cond, ...)                        \
    do {                                        \
        if (!(cond) && ++failures <= 20) {      \
            printf("%s: ", #cond);              \
            printf(__VA_ARGS__);                \
            printf("\n");                       \
        }                                       \
    } while (0)

// The strips of one grid row walked in runs: every tile that the map gives, once.
template <int MAP>
static void check_runs(int32_t m, int32_t gx, int32_t gy, int32_t G)
{
    const TileGrid g{m, 0u, (uint64_t)m * (m + 1) / 2};
    const StripGrid sg{0u, G, 1, gx, gy};
    std::vector<int> seen((size_t)m * m, 0);
    for (int32_t by = 0; by < gy; ++by)
        for (int32_t first = 0; first < gx; first += G)
            for (int32_t k = 0; k < G;) {
                int32_t bi, bj;
                if (first + k >= gx || !tile_at_xy<MAP>(g, first + k, by, bi, bj)) {
                    ++k;
                    continue;
                }
                const int32_t len = strip_run<MAP>(m, sg, first + k, by, k, bi, bj);
                CHECK(len >= 1 && k + len <= G, "map %d m %d G %d by %d k %d len %d", MAP, m, G, by,
                      k, len);
                if (len < 1) return;
                for (int32_t c = 0; c < len; ++c) {  // the run's tiles, by the map itself
                    int32_t ti, tj;
                    const bool ok = first + k + c < gx &&
                                    tile_at_xy<MAP>(g, first + k + c, by, ti, tj);
                    CHECK(ok && ti == bi && tj >= bj && tj < bj + len, "map %d m %d G %d by %d x %d",
                          MAP, m, G, by, first + k + c);
                    if (ok && (uint32_t)ti < (uint32_t)m && (uint32_t)tj < (uint32_t)m)
                        ++seen[(size_t)ti * m + tj];
                }
                k += len;
            }
    for (int32_t i = 0; i < m; ++i)
        for (int32_t j = 0; j < m; ++j)
            CHECK(seen[(size_t)i * m + j] == (j <= i), "map %d m %d G %d tile %d %d", MAP, m, G, i, j);
}

int main()
{
    for (int32_t G : {2, 4, 8, 64})
        for (int32_t m = 1; m <= 130; ++m) {
            check_runs<MAP_BB>(m, m, m, G);
            if (m & 1) check_runs<MAP_RB>(m, m, (m + 1) / 2, G);
            else check_runs<MAP_RB>(m, m + 1, m / 2, G);
            if ((m & (m - 1)) == 0) check_runs<MAP_REC>(m, m > 1 ? m / 2 : 1, m > 1 ? m + 1 : 1, G);
        }
    printf("%d failures\n", failures);
    return failures ? 1 : 0;
}
