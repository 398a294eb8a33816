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

// Launches of more than 2^32 work-items along x are refused by the hardware's grid.
static void check_limits()
{
    for (uint32_t threads : {256u, 512u, 1024u})
        for (int32_t m : {1, 100, 4096, 5792, 5793, 8192, 46875, 92681})
            for (int32_t G : {2, 8, 64}) {
                const int32_t L = strip_len_that_fits(m, G, threads);
                CHECK(L >= G && strip_align_prefix((uint32_t)m, (uint32_t)L) * threads < (1ull << 32),
                      "m %d G %d threads %u: %d", m, G, threads, L);
                CHECK(L == G || strip_align_prefix((uint32_t)m, (uint32_t)L / 2) * threads >= (1ull << 32),
                      "m %d G %d threads %u: %d is longer than needed", m, G, threads, L);
            }
    for (uint32_t flags : {0u, (uint32_t)TRI_FLAG_XCD_SWIZZLE, (uint32_t)TRI_FLAG_ORDER_PAIRS})
        for (uint32_t threads : {256u, 512u, 1024u})
            for (uint32_t T : {1u, 1000u, (1u << 22) - 1, 1u << 22, (1u << 23) + 1, 1u << 24}) {
                TileGrid g{1, flags | (flags <= 1u ? kLambda24 : 0u), T};
                dim3 grid(T);
                grid_that_fits(g, threads, grid);
                CHECK((uint64_t)grid.x * threads < (1ull << 32) && grid.y < 65536u, "T %u", T);
                CHECK((uint64_t)grid.x * grid.y >= T, "T %u", T);
                if (grid.y > 1) {
                    CHECK(grid.x == (1u << 16) && !(g.flags & kLambda24), "T %u", T);
                    CHECK(((g.flags & kLambda32) != 0) == (flags == 0), "T %u flags %u", T, flags);
                } else if (grid.x != (1u << 16)) {
                    CHECK(grid.x == T, "T %u", T);
                }
            }
}

int main()
{
    check_limits();
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
