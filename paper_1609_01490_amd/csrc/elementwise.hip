// Triangular elementwise kernels: one workgroup per tile rho x rho, the tile
// chosen by a parallel-space map (block-space mapping, Section 3.1: the
// block coordinate is mapped, each thread adds its offset inside the block).
//
//  * AXPYT_F32: C[i][j] = fl(fl(a X[i][j]) + Y[j][i]) for j <= i.  The mirror
//    tile of Y is read row-major (coalesced) and transposed through LDS.
//  * XORMUL_I32: C[i][j] = (A[i] xor B[j]) + i j (mod 2^32), the dummy
//    kernel of Sections 4.1 and 5 with a real per-cell store.
//  * EDM4_F32: C[i][j] = |P_i - P_j| for four features per point, the
//    global-memory distance test of Section 5: both points come straight
//    from global memory (they stay in L1/L2), nothing is staged in LDS.
//
// All are HBM-bound: 12 B (axpyt) or 4 B (xormul, edm4) of algorithmic
// traffic per cell.  Rows move as 16-byte vectors where the pitch and the
// matrices allow it.  How they are moved depends on where rows start:
//  * every row on a 128-byte line (ld % 32 == 0, aligned matrices):
//    non-temporal loads and stores (nothing is read twice).
//  * else, axpyt, and tiles below 32: a tile's rows begin and end inside
//    lines that the neighbouring tiles share.  Cached loads and stores, and
//    under lambda the swizzled order, which keeps neighbours on one L2,
//    where the halves of a line meet: n = 20001 (ld 20001), tile 32 1152 ->
//    530 us, 64 823 -> 511, 128 662 -> 522; n = 8001, tile 64 137 -> 83.
//  * else, xormul and edm4 at tiles from 32: k_lines, whose tiles are shifted,
//    row by row, onto the lines.
// UTM (thread space) has no tile and gets its own scalar
// kernel, reading Y[j][i] straight from memory as the map implies.
#include <type_traits>

#include "bodies.hpp"
#include "common.hpp"
#include "maps.hpp"

namespace trimap {

TileGrid plan_tile_grid(const tri_plan *p);
TileGrid plan_tile_grid_swizzled(const tri_plan *p);

typedef float f4 __attribute__((ext_vector_type(4)));
typedef int i4 __attribute__((ext_vector_type(4)));

struct ElemArgs {
    TileGrid g;
    int32_t n;
    int64_t ld;
    const void *x;
    const void *y;
    void *c;
    float a;
};

// Loads and stores of the output, non-temporal or cached.
template <bool NT, typename V>
__device__ __forceinline__ V load_as(const V *p)
{
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

template <bool NT, typename V>
__device__ __forceinline__ void store_as(V v, V *p)
{
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// threads per workgroup and elements per vector for a tile size
template <int TILE, bool VECTOR>
struct ElemShape {
    static constexpr int VEC = (VECTOR && TILE >= 16) ? 4 : 1;
    static constexpr int NT_RAW = TILE * TILE / VEC;
    // tile 128 takes 512 threads: its 66 KB transpose buffer holds the CU to
    // two workgroups, so the extra waves are what keeps more loads in flight
    static constexpr int NT_MAX = TILE >= 128 ? 512 : 256;
    static constexpr int NT = NT_RAW > NT_MAX ? NT_MAX : NT_RAW;
    static constexpr int VPR = TILE / VEC;    // vectors per row
    static constexpr int RPP = NT / VPR;      // rows per pass
    static constexpr int PASSES = TILE / RPP;
    static_assert(RPP * PASSES == TILE, "tile shape");
};

template <int MAP, int TILE, bool VECTOR, bool STREAM>
__global__ void __launch_bounds__((ElemShape<TILE, VECTOR>::NT)) k_axpyt(ElemArgs p)
{
    using S = ElemShape<TILE, VECTOR>;
    int32_t bi, bj;
    if (!tile_of_block<MAP>(p.g, bi, bj)) return;

    __shared__ float ys[TILE][TILE + 1];
    const int tr = threadIdx.x / S::VPR;
    const int tc = (threadIdx.x % S::VPR) * S::VEC;
    const int32_t n = p.n;
    const int64_t ld = p.ld;
    const int32_t i0 = bi * TILE, j0 = bj * TILE;
    const float *X = (const float *)p.x;
    const float *Y = (const float *)p.y;
    float *C = (float *)p.c;
    const float a = p.a;
    // every cell of the tile is in the domain
    const bool full = (bj < bi) && (i0 + TILE <= n);

    // Every load is unconditional, so that all of them are in flight at once
    // (a load under a condition is waited for where the branches rejoin).
    // On tiles that cross the diagonal or the last row the addresses are
    // clamped into the n x ld matrices; the values read there belong to
    // cells that are never stored.  X first, then the mirror tile of Y
    // (rows j0.., columns i0..; Y[j][i] lands in ys[j-j0][i-i0]).
    using V = typename std::conditional<S::VEC == 4, f4, float>::type;
    const int32_t cmax = (int32_t)(ld - S::VEC);  // last column start of a vector
    V xv[S::PASSES], yv[S::PASSES];
#pragma unroll
    for (int ps = 0; ps < S::PASSES; ++ps) {
        const int r = tr + ps * S::RPP;
        int32_t i = i0 + r, jc = j0 + tc;
        if (!full) {
            i = i < n ? i : n - 1;
            jc = jc < cmax ? jc : cmax;
        }
        xv[ps] = load_as<STREAM>((const V *)(X + (int64_t)i * ld + jc));
    }
#pragma unroll
    for (int ps = 0; ps < S::PASSES; ++ps) {
        const int r = tr + ps * S::RPP;
        int32_t jr = j0 + r, ic = i0 + tc;
        if (!full) {
            jr = jr < n ? jr : n - 1;
            ic = ic < cmax ? ic : cmax;
        }
        yv[ps] = load_as<STREAM>((const V *)(Y + (int64_t)jr * ld + ic));
    }
#pragma unroll
    for (int ps = 0; ps < S::PASSES; ++ps) {
        const int r = tr + ps * S::RPP;
        if constexpr (S::VEC == 4) {
            ys[r][tc + 0] = yv[ps].x;
            ys[r][tc + 1] = yv[ps].y;
            ys[r][tc + 2] = yv[ps].z;
            ys[r][tc + 3] = yv[ps].w;
        } else {
            ys[r][tc] = yv[ps];
        }
    }
    __syncthreads();

#pragma unroll
    for (int ps = 0; ps < S::PASSES; ++ps) {
        const int r = tr + ps * S::RPP;
        const int32_t i = i0 + r, jc = j0 + tc;
        if (!full && (i >= n || jc > i)) continue;
        float *crow = C + (int64_t)i * ld + jc;
        if constexpr (S::VEC == 4) {
            const f4 x4 = xv[ps];
            f4 o;
            o.x = __fadd_rn(__fmul_rn(a, x4.x), ys[tc + 0][r]);
            o.y = __fadd_rn(__fmul_rn(a, x4.y), ys[tc + 1][r]);
            o.z = __fadd_rn(__fmul_rn(a, x4.z), ys[tc + 2][r]);
            o.w = __fadd_rn(__fmul_rn(a, x4.w), ys[tc + 3][r]);
            if (full || jc + 3 <= i) {
                store_as<STREAM>(o, (f4 *)crow);
            } else {  // the vector straddles the diagonal
                crow[0] = o.x;
                if (jc + 1 <= i) crow[1] = o.y;
                if (jc + 2 <= i) crow[2] = o.z;
            }
        } else {
            store_as<STREAM>(__fadd_rn(__fmul_rn(a, xv[ps]), ys[tc][r]), crow);
        }
    }
}

// Strip form of AXPYT for tiles 16 and 32 (plans with TRI_FLAG_STRIP): a
// workgroup of four waves walks G consecutive tiles of the map (strip_first
// and strip_tile; every tile still mapped on its own), wave w taking tiles
// w, w + 4, w + 8, ... of the strip, so that the four waves work on adjacent
// tiles and one dispatch serves G tiles instead of one.  A wave moves a
// whole tile by itself: 16-byte vectors, rows per pass 64 / (TILE / 4), and
// its own transpose buffer in LDS (the LDS operations of one wave execute in
// order, so a wave needs no barrier between its tiles).  The loads of the
// wave's next tile are issued before the current tile's transpose and
// stores.  Same arithmetic and operation order as k_axpyt.
template <int MAP, int TILE>
__global__ void __launch_bounds__(256) k_axpyt_strip(ElemArgs p, StripGrid sg)
{
    constexpr int VPR = TILE / 4, RPP = 64 / VPR, PASSES = TILE / RPP;
    static_assert(RPP * PASSES == TILE, "tile shape");
    __shared__ float ysh[4][TILE][TILE + 1];
    const int l = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float (*ys)[TILE + 1] = ysh[w];
    const int tr = l / VPR, tc = (l % VPR) * 4;
    const int32_t n = p.n;
    const int64_t ld = p.ld;
    const float *X = (const float *)p.x;
    const float *Y = (const float *)p.y;
    float *C = (float *)p.c;
    const float a = p.a;
    const int32_t cmax = (int32_t)(ld - 4);  // last column start of a vector
    const uint32_t first = strip_first<MAP>(p.g, sg);

    // the wave's next tile at or after strip index k (k >= G: none)
    auto next = [&](int k, int32_t &bi, int32_t &bj) {
        for (; k < sg.G; k += 4)
            if (strip_tile<MAP>(p.g, sg, first, k, bi, bj)) break;
        bi = __builtin_amdgcn_readfirstlane(bi);
        bj = __builtin_amdgcn_readfirstlane(bj);
        return k;
    };
    f4 xv[PASSES], yv[PASSES];
    // every load unconditional; addresses clamped into the matrices on
    // tiles that cross the diagonal or the last row (values never stored)
    auto load = [&](int32_t bi, int32_t bj) {
        const int32_t i0 = bi * TILE, j0 = bj * TILE;
        const bool full = (bj < bi) && (i0 + TILE <= n);
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) {
            const int r = tr + ps * RPP;
            int32_t i = i0 + r, jc = j0 + tc;
            if (!full) {
                i = i < n ? i : n - 1;
                jc = jc < cmax ? jc : cmax;
            }
            xv[ps] = __builtin_nontemporal_load((const f4 *)(X + (int64_t)i * ld + jc));
        }
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) {
            const int r = tr + ps * RPP;
            int32_t jr = j0 + r, ic = i0 + tc;
            if (!full) {
                jr = jr < n ? jr : n - 1;
                ic = ic < cmax ? ic : cmax;
            }
            yv[ps] = __builtin_nontemporal_load((const f4 *)(Y + (int64_t)jr * ld + ic));
        }
    };

    int32_t bi = 0, bj = 0;
    int k = next(w, bi, bj);
    if (k >= sg.G) return;
    load(bi, bj);
    while (k < sg.G) {
        // this tile's operands into the transpose buffer and registers
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) {
            const int r = tr + ps * RPP;
            ys[r][tc + 0] = yv[ps].x;
            ys[r][tc + 1] = yv[ps].y;
            ys[r][tc + 2] = yv[ps].z;
            ys[r][tc + 3] = yv[ps].w;
        }
        f4 xc[PASSES];
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) xc[ps] = xv[ps];
        const int32_t i0 = bi * TILE, j0 = bj * TILE;
        const bool full = (bj < bi) && (i0 + TILE <= n);
        // the next tile's loads, in flight during this tile's stores
        int32_t nbi = 0, nbj = 0;
        const int nk = next(k + 4, nbi, nbj);
        if (nk < sg.G) load(nbi, nbj);
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) {
            const int r = tr + ps * RPP;
            const int32_t i = i0 + r, jc = j0 + tc;
            if (!full && (i >= n || jc > i)) continue;
            float *crow = C + (int64_t)i * ld + jc;
            f4 o;
            o.x = __fadd_rn(__fmul_rn(a, xc[ps].x), ys[tc + 0][r]);
            o.y = __fadd_rn(__fmul_rn(a, xc[ps].y), ys[tc + 1][r]);
            o.z = __fadd_rn(__fmul_rn(a, xc[ps].z), ys[tc + 2][r]);
            o.w = __fadd_rn(__fmul_rn(a, xc[ps].w), ys[tc + 3][r]);
            if (full || jc + 3 <= i) {
                __builtin_nontemporal_store(o, (f4 *)crow);
            } else {  // the vector straddles the diagonal
                crow[0] = o.x;
                if (jc + 1 <= i) crow[1] = o.y;
                if (jc + 2 <= i) crow[2] = o.z;
            }
        }
        k = nk;
        bi = nbi;
        bj = nbj;
    }
}

// Tile 16 in strips: a wave moves two tiles at once, one per half-wave
// (tiles 2 j and 2 j + 1 of the strip, j = w, w + 4, ...), so that where the
// two are neighbours in a tile row (the usual case) every load and store
// instruction covers whole 128-byte lines: 8 rows x 64 bytes of each tile.
// Each half-wave maps its tile on its own; a half whose tile is missing
// (past the strip or the grid) loads tile (0, 0) and stores nothing.
template <int MAP>
__global__ void __launch_bounds__(256) k_axpyt_strip_pairs(ElemArgs p, StripGrid sg)
{
    constexpr int TILE = 16, RPP = 8, PASSES = 2;
    __shared__ float ysh[8][TILE][TILE + 1];
    const int l = threadIdx.x & 63, h = l >> 5, hl = l & 31;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float (*ys)[TILE + 1] = ysh[2 * w + h];
    const int tr = hl / 4, tc = (hl % 4) * 4;
    const int32_t n = p.n;
    const int64_t ld = p.ld;
    const float *X = (const float *)p.x;
    const float *Y = (const float *)p.y;
    float *C = (float *)p.c;
    const float a = p.a;
    const int32_t cmax = (int32_t)(ld - 4);
    const uint32_t first = strip_first<MAP>(p.g, sg);

    // this half's tile of pair j (false: none)
    auto tile = [&](int j, int32_t &bi, int32_t &bj) {
        const int k = 2 * j + h;
        const bool v = k < sg.G && strip_tile<MAP>(p.g, sg, first, k, bi, bj);
        if (!v) bi = bj = 0;
        return v;
    };
    f4 xv[PASSES], yv[PASSES];
    auto load = [&](int32_t bi, int32_t bj) {
        const int32_t i0 = bi * TILE, j0 = bj * TILE;
        const bool full = (bj < bi) && (i0 + TILE <= n);
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) {
            const int r = tr + ps * RPP;
            int32_t i = i0 + r, jc = j0 + tc;
            if (!full) {
                i = i < n ? i : n - 1;
                jc = jc < cmax ? jc : cmax;
            }
            xv[ps] = __builtin_nontemporal_load((const f4 *)(X + (int64_t)i * ld + jc));
        }
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) {
            const int r = tr + ps * RPP;
            int32_t jr = j0 + r, ic = i0 + tc;
            if (!full) {
                jr = jr < n ? jr : n - 1;
                ic = ic < cmax ? ic : cmax;
            }
            yv[ps] = __builtin_nontemporal_load((const f4 *)(Y + (int64_t)jr * ld + ic));
        }
    };

    int j = w;
    int32_t bi = 0, bj = 0;
    bool v = tile(j, bi, bj);
    load(bi, bj);
    while (2 * j < sg.G) {
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) {
            const int r = tr + ps * RPP;
            ys[r][tc + 0] = yv[ps].x;
            ys[r][tc + 1] = yv[ps].y;
            ys[r][tc + 2] = yv[ps].z;
            ys[r][tc + 3] = yv[ps].w;
        }
        f4 xc[PASSES];
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) xc[ps] = xv[ps];
        const int32_t i0 = bi * TILE, j0 = bj * TILE;
        const bool full = v && (bj < bi) && (i0 + TILE <= n);
        const bool cv = v;
        // the next pair's loads, in flight during this pair's stores
        int32_t nbi = 0, nbj = 0;
        const int nj = j + 4;
        const bool nv = tile(nj, nbi, nbj);
        if (2 * nj < sg.G) load(nbi, nbj);
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) {
            const int r = tr + ps * RPP;
            const int32_t i = i0 + r, jc = j0 + tc;
            if (!cv || (!full && (i >= n || jc > i))) continue;
            float *crow = C + (int64_t)i * ld + jc;
            f4 o;
            o.x = __fadd_rn(__fmul_rn(a, xc[ps].x), ys[tc + 0][r]);
            o.y = __fadd_rn(__fmul_rn(a, xc[ps].y), ys[tc + 1][r]);
            o.z = __fadd_rn(__fmul_rn(a, xc[ps].z), ys[tc + 2][r]);
            o.w = __fadd_rn(__fmul_rn(a, xc[ps].w), ys[tc + 3][r]);
            if (full || jc + 3 <= i) {
                __builtin_nontemporal_store(o, (f4 *)crow);
            } else {  // the vector straddles the diagonal
                crow[0] = o.x;
                if (jc + 1 <= i) crow[1] = o.y;
                if (jc + 2 <= i) crow[2] = o.z;
            }
        }
        j = nj;
        v = nv;
        bi = nbi;
        bj = nbj;
    }
}

// Tile 16 in two-row band strips (TRI_FLAG_STRIP_BAND): a wave moves a
// 2 x 2 block of tiles at once (tiles 4 q .. 4 q + 3 of the strip, rows
// 2 p and 2 p + 1, columns c and c + 1, q = w, w + 4, ...), each of the
// four located by the map on its own.  Within the block every row of X and
// C is a whole 128-byte line across two tiles, and so is every row of the
// mirror block of Y across the two tile rows; the block moves as one
// 32 x 32 transpose through the wave's LDS buffer.  Tile (r, c) of the
// block is tile 4 q + 2 c + r; a lane's 16-byte vector at block row R,
// column C belongs to tile (R / 16, C / 16) for X and C and to tile
// (C / 16, R / 16) for Y, whose rows are the tiles' columns.  A missing
// tile (above the diagonal, past the last row or the strip) loads from
// tile (0, 0) and stores nothing.  Same arithmetic and operation order as
// k_axpyt.
template <int MAP>
__global__ void __launch_bounds__(256) k_axpyt_strip_quads(ElemArgs p, StripGrid sg)
{
    constexpr int TILE = 16, BLK = 32, VPR = BLK / 4, RPP = 64 / VPR, PASSES = BLK / RPP;
    __shared__ float ysh[4][BLK][BLK + 1];
    const int l = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float (*ys)[BLK + 1] = ysh[w];
    const int tr = l / VPR, tc = (l % VPR) * 4;  // block row (pass 0), block column
    const int lc = tc / TILE, tcl = tc % TILE;    // the lane's tile column, column in it
    const int32_t n = p.n;
    const int64_t ld = p.ld;
    const float *X = (const float *)p.x;
    const float *Y = (const float *)p.y;
    float *C = (float *)p.c;
    const float a = p.a;
    const int32_t cmax = (int32_t)(ld - 4);
    const uint32_t first = strip_first<MAP>(p.g, sg);

    struct Quad {
        int32_t bi[2][2], bj[2][2];  // [r][c]
        bool v[2][2];
    };
    auto locate = [&](int q, Quad &Q) {
        bool any = false;
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int k = 4 * q + 2 * c + r;
                int32_t bi = 0, bj = 0;
                bool v = k < sg.G && strip_tile<MAP>(p.g, sg, first, k, bi, bj);
                if (!v) bi = bj = 0;
                Q.bi[r][c] = __builtin_amdgcn_readfirstlane(bi);
                Q.bj[r][c] = __builtin_amdgcn_readfirstlane(bj);
                Q.v[r][c] = v;
                any = any || v;
            }
        return any;
    };
    f4 xv[PASSES], yv[PASSES];
    auto load = [&](const Quad &Q) {
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) {
            const int R = tr + ps * RPP, rt = R / TILE, rl = R % TILE;
            // X: tile (rt, lc), row rl, columns tcl ..
            const int32_t bi = lc ? Q.bi[rt][1] : Q.bi[rt][0];
            const int32_t bj = lc ? Q.bj[rt][1] : Q.bj[rt][0];
            const bool full = (bj < bi) && (bi * TILE + TILE <= n);
            int32_t i = bi * TILE + rl, jc = bj * TILE + tcl;
            if (!full) {
                i = i < n ? i : n - 1;
                jc = jc < cmax ? jc : cmax;
            }
            xv[ps] = __builtin_nontemporal_load((const f4 *)(X + (int64_t)i * ld + jc));
        }
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) {
            const int R = tr + ps * RPP, rt = R / TILE, rl = R % TILE;
            // Y: the mirror of tile (lc, rt): Y row bj * 16 + rl, columns bi * 16 + tcl ..
            const int32_t bi = rt ? Q.bi[lc][1] : Q.bi[lc][0];
            const int32_t bj = rt ? Q.bj[lc][1] : Q.bj[lc][0];
            const bool full = (bj < bi) && (bi * TILE + TILE <= n);
            int32_t jr = bj * TILE + rl, ic = bi * TILE + tcl;
            if (!full) {
                jr = jr < n ? jr : n - 1;
                ic = ic < cmax ? ic : cmax;
            }
            yv[ps] = __builtin_nontemporal_load((const f4 *)(Y + (int64_t)jr * ld + ic));
        }
    };

    int q = w;
    Quad Q;
    bool v = locate(q, Q);
    while (4 * q < sg.G && !v) v = locate(q += 4, Q);
    if (4 * q >= sg.G) return;
    load(Q);
    while (4 * q < sg.G) {
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) {
            const int R = tr + ps * RPP;
            ys[R][tc + 0] = yv[ps].x;
            ys[R][tc + 1] = yv[ps].y;
            ys[R][tc + 2] = yv[ps].z;
            ys[R][tc + 3] = yv[ps].w;
        }
        f4 xc[PASSES];
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) xc[ps] = xv[ps];
        const Quad cq = Q;
        // the next block's loads, in flight during this block's stores
        int nq = q + 4;
        bool nv = false;
        while (4 * nq < sg.G && !(nv = locate(nq, Q))) nq += 4;
        if (4 * nq < sg.G) load(Q);
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) {
            const int R = tr + ps * RPP, rt = R / TILE, rl = R % TILE;
            const int32_t bi = lc ? cq.bi[rt][1] : cq.bi[rt][0];
            const int32_t bj = lc ? cq.bj[rt][1] : cq.bj[rt][0];
            const bool tv = lc ? cq.v[rt][1] : cq.v[rt][0];
            const bool full = tv && (bj < bi) && (bi * TILE + TILE <= n);
            const int32_t i = bi * TILE + rl, jc = bj * TILE + tcl;
            if (!tv || (!full && (i >= n || jc > i))) continue;
            float *crow = C + (int64_t)i * ld + jc;
            f4 o;
            o.x = __fadd_rn(__fmul_rn(a, xc[ps].x), ys[tc + 0][R]);
            o.y = __fadd_rn(__fmul_rn(a, xc[ps].y), ys[tc + 1][R]);
            o.z = __fadd_rn(__fmul_rn(a, xc[ps].z), ys[tc + 2][R]);
            o.w = __fadd_rn(__fmul_rn(a, xc[ps].w), ys[tc + 3][R]);
            if (full || jc + 3 <= i) {
                __builtin_nontemporal_store(o, (f4 *)crow);
            } else {  // the vector straddles the diagonal
                crow[0] = o.x;
                if (jc + 1 <= i) crow[1] = o.y;
                if (jc + 2 <= i) crow[2] = o.z;
            }
        }
        q = nq;
        (void)nv;
    }
}

template <int MAP, int TILE, bool VECTOR, bool STREAM>
__global__ void __launch_bounds__((ElemShape<TILE, VECTOR>::NT)) k_xormul(ElemArgs p)
{
    using S = ElemShape<TILE, VECTOR>;
    int32_t bi, bj;
    if (!tile_of_block<MAP>(p.g, bi, bj)) return;

    const int tr = threadIdx.x / S::VPR;
    const int tc = (threadIdx.x % S::VPR) * S::VEC;
    const int32_t n = p.n;
    const int64_t ld = p.ld;
    const int32_t i0 = bi * TILE, j0 = bj * TILE;
    const uint32_t *A = (const uint32_t *)p.x;
    const uint32_t *B = (const uint32_t *)p.y;
    int32_t *C = (int32_t *)p.c;
    const bool full = (bj < bi) && (i0 + TILE <= n);

#pragma unroll
    for (int ps = 0; ps < S::PASSES; ++ps) {
        const int r = tr + ps * S::RPP;
        const int32_t i = i0 + r, jc = j0 + tc;
        if (!full && (i >= n || jc > i)) continue;
        const uint32_t ai = A[i];
        int32_t *crow = C + (int64_t)i * ld + jc;
        if constexpr (S::VEC == 4) {
            // B[jc .. jc+3]: jc + 3 may pass n on the last tile row, so read
            // element by element there (B holds exactly n values)
            uint32_t b0 = B[jc], b1 = 0, b2 = 0, b3 = 0;
            if (full || jc + 3 < n) { b1 = B[jc + 1]; b2 = B[jc + 2]; b3 = B[jc + 3]; }
            else {
                if (jc + 1 < n) b1 = B[jc + 1];
                if (jc + 2 < n) b2 = B[jc + 2];
            }
            const uint32_t ui = (uint32_t)i;
            i4 o;
            o.x = (int32_t)((ai ^ b0) + ui * (uint32_t)(jc + 0));
            o.y = (int32_t)((ai ^ b1) + ui * (uint32_t)(jc + 1));
            o.z = (int32_t)((ai ^ b2) + ui * (uint32_t)(jc + 2));
            o.w = (int32_t)((ai ^ b3) + ui * (uint32_t)(jc + 3));
            if (full || jc + 3 <= i) {
                store_as<STREAM>(o, (i4 *)crow);
            } else {
                crow[0] = o.x;
                if (jc + 1 <= i) crow[1] = o.y;
                if (jc + 2 <= i) crow[2] = o.z;
            }
        } else {
            const uint32_t v = (ai ^ B[jc]) + (uint32_t)i * (uint32_t)jc;
            store_as<STREAM>((int32_t)v, crow);
        }
    }
}

// |P_i - P_j|^2 with a fixed operation order: differences, squares, the sum
// ((dx^2 + dy^2) + dz^2) + dw^2, each rounded to binary32.  The distance is
// its correctly rounded square root.
__device__ __forceinline__ float square4(f4 a, f4 b)
{
    const float dx = __fsub_rn(a.x, b.x), dy = __fsub_rn(a.y, b.y);
    const float dz = __fsub_rn(a.z, b.z), dw = __fsub_rn(a.w, b.w);
    float s = __fadd_rn(__fmul_rn(dx, dx), __fmul_rn(dy, dy));
    s = __fadd_rn(s, __fmul_rn(dz, dz));
    s = __fadd_rn(s, __fmul_rn(dw, dw));
    return s;
}

// SHORT: the short square root, a few rows at a time (n = 4096, tile 64 12.0 ->
// 10.0 us, n = 8192 35 -> 29).  Where the output is far larger than the caches
// the launch is bound by its stores, and the long one, row by row, spreads
// them better (n = 24000, tile 128 210 us, 222 with the short one; n = 32768
// 384, 412; tile 64 402, 415).
template <int MAP, int TILE, bool VECTOR, bool STREAM, bool SHORT>
__global__ void __launch_bounds__((ElemShape<TILE, VECTOR>::NT)) k_edm4(ElemArgs p)
{
    using S = ElemShape<TILE, VECTOR>;
    int32_t bi, bj;
    if (!tile_of_block<MAP>(p.g, bi, bj)) return;

    const int tr = threadIdx.x / S::VPR;
    const int tc = (threadIdx.x % S::VPR) * S::VEC;
    const int32_t n = p.n;
    const int64_t ld = p.ld;
    const int32_t i0 = bi * TILE, j0 = bj * TILE;
    const f4 *P = (const f4 *)p.x;
    float *C = (float *)p.c;
    const bool full = (bj < bi) && (i0 + TILE <= n);

    // the lane's column points (the same for all its rows), read once from
    // global memory; past n - 1 (the ragged last tile) clamped and unused
    const int32_t jc = j0 + tc;
    f4 pj[S::VEC];
#pragma unroll
    for (int v = 0; v < S::VEC; ++v) pj[v] = P[jc + v < n ? jc + v : n - 1];

    // (VEC values of row i, from column jc)
    const auto put = [&](int32_t i, const float *w) {
        float *crow = C + (int64_t)i * ld + jc;
        if constexpr (S::VEC == 4) {
            if (full || jc + 3 <= i) {
                store_as<STREAM>(f4{w[0], w[1], w[2], w[3]}, (f4 *)crow);
            } else {  // the vector straddles the diagonal
                crow[0] = w[0];
                if (jc + 1 <= i) crow[1] = w[1];
                if (jc + 2 <= i) crow[2] = w[2];
            }
        } else {
            store_as<STREAM>(w[0], crow);
        }
    };
    if constexpr (!SHORT) {
#pragma unroll
        for (int ps = 0; ps < S::PASSES; ++ps) {
            const int32_t i = i0 + tr + ps * S::RPP;
            if (!full && (i >= n || jc > i)) continue;
            const f4 pi = P[i];
            float o[S::VEC];
#pragma unroll
            for (int v = 0; v < S::VEC; ++v) o[v] = __builtin_sqrtf(square4(pi, pj[v]));
            put(i, o);
        }
        return;
    }
    constexpr int PG = S::PASSES < 4 ? S::PASSES : 4;
#pragma unroll
    for (int p0 = 0; p0 < S::PASSES; p0 += PG) {
        float o[PG * S::VEC];
        SqrtRange range;
#pragma unroll
        for (int q = 0; q < PG; ++q) {
            const int32_t i = i0 + tr + (p0 + q) * S::RPP;
            const f4 pi = P[full || i < n ? i : n - 1];
#pragma unroll
            for (int v = 0; v < S::VEC; ++v) {
                o[S::VEC * q + v] = square4(pi, pj[v]);
                range.add(o[S::VEC * q + v]);
            }
        }
        range.roots(o);
#pragma unroll
        for (int q = 0; q < PG; ++q) {
            const int32_t i = i0 + tr + (p0 + q) * S::RPP;
            if (!full && (i >= n || jc > i)) continue;
            put(i, &o[S::VEC * q]);
        }
    }
}

// xormul and edm4 where rows do not start on 128-byte lines.  Row i's tiles
// are shifted left by the row's misalignment s_i (in floats, 0 .. 31): tile
// (bi, bj) takes the columns bj rho - s_i .. bj rho - s_i + rho - 1 of row i, a
// whole number of lines, and the diagonal tile one line more, up to column
// i.  So every store instruction writes two whole lines (one per half-wave,
// two rows), whatever the pitch and the alignment.  The tile's column
// operands, 32 more to the left and right, come from LDS.
// n = 10007, ld 10007, tile 64, lambda: edm4 109 -> 43 us; n = 20001 440 -> 155 (tile 128 363 -> 164);
// xormul n = 8001, tile 32 104 -> 29, tile 64 69 -> 28.
template <int OP, int MAP, int TILE>
__global__ void __launch_bounds__(8 * TILE) k_lines(ElemArgs p)
{
    using V = typename std::conditional<OP == TRI_OP_EDM4_F32, f4, uint32_t>::type;
    using R = typename std::conditional<OP == TRI_OP_EDM4_F32, float, int32_t>::type;
    constexpr int NT = 8 * TILE, NL = TILE / 32;  // threads, lines per tile row
    constexpr int RP = 4;                          // rows per half-wave
    int32_t bi, bj;
    if (!tile_of_block<MAP>(p.g, bi, bj)) return;

    __shared__ V rows[TILE], cols[TILE + 64];  // cols: columns j0 - 32 .. j0 + TILE + 31
    const int32_t n = p.n;
    const int64_t ld = p.ld;
    const int32_t i0 = bi * TILE, j0 = bj * TILE;
    const V *A = (const V *)p.x;
    const V *B = OP == TRI_OP_EDM4_F32 ? A : (const V *)p.y;
    for (int t = threadIdx.x; t < 2 * TILE + 64; t += NT) {
        int32_t k = t < TILE ? i0 + t : j0 - 32 + (t - TILE);
        k = k < 0 ? 0 : (k < n ? k : n - 1);
        if (t < TILE) rows[t] = A[k];
        else cols[t - TILE] = B[k];
    }
    __syncthreads();

    const int hw = threadIdx.x >> 5, lane = threadIdx.x & 31;
    const bool full = bj < bi && bj > 0 && i0 + TILE <= n;  // every cell is in the domain
    // lines k0 .. k0 + NL - 1 of the half-wave's rows hw, hw + TILE / 4, ..
    const auto pass = [&](auto lines, int k0) {
        constexpr int K = lines;
        R v[RP * K];
        SqrtRange range;
#pragma unroll
        for (int u = 0; u < RP; ++u) {
            const int r = hw + u * (TILE / RP);
            const int32_t i = i0 + r;
            const int32_t s = (int32_t)(((uintptr_t)((R *)p.c + (int64_t)i * ld) >> 2) & 31);
            const V a = rows[r];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int t = 32 * (k0 + k) + lane - s;
                const V b = cols[t + 32];
                if constexpr (OP == TRI_OP_EDM4_F32) {
                    v[K * u + k] = square4(a, b);
                    range.add(v[K * u + k]);
                } else {
                    v[K * u + k] = (R)((a ^ b) + (uint32_t)i * (uint32_t)(j0 + t));
                }
            }
        }
        if constexpr (OP == TRI_OP_EDM4_F32) range.roots(v);
#pragma unroll
        for (int u = 0; u < RP; ++u) {
            const int32_t i = i0 + hw + u * (TILE / RP);
            R *const row = (R *)p.c + (int64_t)i * ld;
            const int32_t s = (int32_t)(((uintptr_t)row >> 2) & 31);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int32_t j = j0 + 32 * (k0 + k) + lane - s;
                if (full || (i < n && j >= 0 && j <= i)) __builtin_nontemporal_store(v[K * u + k], row + j);
            }
        }
    };
    pass(std::integral_constant<int, NL>{}, 0);
    if (bi == bj) pass(std::integral_constant<int, 1>{}, NL);
}

// UTM: thread k owns cell utm_cell(k); no tile, no LDS.
template <int OP>
__global__ void __launch_bounds__(kUtmThreads) k_elem_utm(ElemArgs p, int64_t elements)
{
    const uint64_t k = ((uint64_t)blockIdx.y * gridDim.x + blockIdx.x) * kUtmThreads + threadIdx.x;
    if (k >= (uint64_t)elements) return;
    int32_t i, j;
    utm_cell(k, p.n, i, j);
    if ((uint32_t)i >= (uint32_t)p.n || (uint32_t)j > (uint32_t)i) return;
    const int64_t ld = p.ld;
    if constexpr (OP == TRI_OP_AXPYT_F32) {
        const float *X = (const float *)p.x;
        const float *Y = (const float *)p.y;
        ((float *)p.c)[(int64_t)i * ld + j] =
            __fadd_rn(__fmul_rn(p.a, X[(int64_t)i * ld + j]), Y[(int64_t)j * ld + i]);
    } else if constexpr (OP == TRI_OP_EDM4_F32) {
        const f4 *P = (const f4 *)p.x;
        ((float *)p.c)[(int64_t)i * ld + j] = __builtin_sqrtf(square4(P[i], P[j]));
    } else {
        const uint32_t *A = (const uint32_t *)p.x;
        const uint32_t *B = (const uint32_t *)p.y;
        ((int32_t *)p.c)[(int64_t)i * ld + j] =
            (int32_t)((A[i] ^ B[j]) + (uint32_t)i * (uint32_t)j);
    }
}

// How a launch moves rows (see the head of this file).
enum { kScalar = 0, kVector = 1, kStream = 2, kLines = 3, kStreamLong = 4 };

template <int OP, int MAP, int TILE, int ROWS>
static void launch_tile(const tri_plan *p, const ElemArgs &args, hipStream_t s)
{
    const dim3 grid(p->gx, p->gy);
    if constexpr (ROWS == kLines && OP != TRI_OP_AXPYT_F32) {
        static_assert(TILE >= 32, "whole lines");
        ElemArgs a = args;
        dim3 lines = grid;
        if constexpr (MAP == MAP_LAMBDA) grid_that_fits(a.g, 8 * TILE, lines);
        k_lines<OP, MAP, TILE><<<lines, 8 * TILE, 0, s>>>(a);
    } else {
        constexpr bool VECTOR = ROWS != kScalar;
        constexpr bool STREAM = ROWS == kStream || ROWS == kStreamLong;
        constexpr int NT = ElemShape<TILE, VECTOR>::NT;
        if constexpr (OP == TRI_OP_AXPYT_F32)
            k_axpyt<MAP, TILE, VECTOR, STREAM><<<grid, NT, 0, s>>>(args);
        else if constexpr (OP == TRI_OP_EDM4_F32)
            k_edm4<MAP, TILE, VECTOR, STREAM, ROWS != kStreamLong><<<grid, NT, 0, s>>>(args);
        else
            k_xormul<MAP, TILE, VECTOR, STREAM><<<grid, NT, 0, s>>>(args);
    }
}

template <int OP, int MAP, int ROWS>
static bool dispatch_tile(const tri_plan *p, const ElemArgs &args, hipStream_t s)
{
    // xormul and edm4 take lines from tile 32 and the other misaligned forms
    // below it
    constexpr bool big = OP == TRI_OP_AXPYT_F32 || ROWS >= kStream;
    if constexpr (ROWS != kLines) {
        switch (p->tile) {
        case 8: launch_tile<OP, MAP, 8, ROWS>(p, args, s); return true;
        case 16: launch_tile<OP, MAP, 16, ROWS>(p, args, s); return true;
        }
    }
    if constexpr (big) {
        switch (p->tile) {
        case 32: launch_tile<OP, MAP, 32, ROWS>(p, args, s); return true;
        case 64: launch_tile<OP, MAP, 64, ROWS>(p, args, s); return true;
        case 128: launch_tile<OP, MAP, 128, ROWS>(p, args, s); return true;
        }
    }
    return false;
}

template <int MAP, int TILE>
static void launch_axpyt_strip(const tri_plan *p, const ElemArgs &args, hipStream_t s)
{
    dim3 grid;
    const StripGrid sg = strip_grid(MAP, args.g.m, args.g.flags, args.g.T, p->gx, p->gy,
                                    strip_flag_len(p->flags), 1, grid);
    if constexpr (TILE == 16) {
        if (strip_band(p->flags)) k_axpyt_strip_quads<MAP><<<grid, 256, 0, s>>>(args, sg);
        else k_axpyt_strip_pairs<MAP><<<grid, 256, 0, s>>>(args, sg);
    } else
        k_axpyt_strip<MAP, TILE><<<grid, 256, 0, s>>>(args, sg);
}

template <int MAP>
static bool dispatch_axpyt_strip(const tri_plan *p, const ElemArgs &args, hipStream_t s)
{
    if (p->tile == 16) launch_axpyt_strip<MAP, 16>(p, args, s);
    else if (p->tile == 32) launch_axpyt_strip<MAP, 32>(p, args, s);
    else return false;
    return true;
}

template <int OP, int ROWS>
static bool dispatch_map(const tri_plan *p, const ElemArgs &args, hipStream_t s)
{
    switch (p->map) {
    case TRI_MAP_BB: return dispatch_tile<OP, MAP_BB, ROWS>(p, args, s);
    case TRI_MAP_RB: return dispatch_tile<OP, MAP_RB, ROWS>(p, args, s);
    case TRI_MAP_REC: return dispatch_tile<OP, MAP_REC, ROWS>(p, args, s);
    case TRI_MAP_LAMBDA: return dispatch_tile<OP, MAP_LAMBDA, ROWS>(p, args, s);
    }
    return false;
}

static bool axpyt_strips(const tri_plan *p, const ElemArgs &args, hipStream_t s)
{
    switch (p->map) {
    case TRI_MAP_BB: return dispatch_axpyt_strip<MAP_BB>(p, args, s);
    case TRI_MAP_RB: return dispatch_axpyt_strip<MAP_RB>(p, args, s);
    case TRI_MAP_REC: return dispatch_axpyt_strip<MAP_REC>(p, args, s);
    case TRI_MAP_LAMBDA: return dispatch_axpyt_strip<MAP_LAMBDA>(p, args, s);
    }
    return false;
}

template <int OP>
static bool dispatch_rows(const tri_plan *p, ElemArgs args, bool vector, bool lines, hipStream_t s)
{
    if (p->map == TRI_MAP_UTM) {
        k_elem_utm<OP><<<dim3(p->gx, p->gy), kUtmThreads, 0, s>>>(args, p->elements);
        return true;
    }
    // strips of tiles 16 and 32 (16-byte vectors, tile maps)
    if (OP == TRI_OP_AXPYT_F32 && vector && (p->tile == 16 || p->tile == 32) &&
        strip_flag_len(p->flags))
        return axpyt_strips(p, args, s);
    if (lines) {
        // matrices whose triangles take half of the memory-side cache (256 MB) at
        // most: cached accesses save a tenth (n = 2048, tile 32 4.9 -> 4.2 us, n =
        // 4096 18.0 -> 16.3; n = 8192, 400 MB, 77 -> 85)
        if (OP == TRI_OP_AXPYT_F32 && p->elements * 12 <= (128ll << 20))
            return dispatch_map<OP, kVector>(p, args, s);
        // outputs beyond the memory-side cache (256 MB): see k_edm4
        if constexpr (OP == TRI_OP_EDM4_F32)
            if (p->elements * 4 > (256ll << 20)) return dispatch_map<OP, kStreamLong>(p, args, s);
        return dispatch_map<OP, kStream>(p, args, s);
    }
    if (OP != TRI_OP_AXPYT_F32 && p->tile >= 32) return dispatch_map<OP, kLines>(p, args, s);
    if (p->map == TRI_MAP_LAMBDA) args.g = plan_tile_grid_swizzled(p);
    return vector ? dispatch_map<OP, kVector>(p, args, s) : dispatch_map<OP, kScalar>(p, args, s);
}

}  // namespace trimap

using namespace trimap;

extern "C" tri_status tri_launch_elementwise(const tri_plan *p, int op, const void *x,
                                             const void *y, void *c, int64_t ld, float a,
                                             void *stream)
{
    clear_error();
    if (!p) return fail(TRI_E_INVAL, "tri_launch_elementwise: plan is NULL");
    if (op != TRI_OP_XORMUL_I32 && op != TRI_OP_AXPYT_F32 && op != TRI_OP_EDM4_F32)
        return fail(TRI_E_INVAL, "tri_launch_elementwise: op = %d", op);
    if (!p->diag)
        return fail(TRI_E_UNSUPPORTED, "tri_launch_elementwise: needs include_diag = 1");
    if (p->tile > 128)
        return fail(TRI_E_UNSUPPORTED, "tri_launch_elementwise: tile %d > 128", p->tile);
    if (p->n == 0) return TRI_OK;
    if (!x || (!y && op != TRI_OP_EDM4_F32) || !c)
        return fail(TRI_E_INVAL, "tri_launch_elementwise: NULL buffer");
    if (ld < p->n) return fail(TRI_E_INVAL, "tri_launch_elementwise: ld %lld < n %lld",
                               (long long)ld, (long long)p->n);
    if (strip_band(p->flags) && strip_flag_len(p->flags) && strip_flag_len(p->flags) < 4)
        return fail(TRI_E_INVAL, "tri_launch_elementwise: two-row band strips need G >= 4 tiles");
    const uintptr_t cx = (uintptr_t)c, xx = (uintptr_t)x, yx = (uintptr_t)y;
    if ((cx | xx | yx) & 3) return fail(TRI_E_INVAL, "tri_launch_elementwise: unaligned buffer");
    if (op == TRI_OP_EDM4_F32 && (xx & 15))
        return fail(TRI_E_INVAL, "tri_launch_elementwise: EDM4 points need 16-byte alignment");
    bool vector = (ld % 4 == 0) && ((cx & 15) == 0);
    if (op == TRI_OP_AXPYT_F32) vector = vector && ((xx & 15) == 0) && ((yx & 15) == 0);

    ElemArgs args{plan_tile_grid(p), (int32_t)p->n, ld, x, y, c, a};
    hipStream_t s = (hipStream_t)stream;
    // every row of every matrix on a 128-byte line
    bool lines = ld % 32 == 0 && (cx & 127) == 0;
    if (op == TRI_OP_AXPYT_F32) lines = lines && ((xx | yx) & 127) == 0;
    bool ok;
    if (op == TRI_OP_AXPYT_F32) ok = dispatch_rows<TRI_OP_AXPYT_F32>(p, args, vector, lines, s);
    else if (op == TRI_OP_EDM4_F32) ok = dispatch_rows<TRI_OP_EDM4_F32>(p, args, vector, lines, s);
    else ok = dispatch_rows<TRI_OP_XORMUL_I32>(p, args, vector, lines, s);
    if (!ok) return fail(TRI_E_UNSUPPORTED, "tri_launch_elementwise: tile %d", p->tile);
    TRI_HIP(hipGetLastError());
    return TRI_OK;
}
