// Many generations of the Game of Life in the registers of one workgroup.
//
// NW waves hold a window of H rows x W cells as bits: lane (y, x) of LY x LX
// lanes of a wave keeps RR rows of the 64 cells 64 x .. of the window, two
// 32-bit words a row (W = 64 LX, H = NW LY RR, the waves' bands below each
// other).  In a generation the words left and right come from the
// neighbouring lanes by DPP; only the first and last row of each lane's band
// go through LDS to the bands above and below, with one barrier, while the
// band's other rows are computed.  After g generations every cell at least g cells inside the
// window is exact (the light cone of a cell grows by one cell a
// generation), whatever the lanes at the window's edges read; so the window
// yields the tile rows i0 .. i0 + h - 1, cells j0 .. j0 + w - 1 it was
// loaded around, for h <= H - 2 g and w <= W - PX - g, PX the cells left of
// j0 (a multiple of 16, at least g).
//
// Per word and generation: 2 shifts with the neighbour word, 1 DPP move, and
// 10 three-input operations.  With s = west + self + east per row (s0, s1),
// the nine-cell sum of a row is t0 + 2 (u1 + m1 + d1 + c0), (c0, t0) =
// u0 + m0 + d0 for the rows above (u), at (m) and below (d); a cell lives
// next iff the sum is 3, or 4 and it lives now (B3/S23).
//
// Rows move as 16-byte vectors: in round q the lanes of a quad load or store
// the four 16-cell chunks of the quad's lane q, and the packed chunks change
// hands by quad permutes.  With eight lanes a row, quad a's lane b holds column
// 2 b + a, so that the two quads of a round move 128 contiguous bytes, a whole
// line where the row's start allows it; the neighbouring columns are then
// in the other quad, three or four lanes away.  16-byte accesses need 4-byte
// alignment only, so every pitch the stencil takes (a multiple of 4, here at
// least 16) goes this way.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "bodies.hpp"

namespace trimap {

template <int LX, int RR, int NW>
struct LifeWindow {
    static constexpr int LY = 64 / LX;
    static constexpr int W = 64 * LX;       // cells
    static constexpr int HW = LY * RR;      // rows of a wave
    static constexpr int H = NW * HW;       // rows
    static constexpr int WORDS = 2 * 2 * NW * 64 * 2;  // LDS: two buffers of first and last rows
    static_assert((LX == 4 || LX == 8) && RR >= 2, "lane layout");
};

typedef uint32_t u32x4a4 __attribute__((ext_vector_type(4), aligned(4)));

template <int CTRL>
__device__ __forceinline__ uint32_t dpp32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}

// The word v of the lane that holds the column to the left / right (any
// word at a row's ends).  With eight lanes a row: banks 0 and 2 (quad 0 of a
// row) take one move, banks 1 and 3 the other.
template <int LX>
__device__ __forceinline__ uint32_t west_of(uint32_t v)
{
    if constexpr (LX == 4) return dpp32<0x111>(v);  // row_shr 1
    const int a = __builtin_amdgcn_update_dpp((int)v, (int)v, 0x103, 0xf, 0x5, false);  // row_shl 3
    return (uint32_t)__builtin_amdgcn_update_dpp(a, (int)v, 0x114, 0xf, 0xa, false);    // row_shr 4
}

template <int LX>
__device__ __forceinline__ uint32_t east_of(uint32_t v)
{
    if constexpr (LX == 4) return dpp32<0x101>(v);  // row_shl 1
    const int a = __builtin_amdgcn_update_dpp((int)v, (int)v, 0x104, 0xf, 0x5, false);  // row_shl 4
    return (uint32_t)__builtin_amdgcn_update_dpp(a, (int)v, 0x113, 0xf, 0xa, false);    // row_shr 3
}

// Lane q of each quad to the whole quad.
template <int Q>
__device__ __forceinline__ uint32_t quad_of(uint32_t v)
{
    return dpp32<Q * 0x55>(v);
}

// 16 cells (bytes 0 or 1) to 16 bits.
__device__ __forceinline__ uint32_t life_pack16(u32x4a4 v)
{
    const uint32_t a = __builtin_amdgcn_udot4(
        v.y, 0x80402010u, __builtin_amdgcn_udot4(v.x, 0x08040201u, 0u, false), false);
    const uint32_t b = __builtin_amdgcn_udot4(
        v.w, 0x80402010u, __builtin_amdgcn_udot4(v.z, 0x08040201u, 0u, false), false);
    return a | (b << 8);
}

// The inverse for the low 16 bits of b.
__device__ __forceinline__ u32x4a4 life_unpack16(uint32_t b)
{
    u32x4a4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        o[e] = __umul24((b >> (4 * e)) & 0xFu, 0x00204081u) & 0x01010101u;
    return o;
}

// Bits of the cells j <= gi of the word whose first cell is jb, for rows gi
// of the grid.
__device__ __forceinline__ uint32_t life_upto(int32_t gi, int32_t jb)
{
    const int32_t hi = gi - jb;
    const uint32_t m = 0xFFFFFFFFu >> (hi < 31 ? 31 - hi : 0);
    return hi < 0 ? 0u : m;
}

// Advances the cells j0 .. j0 + w - 1 of rows i0 .. i0 + h - 1 by `gens`
// generations (p.cur to p.nxt); px: cells loaded left of j0 (a multiple of
// 16); j0 a multiple of 16.  EDGE: some cell of the window lies outside the
// domain (or the grid): loads are clamped, cells outside the domain are
// cleared after staging and after every generation, and stores are tested.
// Called by every wave of the workgroup, each with the EDGE its own rows need
// (the barriers are the same number in both).  wv, lane: the wave's number and
// the lane's.  lds: S::WORDS words.
template <int LX, int RR, int NW, bool EDGE>
__device__ __forceinline__ void life_window_run(const LifeTile &p, int32_t i0, int32_t j0,
                                                int32_t h, int32_t w, int32_t px, int gens,
                                                int wv, int lane, uint32_t *lds)
{
    using S = LifeWindow<LX, RR, NW>;
    const int32_t n = p.n, ld = (int32_t)p.ld;
    const int x = lane & (LX - 1), y = lane / LX, q4 = lane & 3;
    // the first cell and row of the wave's part of the window
    const int32_t jw = j0 - px, iw = i0 - gens + wv * S::HW;
    const int32_t gi0 = iw + y * RR;             // this lane's first row
    // the chunk it moves in round q: cell jw + xq + kRound q of row gi0, at
    // byte `lane_at` + kRound q from the window's first
    constexpr int kRound = 16 * LX;
    const int32_t xq = 64 * (x >> 2) + 16 * q4;
    const int col_of = LX == 8 ? 2 * q4 + (x >> 2) : x;  // its column of 64 cells
    const uint32_t lane_at = (uint32_t)(y * RR) * (uint32_t)ld + (uint32_t)xq;
    const bool hi2 = (q4 & 2) != 0;

    uint32_t c[RR][2];
    {
        constexpr int RB = RR % 3 == 0 ? 3 : (RR % 2 == 0 ? 2 : 1);  // rows of loads in flight
        static_assert(RR % RB == 0, "load batches");
        const uint32_t psel = (q4 & 1) ? 0x07060302u : 0x05040100u;  // the odd / even halves
#pragma unroll
        for (int k0 = 0; k0 < RR; k0 += RB) {
            u32x4a4 v[RB][4];
#pragma unroll
            for (int k = 0; k < RB; ++k) {
                if constexpr (EDGE) {
                    const int32_t gi = gi0 + k0 + k;
                    const uint8_t *row = p.cur + (int64_t)(gi < 0 ? 0 : (gi >= n ? n - 1 : gi)) * ld;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int32_t jc = jw + xq + kRound * q;
                        v[k][q] =
                            *(const u32x4a4 *)(row + (jc < 0 ? 0 : (jc > ld - 16 ? ld - 16 : jc)));
                    }
                } else {
                    const uint8_t *row = p.cur + (int64_t)(iw + k0 + k) * ld + jw;  // (uniform)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        v[k][q] = *(const u32x4a4 *)(row + (lane_at + (uint32_t)(kRound * q)));
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < RB; ++k) {
                uint32_t b[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if constexpr (EDGE) {
                        b[q] = life_pack16(v[k][q] & 0x01010101u);
                        // a chunk that ends past the pitch was loaded early by
                        // as many cells
                        const int32_t late = jw + xq + kRound * q - (ld - 16);
                        b[q] >>= late < 0 ? 0 : (late > 16 ? 16 : late);
                    } else {
                        b[q] = life_pack16(v[k][q]);
                    }
                }
                // chunk q4 of the quad's lanes 0 .. 3 here; wanted: chunks 0 ..
                // 3 of this lane, chunk e from lane e of the quad, half q4 & 1
                // of its pair q4 >> 1 (every lane takes part in every move:
                // moved first, then chosen)
                const uint32_t p01 = b[0] | (b[1] << 16), p23 = b[2] | (b[3] << 16);
                const uint32_t l0 = quad_of<0>(p01), h0 = quad_of<0>(p23);
                const uint32_t l1 = quad_of<1>(p01), h1 = quad_of<1>(p23);
                const uint32_t l2 = quad_of<2>(p01), h2 = quad_of<2>(p23);
                const uint32_t l3 = quad_of<3>(p01), h3 = quad_of<3>(p23);
                const uint32_t e0 = hi2 ? h0 : l0, e1 = hi2 ? h1 : l1;
                const uint32_t e2 = hi2 ? h2 : l2, e3 = hi2 ? h3 : l3;
                c[k0 + k][0] = __builtin_amdgcn_perm(e1, e0, psel);
                c[k0 + k][1] = __builtin_amdgcn_perm(e3, e2, psel);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // bits of row k, word u that lie in the domain 0 <= j <= gi < n, for gi =
    // g0 + k (g0: gi0, hidden from the compiler in every generation, or it
    // would keep all the masks in registers)
    const int32_t jb = jw + 64 * col_of;  // first cell of the lane's first word
    const uint32_t left[2] = {jb >= 0 ? ~0u : (jb <= -32 ? 0u : ~0u << -jb),
                              jb >= -32 ? ~0u : (jb <= -64 ? 0u : ~0u << (-32 - jb))};
    const auto domain = [&](int32_t g0, int k, int u) {
        const uint32_t m = life_upto(g0 + k, jb + 32 * u) & left[u];
        return g0 + k < n ? m : 0u;
    };
    if constexpr (EDGE) {
        int32_t g0 = gi0;
        asm volatile("" : "+v"(g0));
#pragma unroll
        for (int k = 0; k < RR; ++k)
#pragma unroll
            for (int u = 0; u < 2; ++u) c[k][u] &= domain(g0, k, u);
    }

    struct Sum {
        uint32_t s0[2], s1[2];
    };
    const auto row_sum = [](const uint32_t (&r)[2]) {
        const uint32_t west = west_of<LX>(r[1]), east = east_of<LX>(r[0]);
        const uint32_t W[2] = {__builtin_amdgcn_alignbit(r[0], west, 31),
                               __builtin_amdgcn_alignbit(r[1], r[0], 31)};
        const uint32_t E[2] = {__builtin_amdgcn_alignbit(r[1], r[0], 1),
                               __builtin_amdgcn_alignbit(east, r[1], 1)};
        Sum s;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            s.s0[u] = __builtin_amdgcn_bitop3_b32(W[u], r[u], E[u], 0x96);  // parity
            s.s1[u] = __builtin_amdgcn_bitop3_b32(W[u], r[u], E[u], 0xE8);  // majority
        }
        return s;
    };
    const auto next = [](const Sum &a, const Sum &m, const Sum &d, int u, uint32_t self) {
        const uint32_t t0 = __builtin_amdgcn_bitop3_b32(a.s0[u], m.s0[u], d.s0[u], 0x96);
        const uint32_t c0 = __builtin_amdgcn_bitop3_b32(a.s0[u], m.s0[u], d.s0[u], 0xE8);
        const uint32_t e = __builtin_amdgcn_bitop3_b32(a.s1[u], m.s1[u], d.s1[u], 0x96);
        const uint32_t f = __builtin_amdgcn_bitop3_b32(a.s1[u], m.s1[u], d.s1[u], 0xE8);
        // the twos: e + 2 f + c0, their parity k
        const uint32_t k = e ^ c0;
        // sum 3: t0, k and not f; sum 4: neither t0 nor k, f differs from c0
        const uint32_t four = __builtin_amdgcn_bitop3_b32(f, c0, self, 0x28);  // (f ^ c0) & self
        const uint32_t z = __builtin_amdgcn_bitop3_b32(k, f, four, 0x3A);      // k ? ~f : four
        return __builtin_amdgcn_bitop3_b32(z, t0, k, 0x90);                    // z & ~(t0 ^ k)
    };
    // first (0) and last (1) rows of the bands, two buffers taken in turn, so
    // that one barrier a generation suffices; bands Y - 1 and Y + 1 are LX
    // lanes away (at the window's ends any lane will do)
    typedef uint32_t u32x2w __attribute__((ext_vector_type(2)));
    u32x2w *const ends = (u32x2w *)lds;
    const int me = 64 * wv + lane;
    const int prev = me >= LX ? me - LX : me, foll = me + LX < 64 * NW ? me + LX : me;
    for (int g = 0; g < gens; ++g) {
        int32_t g0 = gi0;
        if constexpr (EDGE && RR > 4) asm volatile("" : "+v"(g0));
        u32x2w *const buf = ends + (g & 1) * (2 * 64 * NW);
        buf[me] = u32x2w{c[0][0], c[0][1]};
        buf[64 * NW + me] = u32x2w{c[RR - 1][0], c[RR - 1][1]};
        const Sum s_first = row_sum(c[0]), s_second = row_sum(c[1]);
        Sum a = s_first, m = s_second;
#pragma unroll
        for (int k = 1; k + 1 < RR; ++k) {
            const Sum d = row_sum(c[k + 1]);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                c[k][u] = next(a, m, d, u, c[k][u]);
                if constexpr (EDGE) c[k][u] &= domain(g0, k, u);
            }
            a = m;
            m = d;
        }
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        const u32x2w va = buf[64 * NW + prev], vb = buf[foll];
        const uint32_t above[2] = {va.x, va.y}, below[2] = {vb.x, vb.y};
        const Sum s_above = row_sum(above), s_below = row_sum(below);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            c[RR - 1][u] = next(a, m, s_below, u, c[RR - 1][u]);
            if constexpr (EDGE) c[RR - 1][u] &= domain(g0, RR - 1, u);
            c[0][u] = next(s_above, s_first, s_second, u, c[0][u]);
            if constexpr (EDGE) c[0][u] &= domain(g0, 0, u);
        }
    }

    // store the tile's rows: round q, the chunks of the quad's lane q
    const int32_t k_lo = gens - wv * S::HW - y * RR, k_hi = k_lo + (i0 + h < n ? h : n - i0);
    const int sh = 16 * (q4 & 1);
    bool col[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) col[q] = xq + kRound * q >= px && xq + kRound * q < px + w;
#pragma unroll
    for (int k = 0; k < RR; ++k) {
        uint8_t *row = p.nxt + (int64_t)(iw + k) * ld + jw;  // (uniform)
        const bool in_rows = k >= k_lo && k < k_hi;
        const uint32_t lo[4] = {quad_of<0>(c[k][0]), quad_of<1>(c[k][0]), quad_of<2>(c[k][0]),
                                quad_of<3>(c[k][0])};
        const uint32_t hi[4] = {quad_of<0>(c[k][1]), quad_of<1>(c[k][1]), quad_of<2>(c[k][1]),
                                quad_of<3>(c[k][1])};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t b = (hi2 ? hi[q] : lo[q]) >> sh;
            if (!in_rows || !col[q]) continue;
            uint8_t *dst = row + (lane_at + (uint32_t)(kRound * q));
            if constexpr (EDGE) {
                const int32_t over = gi0 + k - (jw + xq + kRound * q);  // cells jc .. jc + over
                if (over >= 15) {
                    *(u32x4a4 *)dst = life_unpack16(b);
                } else {
                    for (int e = 0; e <= over; ++e) dst[e] = (uint8_t)((b >> e) & 1u);
                }
            } else {
                *(u32x4a4 *)dst = life_unpack16(b);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <int LX, int RR, int NW>
__device__ __forceinline__ void life_window_body(const LifeTile &p, int32_t i0, int32_t j0,
                                                 int32_t h, int32_t w, int32_t px, int gens,
                                                 int wv, int lane, uint32_t *lds)
{
    using S = LifeWindow<LX, RR, NW>;
    const int32_t jw = j0 - px, iw = i0 - gens + wv * S::HW;
    // every cell of the wave's rows is in the domain
    if (jw >= 0 && jw + S::W - 1 <= iw && iw + S::HW <= p.n)
        life_window_run<LX, RR, NW, false>(p, i0, j0, h, w, px, gens, wv, lane, lds);
    else
        life_window_run<LX, RR, NW, true>(p, i0, j0, h, w, px, gens, wv, lane, lds);
}

// Generations of one launch at most (on small grids the stencil takes more).
constexpr int kLifeWindowGen = 32;

// The tiling a window yields after `gens` generations: the largest G tiles of
// side h, in windows that start at multiples of 16 cells, px cells left of
// the tiles.
struct LifeWindowTiles {
    int32_t h, G, px;
};

template <int LX, int RR, int NW>
inline LifeWindowTiles life_window_tiles(int gens)
{
    using S = LifeWindow<LX, RR, NW>;
    LifeWindowTiles t{0, 0, (gens + 15) / 16 * 16};
    for (int32_t g = 1; g <= 4; ++g) {
        const int32_t step = g == 4 ? 4 : (g == 2 ? 8 : 16);
        const int32_t rows = S::H - 2 * gens, cols = (S::W - t.px - gens) / g;
        const int32_t side = (rows < cols ? rows : cols) / step * step;
        if ((int64_t)g * side * side > (int64_t)t.G * t.h * t.h) {
            t.G = g;
            t.h = side;
        }
    }
    return t;
}

}  // namespace trimap
