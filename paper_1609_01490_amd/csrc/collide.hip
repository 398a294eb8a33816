// Collision detection of n spheres (the shared-memory test of Section 5):
// every pair j < i of the strict lower triangle is tested once and, when the
// spheres overlap, counted for both of them.
//
// Tile maps (BB, RB, REC, lambda): tile (bi, bj) of the strict plan covers
// spheres 1 + bi rho .. (rows) against bj rho .. (columns).
//
// Overlaps are rare (a few per sphere), and the exact test costs 11 vector
// ALU operations per pair in 3-D, 5 in 1-D.  Tiles of 32, 64 and 128 first
// ask a question that never misses an overlap and costs far less per pair,
// and put the exact test only to the pairs that pass it: in 3-D a Gram
// product on the matrix cores (k_collide_gram), in 1-D the nearest of 16
// rows (k_collide_near).  The counts are those of the exact test alone.
// n = 131072, tile 128, lambda: 3-D 1.59 -> 0.30 ms, 1-D 0.80 -> 0.35 ms.
//
// Few spheres, and tiles of 8 and 16 (an MFMA block of 32 rows would be half
// or three quarters empty there), put the exact test to every pair
// (k_collide): both blocks of spheres are staged in LDS, each lane keeps RB
// row spheres in registers and walks CB column spheres read from LDS.
//
// Rows past n are staged as NaN so that they never overlap.
//
// UTM works in thread space: one lane per pair, both spheres read from
// global memory, no LDS (the map cannot form 2-D blocks).
#include "common.hpp"
#include "maps.hpp"

namespace trimap {

TileGrid plan_tile_grid(const tri_plan *p);

typedef float f4 __attribute__((ext_vector_type(4)));

struct CollideArgs {
    TileGrid g;
    int32_t n;
    const f4 *s;       // (x, y, z, r) per sphere
    int32_t *counts;
};

// Squared centre distance below the squared radius sum, binary32 with a
// fixed order (no fused multiply-add), strict comparison.
template <int DIM>
__device__ __forceinline__ bool overlap(f4 a, f4 b)
{
    const float dx = __fsub_rn(a.x, b.x);
    float s = __fmul_rn(dx, dx);
    if constexpr (DIM == 3) {
        const float dy = __fsub_rn(a.y, b.y), dz = __fsub_rn(a.z, b.z);
        s = __fadd_rn(s, __fmul_rn(dy, dy));
        s = __fadd_rn(s, __fmul_rn(dz, dz));
    }
    const float rr = __fadd_rn(a.w, b.w);
    return s < __fmul_rn(rr, rr);
}

template <int TILE>
struct CollideShape {
    static constexpr int NT = TILE * TILE < 256 ? TILE * TILE : 256;
    static constexpr int TX = TILE < 16 ? TILE : 16;  // lanes along columns
    static constexpr int TY = NT / TX;                // lanes along rows
    static constexpr int RB = TILE / TY;              // rows per lane
    static constexpr int CB = TILE / TX;              // columns per lane
    static_assert(RB * TY == TILE && CB * TX == TILE, "collide tile");
};

template <int MAP, int TILE, int DIM>
__global__ void __launch_bounds__((CollideShape<TILE>::NT)) k_collide(CollideArgs p)
{
    using S = CollideShape<TILE>;
    int32_t bi, bj;
    if (!tile_of_block<MAP>(p.g, bi, bj)) return;

    __shared__ f4 rows[TILE];
    __shared__ f4 cols[TILE];
    const int32_t n = p.n;
    const int32_t i0 = 1 + bi * TILE, j0 = bj * TILE;
    const float nan = __builtin_nanf("");
    for (int t = threadIdx.x; t < 2 * TILE; t += S::NT) {
        const int32_t k = t < TILE ? i0 + t : j0 + (t - TILE);
        const f4 v = k < n ? p.s[k] : f4{nan, nan, nan, nan};
        if (t < TILE) rows[t] = v;
        else cols[t - TILE] = v;
    }
    __syncthreads();

    const int ty = threadIdx.x / S::TX, tx = threadIdx.x % S::TX;
    f4 ri[S::RB];
#pragma unroll
    for (int a = 0; a < S::RB; ++a) ri[a] = rows[ty + S::TY * a];
    // First pass: only whether any pair of this lane overlaps (one lane-mask
    // OR per pair); overlaps are rare, so the second pass, which recounts
    // them with the diagonal test and the atomics, seldom runs.
    bool any = false;
#pragma unroll
    for (int b = 0; b < S::CB; ++b) {
        const f4 cj = cols[tx + S::TX * b];
#pragma unroll
        for (int a = 0; a < S::RB; ++a) any |= overlap<DIM>(ri[a], cj);
    }
    if (!any) return;
    const bool diag = (bi == bj);
#pragma unroll
    for (int b = 0; b < S::CB; ++b) {
        const int c = tx + S::TX * b;
        const f4 cj = cols[c];
#pragma unroll
        for (int a = 0; a < S::RB; ++a) {
            const int r = ty + S::TY * a;
            // j = j0 + c < i = 1 + j0 + r on a diagonal tile iff c <= r
            if (overlap<DIM>(ri[a], cj) && (!diag || c <= r)) {
                atomicAdd(&p.counts[i0 + r], 1);
                atomicAdd(&p.counts[j0 + c], 1);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Strips of the filtered kernels: a workgroup takes G tiles of the map
// (row-aligned under lambda, so a strip lies in one tile row; G grid columns
// of one grid row under BB, RB and REC) and walks them in runs of neighbours
// (one tile row, consecutive tile columns), whose columns are one contiguous
// range of spheres.  The rows are staged once per run of one tile row; wave
// w takes the run's columns 64 u .. 64 u + 63, u = w, w + 4, ..., one per
// lane.  Every tile is located by the map on its own.
// ---------------------------------------------------------------------------
constexpr int kCollideWaves = 4;
constexpr int kCollideThreads = 64 * kCollideWaves;

template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_of(float v)
{
    const int b = __builtin_bit_cast(int, v);
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(b, b, CTRL, ROWS, 0xf, false));
}

__device__ __forceinline__ float uniform(float v)
{
    return __builtin_bit_cast(float,
                              __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}

// Maximum over the wave (NaN ignored), in every lane.
__device__ __forceinline__ float wave_max(float v)
{
    v = fmaxf(v, dpp_of<0x111, 0xf>(v));  // row_shr 1, 2, 4, 8
    v = fmaxf(v, dpp_of<0x112, 0xf>(v));
    v = fmaxf(v, dpp_of<0x114, 0xf>(v));
    v = fmaxf(v, dpp_of<0x118, 0xf>(v));
    v = fmaxf(v, dpp_of<0x142, 0xa>(v));  // row_bcast 15, 31
    v = fmaxf(v, dpp_of<0x143, 0xc>(v));
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

// ---------------------------------------------------------------------------
// 3-D filter.  Centres are mapped to whole numbers q = rint(clamp((x - c) s))
// in [-1023, 1023]^3 (c and s from the row block's box) and radii to R =
// ceil(|r| s (1 + 2^-10)) + 1.  The clamp and the rounding are monotone and
// move a coordinate difference by at most one, so spheres that overlap have
//   |q_i - q_j| <= s |x_i - x_j| + sqrt(3) < R_i + R_j,
// i.e. the whole number
//   g = |q_i - q_j|^2 - (R_i + R_j)^2
//     = N_i + N_j - 2 (q_i . q_j + R_i R_j),   N = |q|^2 - R^2,
// is negative.  g is a product over eight terms, row (-2 q, -2 R, h, l, 2048,
// 1) by column (q, R, 2048, 1, h, l) with N = 2048 h + l: one
// v_mfma_f32_32x32x8_f16 gives it for 32 x 32 pairs, exactly (every factor
// is a whole number of at most 11 bits, every partial sum stays below 2^24).
// Only pairs with g < 0 take the exact test.
//
// R above 1000 (or not a number) would not fit: such a sphere gets q = R = 0,
// h = -2048, so that every pair of it passes.  Coordinates beyond 2^60 are
// left out of the box (they clamp to its faces).  The scale is at most
// 900 / max(half the box, largest row radius) and 0 when that maximum is
// below 2^-60, so that squares lost to underflow (differences below
// 2^-74) stay far below the slack 2 - sqrt(3); with scale 0 every pair
// passes.
//
// Per 64 columns and 128 rows: 8 MFMAs (256 cycles of the SIMD's matrix
// core) against about 35 vector operations for the columns' operands and 32
// three-input ORs of the signs; the exact test of every pair took about 1700
// vector operations.
// ---------------------------------------------------------------------------
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct CollideBox {
    float cx, cy, cz, s, sr;  // centre, scale, scale of the radii
};

__device__ __forceinline__ uint32_t pack_h2(float a, float b)
{
    return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(a, b));
}

// The eight terms of a sphere as two pairs of packed halves: lo = (f x, f y,
// f z, f R) with f = -2 for rows and 1 for columns, nm = (h, l).
template <bool ROW>
__device__ __forceinline__ void collide_terms(f4 v, const CollideBox &b, bool live, u32x2 &lo,
                                              uint32_t &nm)
{
    constexpr float kTop = 1023.f, f = ROW ? -2.f : 1.f;
    float x = __builtin_rintf(__builtin_amdgcn_fmed3f((v.x - b.cx) * b.s, -kTop, kTop));
    float y = __builtin_rintf(__builtin_amdgcn_fmed3f((v.y - b.cy) * b.s, -kTop, kTop));
    float z = __builtin_rintf(__builtin_amdgcn_fmed3f((v.z - b.cz) * b.s, -kTop, kTop));
    float R = __builtin_ceilf(__builtin_fmaf(__builtin_fabsf(v.w), b.sr, 1.f));
    const float N = __builtin_fmaf(x, x, __builtin_fmaf(y, y, __builtin_fmaf(z, z, -R * R)));
    float h = __builtin_floorf(N * (1.f / 2048.f));
    float l = __builtin_fmaf(-2048.f, h, N);
    const bool fits = R <= 1000.f && live;
    if (!__all(fits)) {  // (a branch of the wave: rare)
        x = fits ? x : 0.f;
        y = fits ? y : 0.f;
        z = fits ? z : 0.f;
        R = fits ? R : 0.f;
        // every pair passes / none with an ordinary sphere does
        h = fits ? h : (live ? -2048.f : 2047.f);
        l = fits ? l : 0.f;
    }
    lo.x = pack_h2(f * x, f * y);
    lo.y = pack_h2(f * z, f * R);
    nm = pack_h2(h, l);
}

constexpr uint32_t kTermsOne = 0x3c006800u;  // packed halves (2048, 1)

template <int MAP, int TILE>
__global__ void __launch_bounds__(kCollideThreads, 4) k_collide_gram(CollideArgs p, StripGrid sg)
{
    constexpr int NB = TILE / 32;  // row blocks
    __shared__ f4 rows[TILE];
    __shared__ u32x4 terms[TILE];
    __shared__ float red[2][8];
    __shared__ int32_t hits[kCollideWaves][TILE];  // a wave's overlaps per row of a block

    const int t = threadIdx.x, l = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int32_t n = p.n;
    const float nan = __builtin_nanf("");
    const uint32_t first = strip_first<MAP>(p.g, sg);
    int32_t staged = -1;
    CollideBox box{};
    h4 A[NB];

    for (int k = 0; k < sg.G;) {
        int32_t bi, bj;
        if (MAP == MAP_BB && first + (uint32_t)k > blockIdx.y) return;  // above the diagonal
        k = strip_next<MAP>(p.g, sg, first, k, bi, bj);
        if (k >= sg.G) return;  // uniform over the workgroup
        bi = __builtin_amdgcn_readfirstlane(bi);
        bj = __builtin_amdgcn_readfirstlane(bj);
        const int len = strip_run<MAP>(p.g.m, sg, (int32_t)first + k, (int32_t)blockIdx.y, k, bi, bj);
        k += len;
        const int32_t i0 = 1 + bi * TILE;
        if (bi != staged) {
            if (staged >= 0) __syncthreads();  // the previous run is done with the LDS
            staged = bi;
            f4 v{nan, nan, nan, nan};
            if (t < TILE && i0 + t < n) v = p.s[i0 + t];
            if (t < TILE) rows[t] = v;
            if (w < (TILE + 63) / 64) {
                const float far = 0x1p60f, none = -3.0e38f;
                const bool ux = __builtin_fabsf(v.x) < far, uy = __builtin_fabsf(v.y) < far,
                           uz = __builtin_fabsf(v.z) < far;
                const float m0 = wave_max(ux ? v.x : none), m1 = wave_max(ux ? -v.x : none);
                const float m2 = wave_max(uy ? v.y : none), m3 = wave_max(uy ? -v.y : none);
                const float m4 = wave_max(uz ? v.z : none), m5 = wave_max(uz ? -v.z : none);
                const float m6 = wave_max(fmaxf(__builtin_fabsf(v.w), 0.f));
                if (l == 0) {
                    red[w][0] = m0; red[w][1] = m1; red[w][2] = m2; red[w][3] = m3;
                    red[w][4] = m4; red[w][5] = m5; red[w][6] = m6;
                }
            }
            __syncthreads();
            float m[7];
#pragma unroll
            for (int q = 0; q < 7; ++q)
                m[q] = uniform(TILE > 64 ? fmaxf(red[0][q], red[1][q]) : red[0][q]);
            // an axis without a usable coordinate has m = none twice: a
            // negative extent, centre 0
            box.cx = 0.5f * (m[0] - m[1]);
            box.cy = 0.5f * (m[2] - m[3]);
            box.cz = 0.5f * (m[4] - m[5]);
            const float half = 0.5f * fmaxf(fmaxf(m[0] + m[1], m[2] + m[3]), m[4] + m[5]);
            const float big = fmaxf(fmaxf(half * (9.f / 8.f), m[6]), 0.f);
            box.s = uniform(big >= 0x1p-60f ? 900.f / big : 0.f);  // (900 / infinity = 0)
            box.sr = uniform(box.s * (1.f + 0x1p-10f));
            box.cx = uniform(box.cx);
            box.cy = uniform(box.cy);
            box.cz = uniform(box.cz);
            if (t < TILE) {
                u32x2 lo;
                uint32_t nm;
                collide_terms<true>(v, box, i0 + t < n, lo, nm);
                terms[t] = u32x4{lo.x, lo.y, nm, kTermsOne};
            }
            __syncthreads();
#pragma unroll
            for (int a = 0; a < NB; ++a)
                A[a] = __builtin_bit_cast(h4, ((const u32x2 *)&terms[32 * a + (l & 31)])[l >> 5]);
        }

        // the run's columns, 64 per wave and step, one per lane
        const int32_t c0 = bj * TILE, c1 = min(c0 + len * TILE, n);
        int32_t cb = c0 + 64 * w;
        f4 cv = cb + l < c1 ? p.s[cb + l] : f4{nan, nan, nan, nan};
        for (; cb < c1; cb += kCollideThreads) {
            u32x2 lo;
            uint32_t nm;
            collide_terms<false>(cv, box, l < c1 - cb, lo, nm);
            // the next step's columns, in flight during the products
            const int32_t nb = cb + kCollideThreads < c1 ? cb + kCollideThreads : cb;
            cv = (p.s + nb)[min(l, c1 - 1 - nb)];
            // half 0 of a block's operand: (q, R) of column l; half 1: (2048,
            // 1, h, l) of column l - 32: the swap of lane halves gives
            // columns 0..31 and 32..63
            const auto s0 = __builtin_amdgcn_permlane32_swap(lo.x, kTermsOne, false, false);
            const auto s1 = __builtin_amdgcn_permlane32_swap(lo.y, nm, false, false);
#pragma unroll 1
            for (int b = 0; b < 2; ++b) {  // (both at once would hold 128 accumulators)
                const h4 B = __builtin_bit_cast(h4, b ? u32x2{s0[1], s1[1]} : u32x2{s0[0], s1[0]});
                f32x16 g[NB];
                uint32_t neg[NB], any = 0;
#pragma unroll
                for (int a = 0; a < NB; ++a)
                    g[a] = __builtin_amdgcn_mfma_f32_32x32x8f16(A[a], B, f32x16{}, 0, 0, 0);
#pragma unroll
                for (int a = 0; a < NB; ++a) {
                    // three-input ORs as v_bitop3, which two waves can issue
                    // together (v_or3 cannot)
                    neg[a] = __float_as_uint(g[a][0]) | __float_as_uint(g[a][1]);
#pragma unroll
                    for (int r = 2; r < 16; r += 2)
                        neg[a] = __builtin_amdgcn_bitop3_b32(neg[a], __float_as_uint(g[a][r]),
                                                             __float_as_uint(g[a][r + 1]), 0xfe);
                    any |= neg[a];
                }
                if (!__any((int32_t)any < 0)) continue;
                // rare: the exact test of the pairs that passed, each lane its own
                const int32_t j = cb + 32 * b + (l & 31);
                const bool live = j < c1;
                const f4 cj = p.s[live ? j : cb];
                int r0 = 4 * (l >> 5);
                asm volatile("" : "+v"(r0));  // (no address of this path is worth a register outside it)
                uint64_t m = 0;  // bit 16 a + r: the pair of row block a, register r passed
#pragma unroll
                for (int a = 0; a < NB; ++a) {
                    if (!__any((int32_t)neg[a] < 0)) continue;
                    uint32_t ma = 0;
#pragma unroll
                    for (int r = 15; r >= 0; --r)
                        ma = __builtin_amdgcn_alignbit(ma, __float_as_uint(g[a][r]), 31);
                    m |= (uint64_t)ma << (16 * a);
                }
                if (!live) m = 0;
                // Where nearly all lanes have some, the rows' overlaps are counted in
                // the wave's own LDS and added to the counts once per block.  (Two
                // additions to memory for each overlap, nearly all pairs
                // overlapping: n = 1000, tile 128 733 us, in this form 43; the
                // exact test of every pair takes 280.  From 16 lanes on, blocks with
                // a few overlaps took it too: n = 300 to 5000, four per sphere 7.7 ->
                // 8.1 us; n = 9300, 194 per sphere 74 -> 25.)
                if (__builtin_expect(__builtin_popcountll(__ballot(m != 0)) > 56, 0)) {
                    for (int q = l; q < TILE; q += 64) hits[w][q] = 0;
                    __builtin_amdgcn_wave_barrier();
                    int32_t mine = 0;
                    while (m) {
                        const int k = __builtin_ctzll(m), r = k & 15;
                        m &= m - 1;
                        const int row = 32 * (k >> 4) + 8 * (r >> 2) + (r & 3) + r0;
                        if (j < i0 + row && overlap<3>(rows[row], cj)) {
                            atomicAdd(&hits[w][row], 1);
                            ++mine;
                        }
                    }
                    if (mine) atomicAdd(&p.counts[j], mine);
                    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the wave's additions
                    __builtin_amdgcn_wave_barrier();
                    for (int q = l; q < TILE; q += 64)
                        if (const int32_t c = hits[w][q]) atomicAdd(&p.counts[i0 + q], c);
                    continue;
                }
                while (m) {
                    const int k = __builtin_ctzll(m), r = k & 15;
                    m &= m - 1;
                    const int row = 32 * (k >> 4) + 8 * (r >> 2) + (r & 3) + r0;
                    if (j < i0 + row && overlap<3>(rows[row], cj)) {
                        atomicAdd(&p.counts[i0 + row], 1);
                        atomicAdd(&p.counts[j], 1);
                    }
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// 1-D filter.  Centre differences as the exact test takes them, t = fl(x_i -
// x_j): fl(t^2) < fl(rr^2) implies |t| < |rr|, and |rr| = |fl(r_i + r_j)| is
// at most (|r_j| + the rows' largest |r|) (1 + 2^-20).  A lane keeps the
// smallest |t| of 16 rows against its column (two subtractions and one
// three-input minimum per two rows) and the 16 rows take the exact test only
// when some lane's minimum is below its bound.
// ---------------------------------------------------------------------------
template <int MAP, int TILE>
__global__ void __launch_bounds__(kCollideThreads) k_collide_near(CollideArgs p, StripGrid sg)
{
    __shared__ f4 rows[TILE];
    __shared__ __attribute__((aligned(16))) float xs[TILE];
    __shared__ float red[2];

    const int t = threadIdx.x, l = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int32_t n = p.n;
    const float nan = __builtin_nanf(""), inf = __builtin_inff();
    const uint32_t first = strip_first<MAP>(p.g, sg);
    int32_t staged = -1;
    float rmax = 0.f;

    for (int k = 0; k < sg.G;) {
        int32_t bi, bj;
        if (MAP == MAP_BB && first + (uint32_t)k > blockIdx.y) return;  // above the diagonal
        k = strip_next<MAP>(p.g, sg, first, k, bi, bj);
        if (k >= sg.G) return;  // uniform over the workgroup
        bi = __builtin_amdgcn_readfirstlane(bi);
        bj = __builtin_amdgcn_readfirstlane(bj);
        const int len = strip_run<MAP>(p.g.m, sg, (int32_t)first + k, (int32_t)blockIdx.y, k, bi, bj);
        k += len;
        const int32_t i0 = 1 + bi * TILE;
        if (bi != staged) {
            if (staged >= 0) __syncthreads();  // the previous run is done with the LDS
            staged = bi;
            f4 v{nan, nan, nan, nan};
            if (t < TILE && i0 + t < n) v = p.s[i0 + t];
            if (t < TILE) {
                rows[t] = v;
                xs[t] = v.x;
            }
            if (w < (TILE + 63) / 64) {
                const float m = wave_max(fmaxf(__builtin_fabsf(v.w), 0.f));
                if (l == 0) red[w] = m;
            }
            __syncthreads();
            rmax = TILE > 64 ? fmaxf(red[0], red[1]) : red[0];
        }
        const int32_t c0 = bj * TILE, c1 = min(c0 + len * TILE, n);
        int32_t cb = c0 + 64 * w;
        f4 cv = cb + l < c1 ? p.s[cb + l] : f4{nan, nan, nan, nan};
        for (; cb < c1; cb += kCollideThreads) {
            const f4 cj = cv;
            const int32_t j = cb + l;
            const int32_t nc = j + kCollideThreads;
            cv = nc < c1 ? p.s[nc] : f4{nan, nan, nan, nan};
            const float bound = (__builtin_fabsf(cj.w) + rmax) * (1.f + 0x1p-20f);
#pragma unroll 1
            for (int r0 = 0; r0 < TILE; r0 += 16) {
                float m = inf;
#pragma unroll
                for (int r = 0; r < 16; r += 4) {
                    const f4 x = *(const f4 *)&xs[r0 + r];
                    const float t0 = __fsub_rn(x.x, cj.x), t1 = __fsub_rn(x.y, cj.x);
                    const float t2 = __fsub_rn(x.z, cj.x), t3 = __fsub_rn(x.w, cj.x);
                    m = fminf(fminf(__builtin_fabsf(t0), __builtin_fabsf(t1)), m);
                    m = fminf(fminf(__builtin_fabsf(t2), __builtin_fabsf(t3)), m);
                }
                if (!__any(m < bound)) continue;
                // the rows that may overlap this lane's column (the sign of
                // s - rr^2), then the exact test of those
                uint32_t pass = 0;
#pragma unroll
                for (int r = 15; r >= 0; --r) {
                    const f4 ri = rows[r0 + r];
                    const float t = __fsub_rn(ri.x, cj.x), rr = __fadd_rn(ri.w, cj.w);
                    const float d = __fsub_rn(__fmul_rn(t, t), __fmul_rn(rr, rr));
                    pass = __builtin_amdgcn_alignbit(pass, __float_as_uint(d), 31);
                }
                while (pass) {
                    const int r = r0 + __builtin_ctz(pass);
                    pass &= pass - 1;
                    if (j < i0 + r && overlap<1>(rows[r], cj)) {
                        atomicAdd(&p.counts[i0 + r], 1);
                        atomicAdd(&p.counts[j], 1);
                    }
                }
            }
        }
    }
}

template <int DIM>
__global__ void __launch_bounds__(kUtmThreads) k_collide_utm(CollideArgs p, int64_t side,
                                                             int64_t pairs)
{
    const uint64_t k = ((uint64_t)blockIdx.y * gridDim.x + blockIdx.x) * kUtmThreads + threadIdx.x;
    if (k >= (uint64_t)pairs) return;
    int32_t i, j;
    utm_cell(k, side, i, j);
    i += 1;  // strict triangle of side n = diagonal-including triangle of side n - 1, shifted
    if ((uint32_t)i >= (uint32_t)p.n || (uint32_t)j >= (uint32_t)i) return;
    if (overlap<DIM>(p.s[i], p.s[j])) {
        atomicAdd(&p.counts[i], 1);
        atomicAdd(&p.counts[j], 1);
    }
}

__global__ void __launch_bounds__(256) k_zero_i32(int32_t *v, int64_t count)
{
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k < count) v[k] = 0;
}

// Tiles per strip of the filtered kernels: at least one step of 64 columns for
// each of a workgroup's waves, and longer strips (which stage their rows once)
// while they still fill the GPU: 1.5 rounds of the 1024 workgroups of
// k_collide_gram that are resident at once (measured in 3-D at tile 128: n =
// 20000, 12403 tiles, 4 / 8 / 16 / 32 tiles a strip 27.7 / 24.5 / 23.2 / 31.0
// us; n = 50000, 76636 tiles, 16 / 32 / 64 71.8 / 70.6 / 78.9 us; n = 131072,
// 524800 tiles, 32 / 64 314 / 295 us).
static int32_t collide_strip_len(const tri_plan *p)
{
    int32_t G = 64;
    while (G > kCollideThreads / p->tile && p->T / G < 1536) G /= 2;
    return p->map == TRI_MAP_LAMBDA ? strip_len_that_fits((int32_t)p->m, G, kCollideThreads) : G;
}

template <int MAP, int TILE, int DIM>
static void collide_filtered(const tri_plan *p, const CollideArgs &a0, hipStream_t s)
{
    CollideArgs a = a0;
    // row-aligned strips in the plan's workgroup order
    a.g.flags = (p->flags & (TRI_FLAG_XCD_SWIZZLE | TRI_FLAG_ORDER_REVERSE | TRI_FLAG_ORDER_PAIRS)) |
                TRI_FLAG_STRIP_ALIGN;
    dim3 grid;
    const StripGrid sg = strip_grid(MAP, a.g.m, a.g.flags, a.g.T, p->gx, p->gy,
                                    collide_strip_len(p), 1, grid);
    if constexpr (DIM == 3) k_collide_gram<MAP, TILE><<<grid, kCollideThreads, 0, s>>>(a, sg);
    else k_collide_near<MAP, TILE><<<grid, kCollideThreads, 0, s>>>(a, sg);
}

// Whether a plan takes the filtered kernels: where they are faster.  On few
// spheres a launch lasts a few microseconds either way and the filter's
// longer chain (box, terms, product, test) loses to one exact test of every
// pair.  Measured, exact against filtered (us, lambda): 3-D tile 64 n = 3000
// 6.0 / 8.0, 8000 13.7 / 13.6, 12000 22.9 / 17.4; tile 32 n = 3000 6.8 / 8.6,
// 8000 20.0 / 15.1; tile 128 n = 1000 10.0 / 7.7, 20000 59.6 / 24.1; 1-D tile
// 64 n = 9000 11.8 / 14.8, 12000 16.9 / 17.0, 20000 35.8 / 26.7; tile 128
// n = 8000 11.3 / 12.4, 20000 34.3 / 26.8; tile 32 n = 7000 14.0 / 15.3 (3-D 14.8 /
// 15.4), 8000 17.9 / 15.0.  The other maps cross at the same sizes or below (tile
// 32, 1-D: RB n = 6200 11.7 / 13.9, 7000 12.9 / 12.9, BB 7000 16.2 / 10.3).
static bool collide_filters(const tri_plan *p, int dim)
{
    switch (p->tile) {
    case 32: return p->n >= 7424;
    case 64: return p->n >= (dim == 3 ? 9216 : 13312);
    case 128: return dim == 3 || p->n >= 13312;
    }
    return false;
}

template <int MAP, int TILE, int DIM>
static void collide_launch(const tri_plan *p, const CollideArgs &a, hipStream_t s)
{
    if constexpr (TILE >= 32) {
        if (collide_filters(p, DIM)) return collide_filtered<MAP, TILE, DIM>(p, a, s);
    }
    if constexpr (TILE < 128 || DIM == 1)
        k_collide<MAP, TILE, DIM><<<dim3(p->gx, p->gy), CollideShape<TILE>::NT, 0, s>>>(a);
}

template <int MAP, int DIM>
static bool collide_tile(const tri_plan *p, const CollideArgs &a, hipStream_t s)
{
    switch (p->tile) {
    case 8: collide_launch<MAP, 8, DIM>(p, a, s); return true;
    case 16: collide_launch<MAP, 16, DIM>(p, a, s); return true;
    case 32: collide_launch<MAP, 32, DIM>(p, a, s); return true;
    case 64: collide_launch<MAP, 64, DIM>(p, a, s); return true;
    case 128: collide_launch<MAP, 128, DIM>(p, a, s); return true;
    }
    return false;
}

template <int DIM>
static bool collide_map(const tri_plan *p, const CollideArgs &a, hipStream_t s)
{
    switch (p->map) {
    case TRI_MAP_BB: return collide_tile<MAP_BB, DIM>(p, a, s);
    case TRI_MAP_RB: return collide_tile<MAP_RB, DIM>(p, a, s);
    case TRI_MAP_REC: return collide_tile<MAP_REC, DIM>(p, a, s);
    case TRI_MAP_LAMBDA: return collide_tile<MAP_LAMBDA, DIM>(p, a, s);
    case TRI_MAP_UTM:
        k_collide_utm<DIM><<<dim3(p->gx, p->gy), kUtmThreads, 0, s>>>(a, p->ne, p->elements);
        return true;
    }
    return false;
}

}  // namespace trimap

using namespace trimap;

extern "C" tri_status tri_collide(const tri_plan *p, const float *spheres, int dim,
                                  int32_t *counts, void *stream)
{
    clear_error();
    if (!p) return fail(TRI_E_INVAL, "tri_collide: plan is NULL");
    if (p->diag) return fail(TRI_E_INVAL, "tri_collide: the plan must exclude the diagonal");
    if (dim != 1 && dim != 3) return fail(TRI_E_INVAL, "tri_collide: dim = %d", dim);
    if (p->tile > 128) return fail(TRI_E_UNSUPPORTED, "tri_collide: tile %d > 128", p->tile);
    if (p->n == 0) return TRI_OK;
    if (!spheres || !counts) return fail(TRI_E_INVAL, "tri_collide: NULL buffer");
    if ((uintptr_t)spheres & 15)
        return fail(TRI_E_INVAL, "tri_collide: spheres need 16-byte alignment");
    if ((uintptr_t)counts & 3) return fail(TRI_E_INVAL, "tri_collide: unaligned counts");
    hipStream_t s = (hipStream_t)stream;
    k_zero_i32<<<dim3((uint32_t)((p->n + 255) / 256)), 256, 0, s>>>(counts, p->n);
    TRI_HIP(hipGetLastError());
    if (p->n < 2) return TRI_OK;
    CollideArgs a{plan_tile_grid(p), (int32_t)p->n, (const f4 *)spheres, counts};
    const bool ok = dim == 3 ? collide_map<3>(p, a, s) : collide_map<1>(p, a, s);
    if (!ok) return fail(TRI_E_UNSUPPORTED, "tri_collide: tile %d", p->tile);
    TRI_HIP(hipGetLastError());
    return TRI_OK;
}
