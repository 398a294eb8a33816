// Distance-map tiles on the matrix cores with FP32's accuracy, for the single
// domain's kernel and the batched queue.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "bodies.hpp"

namespace trimap {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// The squared distance of two points, summed in the order of the dimensions
// with the loads of eight in flight.
__device__ __forceinline__ float direct_d2_wide(const float *x, int64_t ldx, int32_t d, int32_t i,
                                                int32_t j)
{
    const float *xi = x + (int64_t)i * ldx, *xj = x + (int64_t)j * ldx;
    float s = 0.f;
    int32_t k = 0;
    for (; k + 8 <= d; k += 8) {
        float a[8], b[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            a[u] = xi[k + u];
            b[u] = xj[k + u];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float df = a[u] - b[u];
            s = __builtin_fmaf(df, df, s);
        }
    }
    for (; k < d; ++k) {
        const float df = xi[k] - xj[k];
        s = __builtin_fmaf(df, df, s);
    }
    return s;
}

// Workgroup barrier that orders LDS traffic only: wait for this wave's LDS
// operations, then s_barrier.  Unlike __syncthreads() it does not wait for
// outstanding global stores or prefetch loads.  (A global load that feeds
// LDS is waited for by the data dependency of the LDS store.)
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0), vmcnt and expcnt untouched
    __builtin_amdgcn_s_barrier();
}

// ---------------------------------------------------------------------------
// The FP32 mode on the matrix cores (from kGramMinDims dimensions on, tiles of
// 64 and 128; no workspace, one launch).
//
// d^2 = |y_i|^2 + |y_j|^2 - 2 y_i.y_j with y = sc (x - c): c is the mean of 16
// of the tile's own points, so that the norms are no larger than the tile's
// spread, and sc the power of two that brings those points' spread to 2^8.  sc c
// is rounded to a multiple of 4 (at most 1/128 of the spread): coordinates on a
// grid of a power of two (pixels, counts, flags) stay on it, or on a grid of 4,
// and where the norms' sum is below 2^24 grid squares every sum here is exact and
// the distance the correctly rounded one, as the direct sum's is (the plain mean
// of 16 put pixels off their grid: d = 32 33000 of 530000 distances wrongly
// rounded, d = 784 all but a few).
// The norms are FP32 sums of the squares of y.  The products take y as two
// FP16 values, h + l (23 significant bits or 2^-25; spreads up to 2^7 times the
// samples' fit, see the norm test): h.l + l.h + h.h accumulated in FP32 by
// v_mfma_f32_32x32x16_f16.
//
// Error.  Rounding leaves about 2^-24 (|y_i|^2 + |y_j|^2) in d^2, whatever d,
// while the direct sum's error grows with d.  A pair with d^2 below 3/8 of
// that sum (from 128 dimensions on 1/2), or with a sum that is no finite number well inside FP32's range, is
// recomputed from the differences in the direct body's order.  So is a pair whose
// sum is small in scaled units: a coordinate below 1/4 keeps 2^-25 in its halves
// and no relative precision, which adds up to 2^-24 sqrt(2 d S) to d^2, S the sum
// of the scaled norms.  Points that were no samples can be that much closer
// together than the samples (a few wide outliers among these, or samples that are
// all zeros: errors of 1e-4 and more without this).  From S = kGramFloor d /
// 1.625 on it is at most 0.64 of 2^-24 S; points spread as the samples have S of
// about 10^4 d.
//
// In units of 2^-24 S the rest is at most d / 8 + 4 for the norms' sums, 4 for the
// coordinates' rounding, 4 for their halves' (2^-23 of a coordinate), 4 for the
// product l.l that is left out, and 3 d / 16 for the products' sums (one rounding
// per instruction): with S <= 8/3 d^2 a distance is within (5 d / 12 + 24) 2^-24 of
// the exact one relative to it, near pairs within the direct sum's (d / 2 + 2)
// 2^-24, which is the smaller bound up to d = 264.  These bounds are far off: what
// is found, against 64 bits, uniform points with 1 % near-duplicates, relative
// L2 and largest relative error, direct / here, is
// 4.6e-8 / 3.9e-8 and 2.4e-7 / 2.6e-7 at d = 24, 5.2e-8 / 3.9e-8 and 2.9e-7 /
// 2.4e-7 at d = 32, 6.4e-8 / 3.4e-8 and 3.7e-7 / 2.2e-7 at d = 63, 9.2e-8 /
// 4.0e-8 and 4.8e-7 / 2.6e-7 at d = 128, 1.3e-7 / 3.5e-8 and 6.4e-7 / 2.5e-7 at
// d = 256; d = 128 in clusters of 0.6 times their centres' spread 9.1e-8 /
// 4.0e-8 and 4.5e-7 / 3.7e-7.  Hence the line at 32: below it the largest error
// would be larger than the direct sum's.  Normal points are like it; unit vectors'
// and fourth powers' largest error is up to 6 % above it at d = 32 and 40.  On log-normal, Laplace and half-normal ones the largest error of 8 million pairs
// is up to a quarter larger than the direct sum's below d = 64 (4.6e-7 against
// 3.8e-7, log-normal, d = 40), and on features that are mostly zeros, few of
// whose terms round in the direct sum, it is larger up to d = 127 (a normal variable
// less 0.8, cut at zero, L2 and largest): d = 32 3.8e-8 / 3.8e-8 and 2.2e-7 /
// 3.9e-7, d = 40, the worst found, 4.0e-8 / 3.8e-8 and 2.2e-7 / 4.1e-7, d = 63 4.5e-8 /
// 3.7e-8 and 2.6e-7 / 3.5e-7, d = 96 5.3e-8 / 3.8e-8 and 3.1e-7 / 3.3e-7; less 1.5, d =
// 50 3.3e-8 / 3.4e-8 and 1.9e-7 / 3.5e-7, d = 127 4.1e-8 / 3.9e-8 and 2.4e-7 / 3.3e-7.
// With the wider near line from 128 dimensions on neither was larger on any of these
// (tried at d = 128, 200, 256 and 400).
//
// A tile with many pairs to recompute is left to the direct body, most of the
// time after 32 dimensions.  Where every tile is (ten tight clusters in random
// order), that costs what was tried before: n = 16384 against the direct form
// alone, tile 128 d = 128 715 -> 835 us, d = 64 410 -> 485, tile 64 780 -> 912 and 433 ->
// 543; from about sixty clusters on the products win again (tile 128, d = 128 720 ->
// 618, a hundred 485).  In four quarters of 64 x 64 tile 128's direct body took 970
// us, without the early test 1130.
//
// Work.  The direct form is bound by two vector operations per pair and
// dimension.  Here they are about 5 per staged coordinate and 10 per pair, and
// with the products (half as long, on the matrix cores, partly in their shadow)
// and the power limit's clock they bound the kernel (n = 65536, d = 128: the vector
// units busy 72 % of the cycles, the matrix cores 25 %).  n = 16384: d = 128 706 ->
// 234 us (tile 128) and 770 -> 288 us (tile 64), d = 64 404 -> 172 us; n = 10007,
// d = 256 515 -> 143 us; n = 2000, d = 128 26.0 -> 11.4 us.  Below d = 64 against
// the direct form as it is now, tile 64 / 128: n = 16384, d = 32 247 -> 172 /
// 233 -> 158 us, d = 50 379 -> 201 / 380 -> 174 us; n = 257, d = 32 6.8 -> 6.3 /
// 16.0 -> 9.0 us; n = 2000, d = 32 9.9 -> 10.1 / 17.4 -> 10.1 us.  Tried in its place,
// d = 128: FP32 products (v_mfma_f32_32x32x2_f32, which shares the vector
// units: no overlap) 358 us; three BF16 parts, six products, 288 us.
//
// Layout.  16 dimensions at a time, two buffers, one barrier per chunk: a chunk
// is centred, split and stored while the products of the one before it run.
// Rows are 32 bytes; the two 16-byte slots of a row are swapped every eight
// rows, so that the 16-byte reads of 16 rows fall on distinct banks.  Waves have
// 64 x 32 pairs (tile 64: 32 x 32) and two workgroups share a CU.  The outputs
// are cached, neighbouring tiles on one XCD: the parts of a line that two waves
// or two tiles write meet in its L2 (d = 64: 288 -> 172 us; either alone 209 and
// 267 us).
// ---------------------------------------------------------------------------
constexpr int kGramMinDims = 32;
// The near line, of the norms' sum: 3/8, and from 128 dimensions on, where such pairs
// are rare on ordinary data, 1/2, which costs nothing there (d = 128 223 -> 224 us, d
// = 64 160 -> 176, d = 32 146 -> 169, the batch's d = 32 8 %).
constexpr float kGramNear = 0.375f, kGramNearWide = 0.5f;
constexpr int kGramWideDims = 128;
constexpr float kGramFloor = 8.f;  // per dimension, on d^2 in scaled units
constexpr int kGramK = 16;         // dimensions per staged chunk
constexpr int kGramLaneNear = 4;   // near pairs per lane (of 32 or 16) that a tile may hold

template <int TILE>
struct GramLds {
    static constexpr int kPlane = TILE * kGramK * 2;  // bytes
    static constexpr int kBuffer = kPlane * 4;
    static constexpr int kDirect = EdmF32Shape<TILE, 4 * TILE>::LDS_FLOATS * 4;
    static constexpr int kBytes = kBuffer * 2 > kDirect ? kBuffer * 2 : kDirect;
    __attribute__((aligned(16))) unsigned char operands[kBytes];
    __attribute__((aligned(16))) float norms[2 * TILE];
    float spread[4 * TILE / 64];
    int many;                            // near pairs counted, or more
};

// Byte offset in a plane of 16-byte slot q (dimensions 8 q .. 8 q + 7) of a point.
__device__ __forceinline__ int gram_slot(int point, int q)
{
    return point * (kGramK * 2) + 16 * (q ^ ((point >> 3) & 1));
}

// v = h + l to 23 significant bits or 2^-25, whichever is coarser.
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void gram_split(const f32x4 &v, f16x4 &h, f16x4 &l)
{
    h = __builtin_convertvector(v, f16x4);
    f32x4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = __builtin_fmaf((float)h[e], -1.f, v[e]);
    l = __builtin_convertvector(r, f16x4);
}

// v holds coordinates d - 4 .. d - 1: those from d - 4 + sh on, zeros behind.
__device__ __forceinline__ f32x4 gram_tail(const f32x4 &v, int32_t sh)
{
    f32x4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        r[e] = 0.f;
#pragma unroll
        for (int g = e; g < 4; ++g) r[e] = sh == g - e ? v[g] : r[e];
    }
    return r;
}

template <bool FULL, int WA>
__device__ __forceinline__ void gram_store(char *ob, const f32x16 (&acc)[WA], int32_t R0,
                                           int32_t j, int32_t n, int l)
{
#pragma unroll
    for (int a = 0; a < WA; ++a)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            int32_t i = R0 + 32 * a + 8 * q + 4 * (l >> 5);
            uint32_t off = (uint32_t)((i - R0) * (i + R0 - 1)) / 2u + (uint32_t)j;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float dd = sqrt_near1(acc[a][4 * q + u]);
                if (FULL || (i < n && j < i)) *(float *)(ob + (off << 2)) = dd;
                off += (uint32_t)i;  // start of row i + 1
                ++i;
            }
        }
}

// The distances of tile (bi, bj), by 4 TILE threads (t: this one's number).  sC:
// d floats in whole chunks.  The caller synchronises between tiles.
template <int TILE>
__device__ __forceinline__ void edm_gram_body(const EdmTile &p, int32_t bi, int32_t bj,
                                              GramLds<TILE> &sh, float *sC, int t)
{
    constexpr int NT = 4 * TILE;
    constexpr int WA = TILE / 64;          // a wave has WA blocks of 32 rows, 32 columns
    constexpr int WT = TILE / 2;           // its rows
    unsigned char *const lds = sh.operands;
    float *const sN = sh.norms, *const sSpread = sh.spread;
    int &sMany = sh.many;
    const int l = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int32_t n = p.n, d = p.d;
    const int64_t ldx = p.ldx;
    const int32_t ri0 = 1 + bi * TILE, cj0 = bj * TILE;
    const char *const xi = (const char *)(p.x + (int64_t)ri0 * ldx);  // ri0, cj0 < n
    const char *const xj = (const char *)(p.x + (int64_t)cj0 * ldx);
    const uint32_t pitch = (uint32_t)ldx * 4u;

    const int kq = t % 4, pt = t / 4;      // this thread stages dimensions 4 kq .. of point pt
    const char *const pi = xi + (uint32_t)min(pt, n - 1 - ri0) * pitch;
    const char *const pj = xj + (uint32_t)min(pt, n - 1 - cj0) * pitch;
    f32x4 vi, vj;
    auto load = [&](int32_t k0) {
        const uint32_t o = (uint32_t)min(k0 + 4 * kq, d - 4) * 4u;
        vi = *(const f32x4u *)(pi + o);
        vj = *(const f32x4u *)(pj + o);
    };
    load(0);

    if (t == 0) sMany = 0;
    float spread = 0.f;
    for (int32_t k = t; k < (d + kGramK - 1) / kGramK * kGramK; k += NT) {
        float v[16];
        const uint32_t ko = (uint32_t)min(k, d - 1) * 4u;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            v[u] = *(const float *)(xi + (uint32_t)min(u * (TILE / 8), n - 1 - ri0) * pitch + ko);
            v[8 + u] = *(const float *)(xj + (uint32_t)min(u * (TILE / 8), n - 1 - cj0) * pitch + ko);
        }
        float s = 0.f, lo = v[0], hi = v[0];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            s += v[u];
            lo = fminf(lo, v[u]);
            hi = fmaxf(hi, v[u]);
        }
        sC[k] = k < d ? s * 0.0625f : 0.f;
        spread = fmaxf(spread, hi - lo);
    }
#pragma unroll
    for (int h = 1; h < 64; h *= 2) spread = fmaxf(spread, __shfl_xor(spread, h));
    if (l == 0) sSpread[w] = spread;
    __syncthreads();
    // the power of two that brings the samples' spread to about 2^8
#pragma unroll
    for (int h = 0; h < NT / 64; ++h) spread = fmaxf(spread, sSpread[h]);
    const uint32_t ex = __builtin_bit_cast(uint32_t, spread) >> 23;
    const float sc = ex ? __builtin_bit_cast(float, min(262u - ex, 254u) << 23) : 1.f;
    // the centre in scaled units, to a multiple of 4 (see above)
    for (int32_t k = t; k < (d + kGramK - 1) / kGramK * kGramK; k += NT)
        sC[k] = 4.f * __builtin_rintf(sC[k] * (0.25f * sc));
    lds_barrier();

    const int wr = w & 1, wc = w >> 1, lr = l & 31;
    constexpr int kPlane = GramLds<TILE>::kPlane, kBuffer = GramLds<TILE>::kBuffer;
    const int so = gram_slot(pt, kq >> 1) + 8 * (kq & 1);
    float ni[2] = {0.f, 0.f}, nj[2] = {0.f, 0.f};
    // this thread's vectors of chunk k0, centred and split, into buffer q
    auto stage = [&](int32_t k0, unsigned char *q) {
        const int32_t k = k0 + 4 * kq;
        const f32x4 c = *(const f32x4 *)&sC[k];
        if (k0 + kGramK > d) {             // dimensions from d on are zero, as c is there
            const int32_t sh = k - min(k, d - 4);
            vi = gram_tail(vi, sh);
            vj = gram_tail(vj, sh);
        }
        f32x4 yi, yj;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            yi[e] = __builtin_fmaf(vi[e], sc, -c[e]);
            yj[e] = __builtin_fmaf(vj[e], sc, -c[e]);
            ni[e & 1] = __builtin_fmaf(yi[e], yi[e], ni[e & 1]);
            nj[e & 1] = __builtin_fmaf(yj[e], yj[e], nj[e & 1]);
        }
        f16x4 h, lo;
        gram_split(yi, h, lo);
        *(f16x4 *)(q + so) = h;
        *(f16x4 *)(q + kPlane + so) = lo;
        gram_split(yj, h, lo);
        *(f16x4 *)(q + 2 * kPlane + so) = h;
        *(f16x4 *)(q + 3 * kPlane + so) = lo;
    };
    stage(0, lds);
    if (kGramK < d) load(kGramK);
    lds_barrier();

    int oa[WA];
#pragma unroll
    for (int a = 0; a < WA; ++a) oa[a] = gram_slot(WT * wr + 32 * a + lr, l >> 5);
    const int ob0 = 2 * kPlane + gram_slot(32 * wc + lr, l >> 5);
    f32x16 acc[WA];
#pragma unroll
    for (int a = 0; a < WA; ++a) acc[a] = f32x16{};
    // A point's scaled norm so far, from the four threads that stage it.
    auto norm = [&](const float (&v)[2]) {
        float s = v[0] + v[1];
#pragma unroll
        for (int h = 1; h < 4; h *= 2) s += __shfl_xor(s, h);
        return s;
    };
    const int32_t R0 = ri0 + WT * wr, C0 = cj0 + 32 * wc;
    const int32_t j = C0 + lr;
    bool direct = false;                   // the same for the whole workgroup
    int buf = 0;
    for (int32_t k0 = 0; k0 < d; k0 += kGramK) {
        if (k0 == kGramK) {                // of the 32 dimensions staged so far
            const float mi = norm(ni), mj = norm(nj);
            if (kq == 0) {
                sN[pt] = mi;
                sN[TILE + pt] = mj;
            }
        }
        const unsigned char *const q = lds + buf;
        buf ^= kBuffer;
        f16x8 va[2][WA], vb[2];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            vb[g] = *(const f16x8 *)(q + ob0 + g * kPlane);
#pragma unroll
            for (int a = 0; a < WA; ++a) va[g][a] = *(const f16x8 *)(q + oa[a] + g * kPlane);
        }
        if (k0 + kGramK < d) {             // the next chunk, and the loads of the one after it
            stage(k0 + kGramK, lds + buf);
            if (k0 + 2 * kGramK < d) load(k0 + 2 * kGramK);
        }
        // the small products first
        constexpr int QA[3] = {1, 0, 0}, QB[3] = {0, 1, 0};
#pragma unroll
        for (int g = 0; g < 3; ++g)
#pragma unroll
            for (int a = 0; a < WA; ++a)
                acc[a] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va[QA[g]][a], vb[QB[g]], acc[a],
                                                                0, 0, 0);
        lds_barrier();
        if (k0 == kGramK) {
            // Four of each lane's pairs over the first 32 dimensions: a tile
            // whose pairs are often near is left to the direct body here.
            const f32x4 si = *(const f32x4 *)&sN[WT * wr + 4 * (l >> 5)];
            const float sj = sN[TILE + 32 * wc + lr];
            int many = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float s = si[u] + sj;
                many += __popcll(__ballot(!(__builtin_fmaf(-2.f, acc[0][u], s) >= kGramNear * s) &&
                                          j < R0 + 4 * (l >> 5) + u));
            }
            if (l == 0 && many) atomicAdd(&sMany, many);
            lds_barrier();
            direct = sMany > NT / 4;       // one in sixteen
            if (direct) break;
        }
    }

    // norms; one out of range (the halves of a point whose scaled norm is below
    // 2^30 are finite) makes its pairs' sums NaN, and those pairs near
    const float mi = norm(ni), mj = norm(nj);
    const float inv2 = 1.f / (sc * sc);
    const float line = d >= kGramWideDims ? kGramNearWide : kGramNear;
    const float least = fmaxf(0x1p-90f, kGramFloor * (float)d * inv2);
    if (kq == 0) {
        sN[pt] = mi < 0x1p30f && mi * inv2 < 0x1p93f ? mi * inv2 : __builtin_nanf("");
        sN[TILE + pt] = mj < 0x1p30f && mj * inv2 < 0x1p93f ? mj * inv2 : __builtin_nanf("");
    }
    __syncthreads();

    const bool work = R0 < n && C0 < R0 + WT - 1;  // some pair j < i < n in the wave's block
    const float sj = sN[TILE + 32 * wc + lr];
    bool near = false;
#pragma unroll
    for (int a = 0; a < WA; ++a)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const f32x4 si = *(const f32x4 *)&sN[WT * wr + 32 * a + 8 * q + 4 * (l >> 5)];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float s = si[u] + sj;
                const float v = __builtin_fmaf(-2.f * inv2, acc[a][4 * q + u], s);
                acc[a][4 * q + u] = v;
                near |= !(v >= __builtin_fmaf(s, line, least));
            }
        }
    uint32_t m = 0;                        // this lane's near pairs: bit 16 a + r
    if (!direct && work && __any(near)) {
        int o = 0;                         // keeps the sums above from being held
        asm volatile("" : "+v"(o));
#pragma unroll
        for (int a = 0; a < WA; ++a)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int dr = 32 * a + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3);
                const float s = sN[o + WT * wr + dr] + sj;
                if (!(acc[a][r] >= __builtin_fmaf(s, line, least)) && j < R0 + dr &&
                    R0 + dr < n)
                    m |= 1u << (16 * a + r);
            }
        if (__any(__popc(m) > kGramLaneNear) && l == 0) sMany = NT;
    }
    __syncthreads();
    if (sMany > NT / 4) {
        edm_f32_tile_body<TILE, kEdmStageScalar, NT>(p, bi, bj, (float *)lds, t);
        return;
    }
    if (!work) return;
    char *const ob = (char *)(p.out + (uint64_t)R0 * (uint64_t)(R0 - 1) / 2);
    if (C0 + 31 < R0 && R0 + WT - 1 < n)
        gram_store<true, WA>(ob, acc, R0, j, n, l);
    else
        gram_store<false, WA>(ob, acc, R0, j, n, l);
    while (m) {                            // over the values just stored, by the same lane
        const int r = __builtin_ctz(m);
        m &= m - 1;
        const int32_t i = R0 + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3);
        *(float *)(ob + (((uint32_t)((i - R0) * (i + R0 - 1)) / 2u + (uint32_t)j) << 2)) =
            __builtin_sqrtf(direct_d2_wide(p.x, ldx, d, i, j));
    }
}

// Whether a tile takes the products: its offsets are 32 bits, 128 rows of ldx.
inline bool edm_gram_takes(int tile, int64_t d, int64_t ldx)
{
    return tile >= 64 && d >= kGramMinDims && ldx <= (1 << 22);
}

}  // namespace trimap
