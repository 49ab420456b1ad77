#pragma once
// EDT tiles by pruned search, for maps with every axis <= 512: the tiles
// edt_compute and edt_compute_many use for such maps.
//
// Both passes minimise f_s(q) = h_s + (q - s)^2 over the sites s of a line
// (Sec. III-C, steps 2-4), the smaller s on ties.  An envelope is built and
// walked by one thread per line or band, a chain of dependent steps whose
// length differs from lane to lane.  Here a wave (64 lanes = 64 lines) takes
// blocks of 8 consecutive positions and evaluates every site that can win for
// one of them, with no data-dependent chain:
//
//   * one packed integer (f_s(q) - i^2) << 9 | s per position q = qa + i, so
//     that a minimum keeps the value and the smallest site at once; from one
//     position to the next it changes by the lane-independent 2 (s - qa) << 9,
//     and two sites cost 2 adds and one three-way minimum per position;
//   * sites are skipped by bounds: every group (16 groups per line) and every
//     chunk (C sites) keeps the smallest h of each lane, hmin.  hmin plus the
//     squared distance between the far ends bounds every position's result
//     from above, hmin plus the squared gap bounds what the chunk can offer
//     from below, and a chunk is evaluated iff some lane's lower bound does
//     not exceed its upper bound.  The result at the last position of the
//     block before gives a second upper bound, and its site a lower limit
//     (the winning site never decreases along a line).
//
// No stack and no merge: a line's sites are in LDS, a wave reads the ones it
// evaluates, and each wave finishes its own band of BAND positions after a
// single barrier.
//
// What bounds them is instruction issue: 45 to 100 VALU instructions per voxel
// and pass (17 to 35 evaluated sites per voxel at 1.75 each, the bounds, the
// write-out) and 30 to 45 scalar ones.  The bounds are therefore tests whose
// signs a lane shifts into one mask that is joined across the wave, against
// distances from tables, and only a band's first block takes upper bounds from
// all groups; later ones have the block before.  One xy pass in us, with a
// ballot per test and computed distances and like this: 256 x 256 x 128 frame
// 28.0 -> 26.5, 512 x 512 x 128 73.2 -> 68.6, 512^3 blobs 381 -> 374.
#include "edt_tiles.h"

namespace edtmi {
namespace search {

using tiles::mul24;
using tiles::XY_NONE;

typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

constexpr int AXIS_MAX = 512;   // longest axis
constexpr int NG = 16;          // groups per line
constexpr int QB = 8;           // positions per block
constexpr int SB = 9;           // bits of a site's position in a packed value
// h of an empty position: above every real h + (q - s)^2 (at most 3 * 511^2 =
// 783,363, 2 * 511^2 in the xy pass), and small enough that the packed value
// stays below 2^31: at most 1,511^2 + 511^2 for V_EMPTY seen from any voxel and
// 1,535^2 in the xy pass, + 511^2 for the position, below 2^22
constexpr uint32_t V_EMPTY = 0xFC18u;   // x' = -1000, y' = 0
constexpr int LEFT_NONE = -1024, RIGHT_NONE = 2047;   // x' where a row has none on that side:
                                                      // the left one is the nearer, 1,024 .. 1,535 away
constexpr int D_EMPTY = 1024;           // x - x' of rows past the map's
constexpr int H_EMPTY = 1000000;        // every empty h is at least this
static_assert(1511 * 1511 + 2 * 511 * 511 < (1 << (31 - SB)) && 1535 * 1535 + 511 * 511 < (1 << (31 - SB)),
              "packed values must fit 31 bits");

constexpr int W = 16;           // positions on either side of a block that the short test covers

// ---------------------------------------------------------------------------
// occupancy bits (the input of step 1): bit mis + lin = voxel lin is occupied,
// mis = the occupancy pointer's offset from a 16-byte boundary.  They live in
// the d2 buffer, which the xy pass does not use and the z pass overwrites, and fit
// with the words that a row's last reads touch: a map that takes bits has more than
// 64 voxels, and (n + 15) / 32 + 2 ntx + 1 words are fewer than n.
// ---------------------------------------------------------------------------
__host__ __device__ inline int misalignment(const void* occ) { return (int)((uintptr_t)occ & 15u); }

// 0x80 in every byte of w that is not zero
__device__ __forceinline__ uint32_t nonzero_high(uint32_t w)
{
    return (((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w) & 0x80808080u;
}

// 16 voxels as bits: bytes [16 c, 16 c + 16) from the 16-byte boundary at or
// below occ.  A chunk that sticks out of the map is read byte by byte, so no
// load leaves [occ, occ + n).
__device__ __forceinline__ uint32_t chunk_bits(const uint4& a)
{
    // the eight 0x80 flags of two words, weighted 1 .. 128: 128 times their bits
    uint32_t t = __builtin_amdgcn_udot4(nonzero_high(a.x), 0x08040201u, 0u, false);
    t = __builtin_amdgcn_udot4(nonzero_high(a.y), 0x80402010u, t, false);
    uint32_t h = __builtin_amdgcn_udot4(nonzero_high(a.z), 0x08040201u, 0u, false);
    h = __builtin_amdgcn_udot4(nonzero_high(a.w), 0x80402010u, h, false);
    return (t >> 7) | (h >> 7) << 8;
}

// The words of one wave: BITS_U * 64 chunks from chunk c0 on, a load of the
// wave covering 1 KiB in one piece, all loads in flight; an even lane joins its
// chunk with its neighbour's to a word.  48 self maps of 128^3 32 us with two
// loads in flight, 23 with four and 22 with eight (a work-group first finds its
// map in the set); a single map takes the same with all three (512^3 50 us, the
// map read from HBM while the passes before are written back).
constexpr int BITS_U = 4;

__device__ __forceinline__ void map_bits(const uint8_t* __restrict__ occ, int64_t n, int64_t c0,
                                         uint32_t* __restrict__ bits)
{
    const int mis = misalignment(occ);
    const int lane = threadIdx.x & 63;
    const int64_t f0 = 16 * c0 - mis;   // the wave's first voxel
    if (f0 >= n) return;
    uint4 v[BITS_U];
    uint32_t m[BITS_U];
    const bool whole = f0 >= 0 && f0 + 1024 * BITS_U <= n;   // wave-uniform
    if (whole) {
        const uint4* p = reinterpret_cast<const uint4*>(occ + f0) + lane;
#pragma unroll
        for (int j = 0; j < BITS_U; ++j) v[j] = p[64 * j];
#pragma unroll
        for (int j = 0; j < BITS_U; ++j) m[j] = chunk_bits(v[j]);
    } else {
#pragma unroll
        for (int j = 0; j < BITS_U; ++j) {
            const int64_t f = f0 + 1024 * j + 16 * lane;
            m[j] = 0;
            if (f >= 0 && f + 16 <= n) {
                m[j] = chunk_bits(*reinterpret_cast<const uint4*>(occ + f));
            } else {
                for (int k = 0; k < 16; ++k)
                    if (f + k >= 0 && f + k < n && occ[f + k]) m[j] |= 1u << k;
            }
        }
    }
    uint32_t* w = bits + c0 / 2;
#pragma unroll
    for (int j = 0; j < BITS_U; ++j) {
        // quad_perm 1, 1, 3, 3: the neighbour of an even lane
        const uint32_t o = __builtin_amdgcn_update_dpp(0, m[j], 0xF5, 0xF, 0xF, true);
        if ((lane & 1) == 0 && f0 + 1024 * j + 16 * lane < n) w[32 * j + lane / 2] = m[j] | o << 16;
    }
}

// Squared distances between block b (positions 8 b .. 8 b + 7) and group g of a
// line: of their farthest and of their nearest ends.  Read with scalar loads.
template <int NMAX> struct Bounds {
    int far2[NMAX / QB][NG], gap2[NMAX / QB][NG];
    constexpr Bounds() : far2{}, gap2{}
    {
        constexpr int G = NMAX / NG;
        for (int b = 0; b < NMAX / QB; ++b)
            for (int g = 0; g < NG; ++g) {
                const int lo = G * g - QB * b;   // the group's first position, from the block's
                const int f1 = lo + G - 1, f2 = QB - 1 - lo, far = f1 > f2 ? f1 : f2;
                const int g1 = lo - (QB - 1), g2 = -(lo + G - 1), gap = g1 > g2 ? g1 : g2;
                far2[b][g] = far * far;
                gap2[b][g] = gap > 0 ? gap * gap : 0;
            }
    }
};
template <int NMAX> __constant__ constexpr Bounds<NMAX> BOUNDS{};

// Squared gap between a block whose first chunk is cb and chunk c, at c - cb + NMAX / C.
template <int NMAX, int C> struct ChunkGaps {
    int gap2[2 * NMAX / C];
    constexpr ChunkGaps() : gap2{}
    {
        for (int j = 0; j < 2 * NMAX / C; ++j) {
            const int lo = C * (j - NMAX / C);   // the chunk's first position, from the block's
            const int g1 = lo - (QB - 1), g2 = -(lo + C - 1), gap = g1 > g2 ? g1 : g2;
            gap2[j] = gap > 0 ? gap * gap : 0;
        }
    }
};
template <int NMAX, int C> __constant__ constexpr ChunkGaps<NMAX, C> CHUNK_GAPS{};

__device__ __forceinline__ int band_of_wave() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }
__device__ __forceinline__ bool any_lane(bool p) { return __builtin_amdgcn_ballot_w64(p) != 0; }
__device__ __forceinline__ bool any_lane2(bool p, bool q)
{
    return (__builtin_amdgcn_ballot_w64(p) & __builtin_amdgcn_ballot_w64(q)) != 0;
}

// v of all lanes, joined
__device__ __forceinline__ uint32_t or_lanes(uint32_t v)
{
    v |= __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);   // row_shr:1
    v |= __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);
    return __builtin_amdgcn_readlane(v, 15) | __builtin_amdgcn_readlane(v, 31) |
           __builtin_amdgcn_readlane(v, 47) | __builtin_amdgcn_readlane(v, 63);
}

// ---------------------------------------------------------------------------
// the search of one wave: positions [q0, q1) of its 64 lines
//   np        positions with chunk minima (a multiple of BAND; the ones past
//             the line's end are empty)
//   cmin(c)   the smallest h of chunk c (this lane)
//   gmin(g)   the smallest h of group g
//   site(c, k, a)  h of site k of chunk c, plus a (this lane)
//   emit(q, n, value, s)  positions q .. q + n - 1 (n <= 8) of a line with
//             sites: value[i] = f_s(q + i) for the winning site s[i]
//   none(q)   a position of a line that has no site
// ---------------------------------------------------------------------------
template <int NMAX, int C, class CMin, class GMin, class Site, class Emit, class None>
__device__ __forceinline__ void search_band(int q0, int q1, int np, CMin cmin, GMin gmin, Site site, Emit emit, None none)
{
    constexpr int G = NMAX / NG;
    constexpr int CG = G / C;       // chunks per group
    constexpr int CB = QB / C;      // chunks per block
    constexpr int CW = W / C;       // chunks on either side of a block in the short test
    int gm[NG];
    if (np == NMAX) {
#pragma unroll
        for (int g = 0; g < NG; ++g) gm[g] = gmin(g);
    } else {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            gm[g] = 1 << 21;
            if (g * G < np) gm[g] = gmin(g);
        }
    }
    {
        int m = gm[0];
#pragma unroll
        for (int g = 1; g < NG; ++g) m = min(m, gm[g]);
        if (!any_lane(m < H_EMPTY)) {   // no site: a wave-wide fact
            for (int q = q0; q < q1; ++q) none(q);
            return;
        }
    }
    const int nch = np / C;
    int lo = 0;              // no site below lo can win from here on
    int up = 0x7FFFFFFF;     // upper bound from the block before
    for (int qa = q0; qa < q1; qa += QB) {
        const int cb0 = qa / C;   // the block's first chunk
        int best[QB];
#pragma unroll
        for (int i = 0; i < QB; ++i) best[i] = 0x7FFFFFFF;
        auto evaluate = [&](int c) {
            int p[C], st[C];
#pragma unroll
            for (int k = 0; k < C; ++k) {
                const int sg = c * C + k - qa;
                st[k] = sg << (SB + 1);
                p[k] = (site(c, k, sg * sg) << SB) | (c * C + k);
            }
#pragma unroll
            for (int k = 0; k < C; k += 2) {
#pragma unroll
                for (int i = 0; i < QB; ++i) {
                    best[i] = min(min(best[i], p[k]), p[k + 1]);
                    if (i + 1 < QB) {
                        p[k] -= st[k];
                        p[k + 1] -= st[k + 1];
                    }
                }
            }
        };
        // ---- upper bound for every position of the block from its own
        // chunks and the two beside them
        int U = up;
        U = min(U, cmin(cb0 > 0 ? cb0 - 1 : 0) + (C + QB - 1) * (C + QB - 1));
        U = min(U, cmin(cb0 + CB < nch ? cb0 + CB : cb0) + (C + QB - 1) * (C + QB - 1));
#pragma unroll
        for (int k = 0; k < CB; ++k) U = min(U, cmin(cb0 + k) + (QB - 1) * (QB - 1));
        if (!any_lane(U > W * W)) {
            // nothing farther than W can win: the chunks up to there, directly
            uint32_t cmask = 0;
#pragma unroll
            for (int j = 0; j < CB + 2 * CW; ++j) {
                const int c = cb0 - CW + j;
                const int gap = j < CW ? C * (CW - 1 - j) + 1 : (j < CW + CB ? 0 : C * (j - CW - CB) + 1);
                const int m = cmin(c < 0 ? 0 : (c < nch ? c : nch - 1));
                cmask |= any_lane2(m + gap * gap <= U, C * c + C - 1 >= lo) ? 1u << j : 0u;
            }
            cmask &= (cb0 < CW ? ~0u << (CW - cb0) : ~0u) &
                     (nch - cb0 + CW < 32 ? (1u << (nch - cb0 + CW)) - 1u : ~0u);
            while (cmask) {
                evaluate(cb0 - CW + __builtin_ctz(cmask));
                cmask &= cmask - 1u;
            }
        } else {
            // the groups' bounds first, then the chunks of the groups left
            const int* far2 = BOUNDS<NMAX>.far2[qa / QB];
            const int* gap2 = BOUNDS<NMAX>.gap2[qa / QB];
            if (qa == q0) {
#pragma unroll
                for (int g = 0; g < NG; ++g) U = min(U, gm[g] + far2[g]);
            }
            // a lane's tests shift their sign into its mask; then the lanes' masks are joined
            uint32_t gmask = 0;
#pragma unroll
            for (int g = NG - 1; g >= 0; --g)
                gmask = __builtin_amdgcn_alignbit(gmask, (uint32_t)(gm[g] + gap2[g] + ~U), 31);
            gmask = or_lanes(gmask);
            while (gmask) {
                const int g = __builtin_ctz(gmask);
                gmask &= gmask - 1u;
                uint32_t cmask = 0;
                const int* cgap2 = CHUNK_GAPS<NMAX, C>.gap2 + (NMAX / C - cb0 + g * CG);
#pragma unroll
                for (int k = 0; k < CG; ++k) {
                    const int c = g * CG + k;
                    cmask |= any_lane2(cmin(c) + cgap2[k] <= U, C * c + C - 1 >= lo) ? 1u << k : 0u;
                }
                while (cmask) {
                    evaluate(g * CG + __builtin_ctz(cmask));
                    cmask &= cmask - 1u;
                }
            }
        }
        // ---- results
        int val[QB], at[QB];
#pragma unroll
        for (int i = 0; i < QB; ++i) {
            val[i] = (best[i] >> SB) + i * i;
            at[i] = best[i] & (AXIS_MAX - 1);
        }
        // the last position's site s and value v bound the next block: f_s
        // grows by 2 (q - s) + 1 from q to q + 1, and is convex along the block
        lo = at[QB - 1];
        const int d = qa + QB - 1 - lo;
        up = max(val[QB - 1] + 2 * d + 1, val[QB - 1] + 2 * QB * d + QB * QB);
        emit(qa, min(QB, q1 - qa), val, at);
    }
}

// ---------------------------------------------------------------------------
// z pass (step 4): tile T = 64 consecutive columns of the map's xy plane (a
// column's lane finds its x and y, so rows that are no multiple of 64 leave
// no lane idle), one wave per band of BAND slices.  Reads the packed 2D sites
// from site and overwrites d2 and site in place: every global read happens
// before the barrier, every write after it, and a column belongs to one tile.
//   lds   np * 256 bytes of sites [slice][lane], then np / C * 256 bytes of
//         chunk minima, np = BAND * waves >= nz
// ---------------------------------------------------------------------------
// A wave's place in one column tile, and its band's sites on their way from
// memory.
struct ZTile {
    int32_t *d2, *site;   // the tile's first column
    unsigned plane, off;  // voxels per slice; the lane's column, clamped into the plane
    int nx, nz;
    s16x2 own;            // the lane's x and y
    bool live;
};
template <int BAND> struct ZBand : ZTile {
    uint32_t v[BAND];

    __device__ __forceinline__ void load(int32_t* d2_, int32_t* site_, int nx_, int ny, int nz_, int T, int q0)
    {
        const int lane = threadIdx.x & 63;
        nx = nx_;
        nz = nz_;
        plane = (unsigned)nx * (unsigned)ny;
        const unsigned c0 = (unsigned)T * 64u;
        const unsigned cc = min(c0 + lane, plane - 1u);
        live = c0 + lane < plane;
        off = cc - c0;
        const unsigned y = cc / (unsigned)nx, x = cc - y * (unsigned)nx;
        own = __builtin_bit_cast(s16x2, x | (y << 16));
        d2 = d2_ + c0;
        site = site_ + c0;
        // all loads of the band in flight, clamped into the column
        const uint32_t* in = reinterpret_cast<const uint32_t*>(site);
#pragma unroll
        for (int i = 0; i < BAND; ++i) v[i] = (in + (size_t)min(q0 + i, nz - 1) * plane)[off];
    }
};

// the band's sites and chunk minima into local memory
template <int C, int BAND>
__device__ __forceinline__ void z_stage(ZBand<BAND>& b, int np, uint32_t* lds)
{
    uint32_t* val = lds;
    int* cm = reinterpret_cast<int*>(lds + np * 64);
    const int lane = threadIdx.x & 63;
    const int q0 = band_of_wave() * BAND;
    if (q0 + BAND > b.nz) {
#pragma unroll
        for (int i = 0; i < BAND; ++i)
            if (q0 + i >= b.nz) b.v[i] = XY_NONE;
    }
    uint32_t* vb = val + q0 * 64 + lane;
    int* cb = cm + q0 / C * 64 + lane;
#pragma unroll
    for (int i = 0; i < BAND; i += C) {
        int m = 1 << 21;
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const uint32_t e = b.v[i + k] == XY_NONE ? V_EMPTY : b.v[i + k];
            vb[(i + k) * 64] = e;
            const s16x2 d = b.own - __builtin_bit_cast(s16x2, e);
            m = min(m, __builtin_amdgcn_sdot2(d, d, 0, false));
        }
        cb[i / C * 64] = m;
    }
}

// the band's results
template <int NMAX, int C, int BAND>
__device__ __forceinline__ void z_band(const ZTile& t, int np, uint32_t* lds)
{
    int32_t *__restrict__ d2 = t.d2, *__restrict__ site = t.site;
    const unsigned plane = t.plane, off = t.off;
    const int nx = t.nx, nz = t.nz;
    const s16x2 own = t.own;
    const bool live = t.live;
    const uint32_t* val = lds;
    const int* cm = reinterpret_cast<const int*>(lds + np * 64);
    const int lane = threadIdx.x & 63;
    const int q0 = band_of_wave() * BAND;
    const int q1 = min(nz, q0 + BAND);
    if (q0 >= q1) return;
    const u16x2 lin = __builtin_bit_cast(u16x2, 1u | ((unsigned)nx << 16));
    search_band<NMAX, C>(
        q0, q1, np, [&](int c) { return cm[c * 64 + lane]; },
        [&](int g) {
            constexpr int CG = NMAX / NG / C;
            const int* p = cm + g * (CG * 64) + lane;
            int m = p[0];
#pragma unroll
            for (int k = 1; k < CG; ++k) m = min(m, p[k * 64]);
            return m;
        },
        [&](int c, int k, int a) {
            const s16x2 d = own - __builtin_bit_cast(s16x2, (val + c * (C * 64) + lane)[k * 64]);
            return __builtin_amdgcn_sdot2(d, d, a, false);
        },
        [&](int q, int n, const int (&value)[QB], const int (&s)[QB]) {
            int32_t lx[QB];   // x' + nx y' + plane z'
#pragma unroll
            for (int i = 0; i < QB; ++i)
                lx[i] = (int32_t)__builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, val[s[i] * 64 + lane]), lin,
                                                        __umul24(plane, (unsigned)s[i]), false);
            if (!live) return;
            int32_t* od = d2 + (size_t)q * plane;
            int32_t* os = site + (size_t)q * plane;
#pragma unroll
            for (int i = 0; i < QB; ++i) {
                if (i >= n) break;
                od[off] = value[i];
                os[off] = lx[i];
                od += plane;
                os += plane;
            }
        },
        [&](int q) {
            if (live) {
                (d2 + (size_t)q * plane)[off] = 0x7FFFFFFF;
                (site + (size_t)q * plane)[off] = -1;
            }
        });
}

// ---------------------------------------------------------------------------
// xy pass (steps 2-3): tile T = z * ntx + x0 / 64, one wave per band of BAND
// rows, from the map's occupancy bits, or with occ given (ntx = 1, n voxels) from
// its bytes.  Writes the 2D site x' | y' << 16 of every voxel of the tile
// (0xFFFFFFFF if the slice is empty).
//   lds   np * 128 bytes of x - x' [row][lane], then np / C * 128 bytes of
//         chunk minima of |x - x'|, np = BAND * waves >= ny
// ---------------------------------------------------------------------------
// leading / trailing zeros, 0xFFFFFFFF for 0
__device__ __forceinline__ uint32_t ffbh(uint32_t v)
{
    uint32_t r;
    asm("v_ffbh_u32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}
__device__ __forceinline__ uint32_t ffbl(uint32_t v)
{
    uint32_t r;
    asm("v_ffbl_b32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}

// The occupancy bits of a wave's band, voxels f0 .. f1 - 1 (at most 64 BAND), into
// local memory (at most 2 BAND + 2 words): bit mis + i = voxel f0 + i, mis returned.
template <int BAND>
__device__ __forceinline__ int band_bits(const uint8_t* __restrict__ occ, int64_t n, int64_t f0, int64_t f1,
                                         uint32_t* words)
{
    const int mis = misalignment(occ + f0);
    const int lane = threadIdx.x & 63;
    constexpr int U = (64 * BAND + 15 + 1023) / 1024;   // 64 chunks of 16 voxels each
    uint32_t m[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
        const int64_t f = f0 - mis + 1024 * j + 16 * lane;
        m[j] = 0;
        if (f < f1) {
            if (f >= 0 && f + 16 <= n) {
                m[j] = chunk_bits(*reinterpret_cast<const uint4*>(occ + f));
            } else {
                for (int k = 0; k < 16; ++k)
                    if (f + k >= 0 && f + k < n && occ[f + k]) m[j] |= 1u << k;
            }
        }
    }
#pragma unroll
    for (int j = 0; j < U; ++j) {
        const uint32_t o = __builtin_amdgcn_update_dpp(0, m[j], 0xF5, 0xF, 0xF, true);   // as in map_bits
        const int c = 64 * j + lane;
        if ((lane & 1) == 0 && c / 2 < 2 * BAND + 2) words[c / 2] = m[j] | o << 16;
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    return mis;
}

template <int NMAX, int C, int BAND>
__device__ __forceinline__ void xy_tile(const uint32_t* __restrict__ bits, int mis, const uint8_t* __restrict__ occ,
                                        int64_t n, uint32_t* __restrict__ out, int nx, int ny, int ntx, int T, int np,
                                        uint32_t* lds)
{
    int16_t* dx = reinterpret_cast<int16_t*>(lds);
    uint16_t* cm = reinterpret_cast<uint16_t*>(dx + np * 64);
    const int lane = threadIdx.x & 63;
    const int band = band_of_wave();
    const int z = T / ntx;
    // the CUs take their second work-groups 256 tiles after their first ones:
    // shift the column tiles by half a row from there on, or a CU gets a map's
    // busy columns twice (256 x 256 x 128 frame 29.9 -> 28.0 us)
    const int zn = z * ntx;
    const int tx = (T - zn + (zn >> 8) * (ntx >> 1)) % ntx;
    // a lane past the row's end does what the row's last column does
    const int bit = min(lane, nx - 1 - tx * 64);
    const int xc = tx * 64 + bit;
    const bool live = bit == lane;
    const int q0 = band * BAND;
    const int q1 = min(ny, q0 + BAND);
    {
        // lane r takes row q0 + r: the tile's 64-column word and the nearest
        // occupied columns left and right of it, from the row's words (each
        // cut out of the bits with funnel shifts)
        constexpr int NW = AXIS_MAX / 64;
        uint32_t wl = 0, wh = 0;
        int l = LEFT_NONE, r = RIGHT_NONE;
        if (occ) {
            // in the place of the band's first rows, which come after
            uint32_t* words = lds + q0 * 32;
            const int64_t f0 = ((int64_t)z * ny + q0) * nx;
            const int off = band_bits<BAND>(occ, n, f0, f0 + max(q1 - q0, 0) * nx, words);
            if (lane < BAND && q0 + lane < q1) {
                const unsigned b = off + lane * nx;
                const uint32_t *p = words + (b >> 5), d0 = p[0], d1 = p[1], d2 = p[2];
                wl = __builtin_amdgcn_alignbit(d1, d0, b);
                wh = __builtin_amdgcn_alignbit(d2, d1, b);
                wl &= nx < 32 ? (1u << nx) - 1u : ~0u;
                wh &= nx < 64 ? (nx > 32 ? (1u << (nx - 32)) - 1u : 0u) : ~0u;
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
        } else if (lane < BAND && q0 + lane < q1) {
            const unsigned b = ((unsigned)z * ny + q0 + lane) * nx + mis;
            const uint32_t* p = bits + (b >> 5);
            uint32_t d[2 * NW + 1];
#pragma unroll
            for (int i = 0; i <= 2 * NW; ++i)
                if (i <= 2 * ntx) d[i] = p[i];
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                if (w >= ntx) break;
                uint32_t a = __builtin_amdgcn_alignbit(d[2 * w + 1], d[2 * w], b);
                uint32_t c = __builtin_amdgcn_alignbit(d[2 * w + 2], d[2 * w + 1], b);
                const int valid = nx - 64 * w;   // columns past the row's end
                if (valid < 64) {
                    a &= valid < 32 ? (1u << valid) - 1u : ~0u;
                    c &= valid > 32 ? (1u << (valid - 32)) - 1u : 0u;
                }
                if (w < tx) {
                    if (a | c) l = 64 * w + (c ? 63 - __builtin_clz(c) : 31 - __builtin_clz(a));
                } else if (w == tx) {
                    wl = a;
                    wh = c;
                } else if (r == RIGHT_NONE) {
                    if (a | c) r = 64 * w + (a ? __builtin_ctz(a) : 32 + __builtin_ctz(c));
                }
            }
        }
        const uint64_t rows = __builtin_amdgcn_ballot_w64((wl | wh) != 0 || l >= 0 || r < RIGHT_NONE);
        // the lane's columns up to and from its own, the row's neighbours as
        // distances from the tile's last and first column
        const uint32_t upto_l = bit < 32 ? ~0u >> (31 - bit) : ~0u, upto_h = bit < 32 ? 0u : ~0u >> (63 - bit);
        const uint32_t from_l = bit < 32 ? ~0u << bit : 0u, from_h = bit < 32 ? ~0u : ~0u << (bit - 32);
        const uint32_t lr = (uint32_t)(tx * 64 + 63 - l) | ((uint32_t)(r - tx * 64) << 16);
        int16_t* db = dx + q0 * 64 + lane;
        uint16_t* cb = cm + q0 / C * 64 + lane;
#pragma unroll
        for (int i = 0; i < BAND; i += C) {
            uint32_t m = D_EMPTY;
            if (((rows >> i) & ((1u << C) - 1u)) == 0) {   // wave-uniform
#pragma unroll
                for (int k = 0; k < C; ++k) db[(i + k) * 64] = (int16_t)D_EMPTY;
            } else {
                m = 2 * D_EMPTY;
#pragma unroll
                for (int k = 0; k < C; ++k) {
                    // step 1: the nearest occupied column of a row, ties to the left
                    const uint32_t wl_ = __builtin_amdgcn_readlane(wl, i + k), wh_ = __builtin_amdgcn_readlane(wh, i + k);
                    const uint32_t s = __builtin_amdgcn_readlane(lr, i + k);
                    const uint32_t el = min(min(ffbh(wh_ & upto_h), __builtin_elementwise_add_sat(ffbh(wl_ & upto_l), 32u)),
                                            s & 0xFFFFu);
                    const uint32_t er = min(min(ffbl(wl_ & from_l), __builtin_elementwise_add_sat(ffbl(wh_ & from_h), 32u)),
                                            s >> 16);
                    const uint32_t dl = el + bit - 63u, dr = er - bit;
                    db[(i + k) * 64] = (int16_t)(dl <= dr ? (int)dl : -(int)dr);
                    m = min(m, min(dl, dr));
                }
            }
            cb[i / C * 64] = (uint16_t)m;
        }
    }
    __syncthreads();
    if (q0 >= q1) return;
    uint32_t* o = out + (size_t)z * ny * nx + tx * 64;
    search_band<NMAX, C>(
        q0, q1, np,
        [&](int c) {
            const int m = cm[c * 64 + lane];
            return mul24(m, m);
        },
        [&](int g) {
            constexpr int CG = NMAX / NG / C;
            const uint16_t* p = cm + g * (CG * 64) + lane;
            int m = p[0];
#pragma unroll
            for (int k = 1; k < CG; ++k) m = min(m, (int)p[k * 64]);
            return mul24(m, m);
        },
        [&](int c, int k, int a) {
            const int d = (dx + c * (C * 64) + lane)[k * 64];
            return mul24(d, d) + a;
        },
        [&](int q, int n, const int (&)[QB], const int (&s)[QB]) {
            uint32_t w[QB];
#pragma unroll
            for (int i = 0; i < QB; ++i) w[i] = (uint32_t)(xc - dx[s[i] * 64 + lane]) | ((uint32_t)s[i] << 16);
            if (!live) return;
            uint32_t* ow = o + (size_t)q * nx;
#pragma unroll
            for (int i = 0; i < QB; ++i) {
                if (i >= n) break;
                ow[lane] = w[i];
                ow += nx;
            }
        },
        [&](int q) {
            if (live) (o + (size_t)q * nx)[lane] = XY_NONE;
        });
}

}  // namespace search
}  // namespace edtmi
