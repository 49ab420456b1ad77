// Statistical outlier filtering of a raw point cloud (Sec. III-A: the
// points are filtered by their Euclidean distance to their neighbours).
//
// Per finite point i: d_i = mean distance to its k nearest other points
// within radius R, a missing neighbour counting as R; over the finite
// points mu and the sample standard deviation sigma of d_i (exact
// fixed-point sums, so independent of the order of accumulation); keep i
// iff d_i <= mu + alpha * sigma.
//
// Neighbour search: a grid of cells wrapped onto A x B x C buckets (powers of
// two, each at least 8).  Cells that differ by whole periods share a bucket, the
// cells around any cell fall into distinct buckets, and the cells of an x run
// into consecutive ones.  Points are counted per bucket, every bucket gets a
// place in the sorted points, and the points are scattered there, so the points
// of an x run of cells are one contiguous range (two where the run wraps).
//
// k_sor_knn holds two searches with the same results, the faster one chosen on
// the device from the cloud's density (k_sor_zero):
//   * cells of 1.001 R: every neighbour lies in the 3 x 3 x 3 cells around a point,
//     which takes all their points, from local memory;
//   * for dense clouds cells of 1.001 R / 2: 5 x 5 x 5 cells, nearest first, cells
//     beyond the k-th nearest point left out (search_dense).
// The 0.1% covers the rounding of coordinates below about 80 m.
#include <algorithm>
#include <climits>
#include <cmath>

#include "common.h"

namespace edtmi {
namespace {

constexpr int KMAX = 16;

constexpr double SCALE1 = 1099511627776.0;   // 2^40: units of d
constexpr double SCALE2 = 281474976710656.0; // 2^48: units of d^2

// Bucket of a cell: (ix mod A) + A ((iy mod B) + B (iz mod C)).
struct Wrap {
    unsigned mx, my, mz;   // A - 1, B - 1, C - 1
    int sy, sz;            // log2 A, log2 (A B)
};

struct SorLayout {
    size_t count, table, spts, acc, total;
    unsigned tmask;
    Wrap wrap;
};

// table size: a power of two >= 2 n, at least 1024, at most 2^23
__host__ inline SorLayout sor_layout(int64_t n)
{
    int64_t T = 1024;
    while (T < 2 * n && T < (int64_t(1) << 23)) T <<= 1;
    SorLayout L;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += (bytes + 255) / 256 * 256;
        return at;
    };
    L.count = take((size_t)T * 4);
    L.table = take((size_t)T * 8);
    L.spts = take((size_t)std::max<int64_t>(n, 1) * 16);
    L.acc = take((size_t)(64 + 1) * 128);   // ACC_SLOTS lines and one more
    L.total = o;
    L.tmask = (unsigned)(T - 1);
    int t = 0;
    while ((int64_t(1) << t) < T) ++t;
    // T >= 2^10, so A, B and C are each at least 8, and A is at most 256
    const int a = (t + 2) / 3, b = (t - a + 1) / 2, c = t - a - b;
    L.wrap.mx = (1u << a) - 1u;
    L.wrap.my = (1u << b) - 1u;
    L.wrap.mz = (1u << c) - 1u;
    L.wrap.sy = a;
    L.wrap.sz = a + b;
    return L;
}

__device__ __forceinline__ bool finite3(float x, float y, float z)
{
    return __builtin_isfinite(x) && __builtin_isfinite(y) && __builtin_isfinite(z);
}

__device__ __forceinline__ int cell_of(float x, float h)
{
    const float c = floorf(x / h);
    return (int)fminf(fmaxf(c, -1.0e9f), 1.0e9f);
}

__device__ __forceinline__ unsigned bucket(int ix, int iy, int iz, const Wrap& w)
{
    return ((unsigned)ix & w.mx) | (((unsigned)iy & w.my) << w.sy) | (((unsigned)iz & w.mz) << w.sz);
}

// The sums of d and d^2 and the finite points are kept in ACC_SLOTS places, a
// cache line each, work-groups taking turns: on one line the 14,400 atomic
// additions of a frame would take 200 us.  The line after them counts the
// sorted points given out.
constexpr int ACC_SLOTS = 64, ACC_LINE = 16;
constexpr int ACC_GIVEN = ACC_SLOTS * ACC_LINE;
constexpr int ACC_DENSE = ACC_GIVEN + 1;   // 1: cells of R / 2 and search_dense

// search_dense takes over where a point's cell of 3 R holds more than DENSE other
// points on average, about the candidates the other search would take.  The whole
// filter with that one and with search_dense, us, by this average: a frame of
// 307,200 points 115 against 189 at 2, 217 / 193 at 59, 360 / 211 at 225, 605 / 395
// at 795; 200,000 points in a volume 90 / 137 at 146, 180 / 113 at 595; 100,000
// points in a ball 2,000 / 480 at 7,900.
constexpr float DENSE = 180.0f;
// Up to FEW points the first search is the faster one or close to it at any
// density (1,000 points in a ball: 120 / 107 to 160 / 350), and goes without the
// estimate's 4 us.
constexpr int FEW = 2048;
constexpr int SAMPLES = 1024, SLOTS = 2 * SAMPLES;

// Clears the counters.  With est = 1, work-group 0 meanwhile estimates the
// density: it counts the pairs of SAMPLES evenly spread points (one per thread, step
// points apart) that share a cell of 3 R, in a hash table in local memory.
__global__ __launch_bounds__(SAMPLES) void k_sor_zero(uint4* __restrict__ count, int T4,
                                                      unsigned long long* __restrict__ acc, int est,
                                                      const float* __restrict__ pts, int64_t n, int64_t step, float R)
{
    __shared__ __attribute__((aligned(16))) unsigned table[2][SLOTS];   // keys, points
    __shared__ unsigned pairs;
    const int t = threadIdx.x;
    if ((int)blockIdx.x >= est) {
        const int i = ((int)blockIdx.x - est) * SAMPLES + t;
        if (i < T4) count[i] = make_uint4(0u, 0u, 0u, 0u);
        if (i <= ACC_DENSE - est) acc[i] = 0ull;
        return;
    }
    const int m = (int)min(n, (int64_t)SAMPLES);
    float p[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) p[c] = t < m ? pts[3 * (t * step) + c] : __builtin_nanf("");
    reinterpret_cast<uint4*>(table)[t] = make_uint4(0u, 0u, 0u, 0u);
    if (t == 0) pairs = 0u;
    __syncthreads();
    if (finite3(p[0], p[1], p[2])) {
        unsigned key = 0;
#pragma unroll
        for (int c = 0; c < 3; ++c) key = (key ^ (unsigned)cell_of(p[c], 3.0f * R)) * 0x9E3779B1u + (key >> 15);
        key |= 1u;
        for (unsigned at = key >> 16;; ++at) {   // at most SAMPLES of the SLOTS are taken
            const unsigned old = atomicCAS(&table[0][at % SLOTS], 0u, key);
            if (old == 0u || old == key) {
                const unsigned others = atomicAdd(&table[1][at % SLOTS], 1u);
                if (others) atomicAdd(&pairs, others);
                break;
            }
        }
    }
    __syncthreads();
    if (t == 0) {
        const float others = m > 1 ? 2.0f * (float)pairs / ((float)m * (float)(m - 1)) * (float)n : 0.0f;
        acc[ACC_DENSE] = others > DENSE ? 1ull : 0ull;
    }
}
static_assert(2 * SLOTS == 4 * SAMPLES, "one 16-byte store per thread clears the table");

// Cell sizes of the two searches.
struct Cells {
    float r, half_r;   // 1.001 R and half of it
};
__device__ __forceinline__ float cell_size(const Cells& c, const unsigned long long* acc)
{
    return acc[ACC_DENSE] ? c.half_r : c.r;
}

// Neighbouring points of a frame tend to share a bucket, and atomics on one
// address take turns: of every run of lanes with the same bucket (among the
// active lanes of the wave, in lane order) the first lane acts for all n, and
// rank is the lane's place in its run.
struct Run {
    bool first;
    int n, rank, leader;
};
__device__ __forceinline__ Run same_bucket_run(unsigned b)
{
    const int lane = threadIdx.x & 63;
    const uint64_t act = __ballot(1);
    const uint64_t below = act & ((1ull << lane) - 1ull);
    const int prev = below ? 63 - __clzll(below) : -1;
    const unsigned pb = __shfl(b, prev < 0 ? lane : prev, 64);
    const bool first = prev < 0 || pb != b;
    const uint64_t heads = __ballot(first);
    const uint64_t upto = heads & ((lane < 63 ? 1ull << (lane + 1) : 0ull) - 1ull);
    const uint64_t after = heads & ~((lane < 63 ? 1ull << (lane + 1) : 0ull) - 1ull);
    const int leader = 63 - __clzll(upto);
    const int next = after ? __ffsll((unsigned long long)after) - 1 : 64;
    const uint64_t from = ~0ull << leader;
    Run r;
    r.first = first;
    r.leader = leader;
    r.n = __popcll(act & from & (next < 64 ? (1ull << next) - 1ull : ~0ull));
    r.rank = __popcll(act & from & ((1ull << lane) - 1ull));
    return r;
}

// Counts the finite points per bucket; a point that is not finite gets its
// mean distance (NaN) here, since the neighbour search never sees it.
__global__ void k_sor_count(const float* __restrict__ pts, int64_t n, Cells cells, Wrap w,
                            unsigned* __restrict__ count, float* __restrict__ dmean,
                            const unsigned long long* __restrict__ acc)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float x = pts[3 * i], y = pts[3 * i + 1], z = pts[3 * i + 2];
    if (!finite3(x, y, z)) {
        dmean[i] = __builtin_nanf("");
        return;
    }
    const float h = cell_size(cells, acc);
    const unsigned b = bucket(cell_of(x, h), cell_of(y, h), cell_of(z, h), w);
    const Run r = same_bucket_run(b);
    if (r.first) atomicAdd(count + b, (unsigned)r.n);
}

// Places the buckets in the sorted points: {first point, points} per bucket.
// A work-group scans 4096 consecutive buckets (whole x rows of cells) and
// takes their points' places from a counter, so the order of the blocks
// varies, but a row's buckets follow each other.
constexpr int PLACE_PER = 4;                    // uint4 of counts per thread
__global__ __launch_bounds__(256) void k_sor_place(const uint4* __restrict__ count, int T4,
                                                   uint4* __restrict__ table,
                                                   unsigned long long* __restrict__ acc)
{
    __shared__ unsigned wsum[4], base;
    const int i0 = (blockIdx.x * 256 + threadIdx.x) * PLACE_PER;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint4 v[PLACE_PER];
    unsigned t = 0;
#pragma unroll
    for (int k = 0; k < PLACE_PER; ++k) {
        v[k] = i0 + k < T4 ? count[i0 + k] : make_uint4(0u, 0u, 0u, 0u);
        t += v[k].x + v[k].y + v[k].z + v[k].w;
    }
    unsigned s = t;   // inclusive scan of the wave
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned u = __shfl_up(s, off, 64);
        s += lane >= off ? u : 0u;
    }
    if (lane == 63) wsum[wave] = s;
    __syncthreads();
    if (threadIdx.x == 0)
        base = (unsigned)atomicAdd(acc + ACC_GIVEN, (unsigned long long)(wsum[0] + wsum[1] + wsum[2] + wsum[3]));
    __syncthreads();
    unsigned first = base + s - t;
    for (int k = 0; k < wave; ++k) first += wsum[k];
#pragma unroll
    for (int k = 0; k < PLACE_PER; ++k) {
        if (i0 + k >= T4) break;
        const unsigned a = first, b = a + v[k].x, c = b + v[k].y, d = c + v[k].z;
        table[2 * (i0 + k)] = make_uint4(a, v[k].x, b, v[k].y);
        table[2 * (i0 + k) + 1] = make_uint4(c, v[k].z, d, v[k].w);
        first = d + v[k].w;
    }
}

// Takes the places of a bucket from its last one down: count is used up.
__global__ void k_sor_scatter(const float* __restrict__ pts, int64_t n, Cells cells, Wrap w,
                              const uint2* __restrict__ table, unsigned* __restrict__ count,
                              float4* __restrict__ spts, const unsigned long long* __restrict__ acc)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float x = pts[3 * i], y = pts[3 * i + 1], z = pts[3 * i + 2];
    if (!finite3(x, y, z)) return;
    const float h = cell_size(cells, acc);
    const unsigned b = bucket(cell_of(x, h), cell_of(y, h), cell_of(z, h), w);
    const Run r = same_bucket_run(b);
    unsigned left = 0;   // points of the bucket still to place before the run's
    if (r.first) left = atomicSub(count + b, (unsigned)r.n);
    left = __shfl(left, r.leader, 64);
    spts[table[b].x + left - 1u - (unsigned)r.rank] = make_float4(x, y, z, __int_as_float((int)i));
}

__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// The mean distance from the k smallest squared distances, in ascending order.
template <int K>
__device__ __forceinline__ float mean_distance(const float (&best)[K], int found, int k, float R)
{
    const int m = min(found, k);
    float sum = 0.0f;
#pragma unroll
    for (int u = 0; u < K; ++u)
        if (u < m) sum = sum + sqrtf(best[u]);
    sum = sum + (float)(k - m) * R;
    return sum / (float)k;
}

// A wave's share of the statistics: integer sums, reduced per wave before one
// atomic addition per wave, so the order of the waves does not matter.
__device__ __forceinline__ void add_statistics(bool active, float d, unsigned long long* __restrict__ acc)
{
    const double dd = (double)d;
    const unsigned long long a1 = wave_sum(active ? (unsigned long long)(long long)rint(dd * SCALE1) : 0ull);
    const unsigned long long a2 = wave_sum(active ? (unsigned long long)(long long)rint(dd * dd * SCALE2) : 0ull);
    const unsigned long long a3 = wave_sum(active ? 1ull : 0ull);
    if ((threadIdx.x & 63) == 0 && a3) {
        unsigned long long* a = acc + (blockIdx.x % ACC_SLOTS) * ACC_LINE;
        atomicAdd(a + 0, a1);
        atomicAdd(a + 1, a2);
        atomicAdd(a + 2, a3);
    }
}

// The search for clouds with many points per cell of R, where taking all points
// of 27 such cells costs more than looking for the near ones.  One thread per
// finite point in bucket order.  A query visits its own cell, then the 25 x runs
// (dy, dz in -2..2) of the 5 x 5 x 5 cells around it, nearest first, each run a
// contiguous range of cells dx in lo..hi (its own cell left out of the own run).
// Exact as above.  Once k neighbours are in hand, a cell whose box (widened by a
// rounding slack) lies farther than the current k-th nearest is left out: its
// points cannot change the k smallest distances, and the count m = min(found, k)
// is already k.  The visiting order changes nothing: the k smallest values are
// summed in ascending order.  Bound by the latency of the candidates' loads.
template <int K>
__device__ __forceinline__ float search_dense(const float4 P, int k, float R, float h, const Wrap& w,
                                              const uint2* __restrict__ table, const float4* __restrict__ spts)
{
    const int i = __float_as_int(P.w);
    const float px = P.x, py = P.y, pz = P.z;
    const float rr = R * R;
    const int cx = cell_of(px, h), cy = cell_of(py, h), cz = cell_of(pz, h);
    // a point's cell can differ from its coordinates' box by rounding;
    // the pruning bound below is shrunk by this slack
    const float slack = 1e-4f * h + 1e-6f * (fabsf(px) + fabsf(py) + fabsf(pz));
    float best[K];
#pragma unroll
    for (int u = 0; u < K; ++u) best[u] = __builtin_huge_valf();
    int found = 0;
    // candidates e .. e + 3 of a range that ends at e1
    auto take = [&](const float4 (&q)[4], unsigned e, unsigned e1) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (e + u >= e1 || __float_as_int(q[u].w) == i) continue;
            const float ex = q[u].x - px, ey = q[u].y - py, ez = q[u].z - pz;
            const float sd = (ex * ex + ey * ey) + ez * ez;
            if (!(sd <= rr)) continue;
            ++found;
            // no smaller than the largest kept value: best[] would not change
            if (sd >= best[K - 1]) continue;
#pragma unroll
            for (int v = K - 1; v > 0; --v) best[v] = __builtin_amdgcn_fmed3f(best[v - 1], best[v], sd);
            best[0] = fminf(best[0], sd);
        }
    };
    // two sets of four candidates in turn, the next one in flight: the local memory
    // of the other search leaves only 13 waves per CU to cover the loads
    auto scan = [&](unsigned e0, unsigned e1) {
        if (e0 >= e1) return;
        float4 qa[4], qb[4];
        auto fetch = [&](float4 (&q)[4], unsigned e) {
            if (e < e1) {
#pragma unroll
                for (int u = 0; u < 4; ++u) q[u] = spts[min(e + u, e1 - 1)];
            }
        };
        fetch(qa, e0);
        for (unsigned e = e0; e < e1; e += 8) {
            fetch(qb, e + 4);
            take(qa, e, e1);
            fetch(qa, e + 8);
            take(qb, e + 4, e1);
        }
    };
    // the cells x0..x1 (offsets from cx, x0 <= x1) of one row: one range,
    // or two where the run wraps round the table
    auto scan_cells = [&](unsigned row, int x0, int x1) {
        const unsigned xs = (unsigned)(cx + x0) & w.mx, xe = (unsigned)(cx + x1) & w.mx;
        const bool wraps = xs > xe;
        const uint2 c = table[row | (wraps ? w.mx : xe)];
        unsigned r0 = table[row | xs].x, r1 = c.x + c.y, s0 = 0, s1 = 0;
        if (wraps) {
            const uint2 b = table[row | xe];
            s0 = table[row].x;
            s1 = b.x + b.y;
        }
#pragma unroll 1
        for (int part = 0; part < 2; ++part) {
            scan(r0, r1);
            r0 = s0;
            r1 = s1;
        }
    };
    // distance from the point to the box of the cell at offset o along one
    // axis (0 for its own cell), less the slack
    auto gap = [&](int o, int cc, float pp) {
        const float lo = (float)(cc + o) * h, hi = (float)(cc + o + 1) * h;
        const float gg = o < 0 ? pp - hi : (o > 0 ? lo - pp : 0.0f);
        return fmaxf(gg - slack, 0.0f);
    };
    auto kth = [&]() {
        float v = __builtin_huge_valf();
#pragma unroll
        for (int u = 0; u < K; ++u)
            if (u == k - 1) v = best[u];
        return found >= k ? v : __builtin_huge_valf();
    };
    // the own cell
    scan_cells(bucket(0, cy, cz, w), 0, 0);
    // the 25 runs, nearest first: (dy, dz) by |dy| + |dz|, then max
    constexpr int RY[25] = {0, -1, 1, 0, 0, -1, 1, -1, 1, -2, 2, 0, 0, -2, 2, -2, 2, -1, 1, -1, 1, -2, 2, -2, 2};
    constexpr int RZ[25] = {0, 0, 0, -1, 1, -1, -1, 1, 1, 0, 0, -2, 2, -1, -1, 1, 1, -2, -2, 2, 2, -2, -2, 2, 2};
#pragma unroll 1
    for (int r = 0; r < 25; ++r) {
        const int oy = RY[r], oz = RZ[r];
        const float gy = gap(oy, cy, py), gz = gap(oz, cz, pz);
        const float base = gy * gy + gz * gz;
        const float kb = kth();
        if (base > kb) continue;
        // the x offsets still within reach: gaps grow with |dx|
        int x0 = -2, x1 = 2;
        while (x0 < 0) {
            const float g = gap(x0, cx, px);
            if (base + g * g <= kb) break;
            ++x0;
        }
        while (x1 > 0) {
            const float g = gap(x1, cx, px);
            if (base + g * g <= kb) break;
            --x1;
        }
        const unsigned row = bucket(0, cy + oy, cz + oz, w);
        if (r == 0) {   // the own run without the own cell
            if (x0 < 0) scan_cells(row, x0, -1);
            if (x1 > 0) scan_cells(row, 1, x1);
        } else {
            scan_cells(row, x0, x1);
        }
    }
    return mean_distance(best, found, k, R);
}

// One thread per finite point, points in bucket order (neighbouring cells
// sit side by side in spts, so a wave's points share candidate ranges).  A
// query takes the nine x runs (dy, dz in -1..1) of the 3 x 3 x 3 cells around
// it.  That is exact: a point within R lies in one of the 27 cells, whose
// ranges are disjoint, so it is counted once; candidates from cells a whole
// period away lie farther than R and fail the radius test.
//
// Read lane by lane from memory, the candidates (about 65 a point in a depth
// frame, each lane at its own place) cost the texture unit 80 cycles per load
// instruction, 205 us in all.  So a wave first copies what its points need into
// LDS: its points lie in two or three rows of cells, and the points of a row's x
// range in each of the nine rows around it are one contiguous range.  Each lane
// then streams its own nine ranges from LDS four candidates at a time, the next
// four in flight, and keeps the k smallest squared distances sorted in registers,
// one median per kept value and candidate.  307,200 points of a depth frame, R =
// 1 cm: 77 us of the filter's 116.
//
// Points a wave's LDS holds; a wave that needs more reads from memory.  307,200
// points, the whole filter: 116-124 us with 768, 131 with 1024, 148 with 1536 (fewer
// waves per CU).
constexpr int CAP = 768;
// Rows of cells up to which a wave copies: it takes them one after the other, a
// load's latency each, and points that share few rows' candidates gain little.  The
// whole filter with no limit / 16 / 8 / 4: 20,000 points of a frame 52 / 52 / 46 /
// 42 us, 307,200 with R = 5 mm 106 / 100 / 93 / 90, with R = 1 cm 116 with any.
constexpr int COPY_ROWS = 4;
static_assert(3 * CAP >= 36 * 64, "18 ranges per lane");

template <int K>
__global__ __launch_bounds__(64) void k_sor_knn(int k, float R, Cells cells, Wrap w,
                                                const uint2* __restrict__ table,
                                                const float4* __restrict__ spts,
                                                float* __restrict__ dmean,
                                                unsigned long long* __restrict__ acc)
{
    // x, y and z of the wave's points; later a lane's ranges in spts
    __shared__ uint32_t buf[3 * CAP];
    __shared__ uint32_t ranges[9][64];   // a lane's non-empty ranges in buf: first | end << 16
    uint32_t *sx = buf, *sy = buf + CAP, *sz = buf + 2 * CAP;
    const int lane = threadIdx.x;
    const unsigned t = blockIdx.x * 64u + lane;
    const unsigned nfin = (unsigned)acc[ACC_GIVEN];
    const bool active = t < nfin;
    float d = 0.0f;
    const float4 P = active ? spts[t] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    const int i = __float_as_int(P.w);
    if (acc[ACC_DENSE]) {
        if (active) {
            d = search_dense<K>(P, k, R, cells.half_r, w, table, spts);
            dmean[i] = d;
        }
        add_statistics(active, d, acc);
        return;
    }
    const float h = cells.r;
    const float px = P.x, py = P.y, pz = P.z;
    const float rr = R * R;
    const int cx = cell_of(px, h), cy = cell_of(py, h), cz = cell_of(pz, h);
    // the x run in bucket coordinates; where it wraps round the table, the
    // cell on the other side is left for later
    const unsigned xw = (unsigned)cx & w.mx;
    const unsigned xs = xw > 0 ? xw - 1 : 0, xe = min(xw + 1, w.mx);
    constexpr int RY[9] = {0, -1, 1, 0, 0, -1, 1, -1, 1}, RZ[9] = {0, 0, 0, -1, 1, -1, -1, 1, 1};
    unsigned e0[9], e1[9];
#pragma unroll
    for (int r = 0; r < 9; ++r) {
        e0[r] = e1[r] = 0;
        if (active) {
            const unsigned row = bucket(0, cy + RY[r], cz + RZ[r], w);
            e0[r] = table[row | xs].x;
            const uint2 c = table[row | xe];
            e1[r] = c.x + c.y;
        }
    }
    // ---- the wave's candidates into LDS: for every row of cells that its
    // lanes lie in (consecutive lanes, ascending x), the nine rows around it from
    // the first lane's first cell to the last lane's last
    const unsigned key = bucket(0, cy, cz, w);
    int used = 0, nr = 0, self = 0;
    const unsigned before = __shfl_up(key, 1, 64);   // lanes of a row follow each other
    bool fits = __popcll(__ballot(active && (lane == 0 || before != key))) <= COPY_ROWS;
    for (uint64_t todo = __ballot(active); todo && fits;) {
        const int first = __ffsll((unsigned long long)todo) - 1;
        const unsigned gk = __builtin_amdgcn_readlane(key, first);
        const bool mine = active && key == gk;
        const uint64_t grp = __ballot(mine) & todo;
        const int last = 63 - __clzll(grp);
        todo &= ~grp;
        unsigned s0[9];
        int len[9], total = 0;
#pragma unroll
        for (int r = 0; r < 9; ++r) {
            s0[r] = __builtin_amdgcn_readlane(e0[r], first);
            const unsigned n = (unsigned)__builtin_amdgcn_readlane(e1[r], last) - s0[r];
            len[r] = (int)min(n, (unsigned)CAP + 1u);
            total += len[r];
        }
        if (used + total > CAP) {
            fits = false;
            break;
        }
        float4 q[9];
#pragma unroll
        for (int r = 0; r < 9; ++r)
            if (lane < len[r]) q[r] = spts[s0[r] + lane];
#pragma unroll
        for (int r = 0; r < 9; ++r) {
            if (lane < len[r]) {
                sx[used + lane] = __float_as_uint(q[r].x);
                sy[used + lane] = __float_as_uint(q[r].y);
                sz[used + lane] = __float_as_uint(q[r].z);
            }
            for (int c = 64 + lane; c < len[r]; c += 64) {
                const float4 v = spts[s0[r] + c];
                sx[used + c] = __float_as_uint(v.x);
                sy[used + c] = __float_as_uint(v.y);
                sz[used + c] = __float_as_uint(v.z);
            }
            if (mine) {
                if (r == 0) self = (int)(t - s0[0]) + used;
                if (e0[r] < e1[r])
                    ranges[nr++][lane] = (e0[r] - s0[r] + used) | ((e1[r] - s0[r] + used) << 16);
            }
            used += len[r];
        }
    }
    __syncthreads();
    if (active) {
        float best[K];
#pragma unroll
        for (int u = 0; u < K; ++u) best[u] = __builtin_huge_valf();
        int found = 0;
        // one candidate; best[] stays sorted ascending, one median per kept value
        auto take = [&](float x, float y, float z, bool other) {
            const float ex = x - px, ey = y - py, ez = z - pz;
            const float sd = (ex * ex + ey * ey) + ez * ez;
            const bool ok = sd <= rr && other;
            found += ok;
            const float v = ok ? sd : __builtin_huge_valf();
#pragma unroll
            for (int u = K - 1; u > 0; --u) best[u] = __builtin_amdgcn_fmed3f(best[u - 1], best[u], v);
            best[0] = fminf(best[0], v);
        };
        int ng = 0;   // ranges of spts left to read from memory, in buf
        auto later = [&](unsigned g0, unsigned g1) {
            if (g0 < g1) {
                buf[(2 * ng) * 64 + lane] = g0;
                buf[(2 * ng + 1) * 64 + lane] = g1;
                ++ng;
            }
        };
        if (fits) {
            // a slot past its range's end reads the point itself, which is no
            // candidate
            constexpr int S = 4;
            int ri = 0, cur = 0, end = 0;
            int at[S];
            float qx[S], qy[S], qz[S];
            auto fetch = [&]() -> bool {
                if (cur >= end) {
                    if (ri >= nr) return false;
                    const uint32_t g = ranges[ri++][lane];
                    cur = (int)(g & 0xFFFFu);
                    end = (int)(g >> 16);
                }
#pragma unroll
                for (int u = 0; u < S; ++u) {
                    at[u] = cur + u < end ? cur + u : self;
                    qx[u] = __uint_as_float(sx[at[u]]);
                    qy[u] = __uint_as_float(sy[at[u]]);
                    qz[u] = __uint_as_float(sz[at[u]]);
                }
                cur += S;
                return true;
            };
            bool more = fetch();
            while (more) {
                float x[S], y[S], z[S];
                bool other[S];
#pragma unroll
                for (int u = 0; u < S; ++u) {
                    x[u] = qx[u];
                    y[u] = qy[u];
                    z[u] = qz[u];
                    other[u] = at[u] != self;
                }
                more = fetch();
#pragma unroll
                for (int u = 0; u < S; ++u) take(x[u], y[u], z[u], other[u]);
            }
        } else {
#pragma unroll
            for (int r = 0; r < 9; ++r) later(e0[r], e1[r]);
        }
        // from here on a lane overwrites candidates: every lane is past its own
        __builtin_amdgcn_wave_barrier();
        if (xw == 0 || xw == w.mx) {   // the cell on the other side of the table
            uint2 c[9];
#pragma unroll
            for (int r = 0; r < 9; ++r) c[r] = table[bucket(0, cy + RY[r], cz + RZ[r], w) | (xw == 0 ? w.mx : 0u)];
#pragma unroll
            for (int r = 0; r < 9; ++r) later(c[r].x, c[r].x + c[r].y);
        }
#pragma unroll 1
        for (int g = 0; g < ng; ++g) {
            const unsigned g0 = buf[(2 * g) * 64 + lane], g1 = buf[(2 * g + 1) * 64 + lane];
#pragma unroll 1
            for (unsigned e = g0; e < g1; e += 4) {
                float4 q[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) q[u] = spts[min(e + u, g1 - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u) take(q[u].x, q[u].y, q[u].z, e + u < g1 && __float_as_int(q[u].w) != i);
            }
        }
        d = mean_distance(best, found, k, R);
        dmean[i] = d;
    }
    add_statistics(active, d, acc);
}

// By whole waves: lane l adds up slot l.
__device__ __forceinline__ double sor_threshold(const unsigned long long* acc, double alpha,
                                                double* mu_out, double* sigma_out)
{
    static_assert(ACC_SLOTS == 64, "one slot per lane");
    const unsigned long long* a = acc + (threadIdx.x & 63) * ACC_LINE;
    const long long S1 = (long long)wave_sum(a[0]), S2 = (long long)wave_sum(a[1]), cnt = (long long)wave_sum(a[2]);
    double mu = 0.0, sigma = 0.0;
    if (cnt > 0) mu = (double)S1 / SCALE1 / (double)cnt;
    if (cnt > 1) {
        const double var = ((double)S2 / SCALE2 - (double)cnt * mu * mu) / (double)(cnt - 1);
        sigma = var > 0.0 ? sqrt(var) : 0.0;
    }
    *mu_out = mu;
    *sigma_out = sigma;
    return mu + alpha * sigma;
}

__global__ void k_sor_keep(const float* __restrict__ pts, int64_t n, const float* __restrict__ dmean,
                           const unsigned long long* __restrict__ acc, double alpha,
                           uint8_t* __restrict__ keep, double* __restrict__ stats)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double mu, sigma;
    const double thr = sor_threshold(acc, alpha, &mu, &sigma);
    if (i == 0 && stats) {
        stats[0] = mu;
        stats[1] = sigma;
        stats[2] = thr;
    }
    if (i >= n) return;
    const bool fin = finite3(pts[3 * i], pts[3 * i + 1], pts[3 * i + 2]);
    keep[i] = fin && (double)dmean[i] <= thr ? 1 : 0;
}

}  // namespace
}  // namespace edtmi

using namespace edtmi;

extern "C" {

size_t edt_outlier_workspace_bytes(int64_t n_points)
{
    if (n_points < 0 || n_points > EDT_OUTLIER_MAX_POINTS) return 0;
    return sor_layout(n_points).total + (size_t)std::max<int64_t>(n_points, 1) * 4;
}

constexpr double OUTLIER_SUM2_MAX = 32000.0;     // m^2, below 2^15
constexpr double OUTLIER_SUM1_MAX = 8000000.0;   // m, below 2^23

int edt_outlier_filter(const float* pts, int64_t n, int32_t k, float radius, float alpha,
                       uint8_t* keep, float* mean_dist, double* stats, void* ws, size_t ws_bytes,
                       void* stream)
{
    if (n < 0 || n > EDT_OUTLIER_MAX_POINTS || (n > 0 && (!pts || !keep)) || !ws) {
        set_error("edt_outlier_filter: bad pointer or point count (0..%d)", EDT_OUTLIER_MAX_POINTS);
        return EDT_ERR_ARG;
    }
    if (k < 1 || k > KMAX || !(radius > 0.0f) || !std::isfinite(radius) || !std::isfinite(alpha)) {
        set_error("edt_outlier_filter: need 1 <= k <= %d, a finite radius > 0 and a finite alpha", KMAX);
        return EDT_ERR_ARG;
    }
    // every d_i is at most the radius, so the fixed-point sums (d_i in units
    // of 2^-40, d_i^2 in units of 2^-48) stay below 2^63 while n * radius^2
    // and n * radius stay below 2^15 m^2 and 2^23 m; a margin keeps rounding
    // of the last unit inside
    if ((double)n * (double)radius * (double)radius >= OUTLIER_SUM2_MAX ||
        (double)n * (double)radius >= OUTLIER_SUM1_MAX) {
        set_error("edt_outlier_filter: n * radius^2 = %g m^2 reaches %g (the exact sums would overflow)",
                  (double)n * (double)radius * (double)radius, OUTLIER_SUM2_MAX);
        return EDT_ERR_ARG;
    }
    if (ws_bytes < edt_outlier_workspace_bytes(n)) {
        set_error("edt_outlier_filter: workspace of %zu bytes is below %zu", ws_bytes,
                  edt_outlier_workspace_bytes(n));
        return EDT_ERR_WORKSPACE;
    }
    const SorLayout L = sor_layout(n);
    char* w = static_cast<char*>(ws);
    unsigned* count = reinterpret_cast<unsigned*>(w + L.count);
    uint2* table = reinterpret_cast<uint2*>(w + L.table);
    float4* spts = reinterpret_cast<float4*>(w + L.spts);
    unsigned long long* acc = reinterpret_cast<unsigned long long*>(w + L.acc);
    float* dm = mean_dist ? mean_dist : reinterpret_cast<float*>(w + L.total);
    const int T = (int)L.tmask + 1;
    const Cells cells{radius * 1.001f, radius * 0.5005f};
    const hipStream_t st = as_stream(stream);
    const unsigned pblocks = (unsigned)((std::max<int64_t>(n, 1) + 255) / 256);
    const int est = n > FEW ? 1 : 0;
    hipLaunchKernelGGL(k_sor_zero, dim3(est + (std::max(T / 4, ACC_DENSE + 1) + SAMPLES - 1) / SAMPLES), dim3(SAMPLES), 0, st,
                       reinterpret_cast<uint4*>(count), T / 4, acc, est, pts, n, std::max<int64_t>(1, n / SAMPLES), radius);
    int rc = check_launch("k_sor_zero");
    if (rc) return rc;
    if (n > 0) {
        hipLaunchKernelGGL(k_sor_count, dim3(pblocks), dim3(256), 0, st, pts, n, cells, L.wrap, count, dm, acc);
        if ((rc = check_launch("k_sor_count"))) return rc;
        hipLaunchKernelGGL(k_sor_place, dim3((T / 4 + 256 * PLACE_PER - 1) / (256 * PLACE_PER)), dim3(256), 0, st,
                           reinterpret_cast<const uint4*>(count), T / 4, reinterpret_cast<uint4*>(table), acc);
        if ((rc = check_launch("k_sor_place"))) return rc;
        hipLaunchKernelGGL(k_sor_scatter, dim3(pblocks), dim3(256), 0, st, pts, n, cells, L.wrap, table, count, spts,
                           acc);
        if ((rc = check_launch("k_sor_scatter"))) return rc;
        const dim3 waves((unsigned)((n + 63) / 64));
        if (k <= 8)
            hipLaunchKernelGGL(k_sor_knn<8>, waves, dim3(64), 0, st, (int)k, radius, cells, L.wrap, table, spts, dm,
                               acc);
        else
            hipLaunchKernelGGL(k_sor_knn<KMAX>, waves, dim3(64), 0, st, (int)k, radius, cells, L.wrap, table, spts, dm,
                               acc);
        if ((rc = check_launch("k_sor_knn"))) return rc;
    }
    hipLaunchKernelGGL(k_sor_keep, dim3(pblocks), dim3(256), 0, st, pts, n, dm, acc, (double)alpha,
                       keep, stats);
    return check_launch("k_sor_keep");
}

}  // extern "C"
