// The exact squared EDT on gfx950 for one map: the xy-tile kernel (steps 1-3
// of Sec. III-C in every slice) and the z-tile kernel (step 4), their
// launchers and the tile heuristics.  The tile code is in edt_search.h (maps
// with every axis up to 512) and edt_tiles.h (every shape and tiling).
#include <algorithm>
#include <atomic>

#include "edt_search.h"

namespace edtmi {

namespace {

using namespace tiles;

// Map of launch tile T (the maps' tile ranges are consecutive).
__device__ __forceinline__ int map_of(const EdtMapSet& s, int T)
{
    int m = 0;
    while (m + 1 < s.n && s.m[m + 1].begin <= T) ++m;
    return __builtin_amdgcn_readfirstlane(m);
}

// True while the map's gate (if any) holds 0: its work-groups return at once.
__device__ __forceinline__ bool gated_off(const EdtMap& d)
{
    return d.gate && __builtin_amdgcn_readfirstlane(*d.gate) == 0;
}

template <int TW, bool WIDE, int NTX>
__global__ __launch_bounds__(NTX) void k_edt_xy(EdtMapSet s)
{
    extern __shared__ uint32_t lds[];
    // the tiles of a slice read the same occupancy bytes: chunks of 16 tiles
    // (one or two slices) share an XCD's L2, and the slices, whose work is
    // very uneven, rotate over the XCDs
    const int T = xcd_chunk_remap(blockIdx.x, s.total, 16);
    const EdtMap& d = s.m[map_of(s, T)];
    if (gated_off(d)) return;
    edt_xy_tile<TW, WIDE, NTX>(d.occ, reinterpret_cast<uint32_t*>(d.site), d.nx, d.ny, d.nz, d.ntx,
                               T - d.begin, lds);
}

// Row records (step 1) of every map of the set: each wave takes
// record_rows_per_wave(nx) whole rows of one map, four waves per work-group;
// s.m[i].begin is the map's first wave.
__global__ __launch_bounds__(256) void k_row_records(EdtMapSet s)
{
    const int wv = __builtin_amdgcn_readfirstlane((int)blockIdx.x * 4 + (int)(threadIdx.x >> 6));
    if (wv >= s.total) return;
    const EdtMap& d = s.m[map_of(s, wv)];
    if (gated_off(d)) return;
    const int per = record_rows_per_wave(d.occ, d.nx);
    const int row0 = (wv - d.begin) * per;
    const int nrows = min(per, d.ny * d.nz - row0);
    if (record_words(d.occ, d.nx))
        row_summary_words(d.occ, d.nx, (size_t)row0, nrows, row_records(d.d2, d.nx, d.ny, d.nz));
    else
        row_summary(d.occ, d.nx, (size_t)row0, nrows, row_records(d.d2, d.nx, d.ny, d.nz));
}

// Steps 2-3 from the row records.
template <int TW, bool WIDE, int NTX>
__global__ __launch_bounds__(NTX) void k_edt_xy_rows(EdtMapSet s)
{
    extern __shared__ uint32_t lds[];
    // as in k_edt_xy: chunks of 16 tiles per XCD, rotating over the XCDs
    const int T = xcd_chunk_remap(blockIdx.x, s.total, 16);
    const EdtMap& d = s.m[map_of(s, T)];
    if (gated_off(d)) return;
    edt_xy_tile_rows<TW, WIDE, NTX>(row_records(d.d2, d.nx, d.ny, d.nz), reinterpret_cast<uint32_t*>(d.site),
                                    d.nx, d.ny, d.ntx, T - d.begin, lds);
}

template <int TW, bool WIDE, int NTZ>
__global__ __launch_bounds__(NTZ) void k_edt_z(EdtMapSet s)
{
    extern __shared__ uint32_t lds[];
    // tiles narrower than 64 columns share cache lines with their neighbours:
    // the tiles of 64 columns of a row stay on one XCD, and rows (whose work
    // is very uneven) rotate over all eight
    const int T = TW >= 64 ? (int)blockIdx.x : xcd_chunk_remap(blockIdx.x, s.total, 64 / TW);
    const EdtMap& d = s.m[map_of(s, T)];
    if (gated_off(d)) return;
    edt_z_tile<TW, WIDE, NTZ>(d.d2, d.site, d.nx, d.ny, d.nz, d.ntx, T - d.begin, lds);
}

// Search tiles (edt_search.h).  A launch for one map takes the map itself as
// its argument (Set = EdtMap): one scalar load brings all of it, where a set
// costs a chain of dependent ones (the count, the begins, the gate, the map).
__device__ __forceinline__ const EdtMap& tile_map(const EdtMap& m, int) { return m; }
__device__ __forceinline__ const EdtMap& tile_map(const EdtMapSet& s, int T) { return s.m[map_of(s, T)]; }

// Occupancy bits of every map, 16 * 256 * BITS_U voxels per work-group
// (d.begin: the map's first work-group).
template <class Set>
__global__ __launch_bounds__(256) void k_map_bits(Set s)
{
    const int B = (int)blockIdx.x;
    const EdtMap& d = tile_map(s, B);
    if (gated_off(d)) return;
    search::map_bits(d.occ, (int64_t)d.nx * d.ny * d.nz,
                     ((int64_t)(B - d.begin) * 4 + search::band_of_wave()) * (64 * search::BITS_U),
                     reinterpret_cast<uint32_t*>(d.d2));
}

template <int NMAX, int C, int BAND, class Set>
__global__ __launch_bounds__(64 * NMAX / BAND) void k_edt_z_search(Set s, int waves, int)
{
    extern __shared__ uint32_t lds[];
    const int T = (int)blockIdx.x;
    const EdtMap& d = tile_map(s, T);
    if (gated_off(d)) return;
    search::ZBand<BAND> b;
    b.load(d.d2, d.site, d.nx, d.ny, d.nz, T - d.begin, search::band_of_wave() * BAND);
    search::z_stage<C>(b, BAND * waves, lds);
    __syncthreads();
    search::z_band<NMAX, C, BAND>(b, BAND * waves, lds);
}

// The same for lines of more than 256 positions, whose tile takes most of a
// CU's local memory: one work-group per CU walks over the tiles, and the sites
// of its next tile are on their way while it searches the present one, which a
// second resident work-group does for shorter lines.  A tile reads and writes
// its own columns only, so the loads of one may pass the stores of another.
// z pass of 512^3 blobs 457 -> 420 us, of a 256 x 256 x 512 frame 117 -> 113; 265 us
// of the 420 are VALU issue, the rest is mostly waiting for a tile's slowest band.
template <int NMAX, int C, int BAND, class Set>
__global__ __launch_bounds__(64 * NMAX / BAND) void k_edt_z_stream(Set s, int waves, int total)
{
    extern __shared__ uint32_t lds[];
    const int q0 = search::band_of_wave() * BAND, np = BAND * waves;
    search::ZBand<BAND> next;
    auto fetch = [&](int T) -> bool {   // the same for the whole work-group
        const EdtMap& d = tile_map(s, T);
        if (gated_off(d)) return false;
        next.load(d.d2, d.site, d.nx, d.ny, d.nz, T - d.begin, q0);
        return true;
    };
    int T = (int)blockIdx.x;
    bool on = fetch(T);
    for (;;) {
        const search::ZTile tile = next;
        if (on) search::z_stage<C>(next, np, lds);
        __syncthreads();
        const bool now = on;
        T += (int)gridDim.x;
        on = T < total && fetch(T);
        if (now) search::z_band<NMAX, C, BAND>(tile, np, lds);
        if (T >= total) return;
        __syncthreads();
    }
}

template <int NMAX, int C, int BAND, class Set>
__global__ __launch_bounds__(64 * NMAX / BAND) void k_edt_xy_search(Set s, int waves, int)
{
    extern __shared__ uint32_t lds[];
    // tiles in launch order: a tile reads 1 bit per voxel and writes whole
    // cache lines, so neighbours share next to nothing, and chunks of tiles per
    // XCD leave some XCDs more of the busy slices than others (48 self maps 449
    // us in chunks of 16, 438 like this; single maps within 3% either way)
    const int T = (int)blockIdx.x;
    const EdtMap& d = tile_map(s, T);
    if (gated_off(d)) return;
    search::xy_tile<NMAX, C, BAND>(reinterpret_cast<const uint32_t*>(d.d2), search::misalignment(d.occ),
                                   d.ntx == 1 ? d.occ : nullptr, (int64_t)d.nx * d.ny * d.nz,
                                   reinterpret_cast<uint32_t*>(d.site), d.nx, d.ny, d.ntx, T - d.begin,
                                   BAND * waves, lds);
}

// Allow dynamic LDS beyond the 64 KiB default (gfx950 has 160 KiB per
// work-group); once per kernel instantiation and device, whose bit in done says so.
using DeviceBits = std::atomic<uint64_t>;
template <typename K>
int allow_lds(K kernel, DeviceBits& done)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0ull;
    if (e == hipSuccess && (done.load(std::memory_order_relaxed) & bit)) return EDT_OK;
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                160 * 1024 - 8192);
    if (e != hipSuccess) {
        set_error("hipFuncSetAttribute: %s", hipGetErrorString(e));
        return EDT_ERR_HIP;
    }
    done.fetch_or(bit, std::memory_order_relaxed);
    return EDT_OK;
}

// Step 1 once per row when every map's rows are at least 256 voxels long,
// else inside every tile from the slice.  The records need rows of 64 or more
// to fit in d2; below 256 a slice is staged by few tiles, and the extra
// kernel costs more than the staging it saves (measured on maps of 64-256).
bool rows_first(const EdtMapSet& s)
{
    for (int i = 0; i < s.n; ++i)
        if (s.m[i].nx < 256 || !s.m[i].d2) return false;
    return true;
}

// The rows of a map of up to 64 columns are read by one tile each, which takes the
// bytes themselves; the others' bits are written first, into d2.  A call for such
// maps alone is two launches: 20^3 maps with five sites 14.4 us with a pass over the
// bits, 11.7 like this; 64^3 14.2 and 11.6.
bool takes_bits(const EdtMap& m) { return m.nx > 64; }

// The search tiles take maps with every axis <= 512.
bool search_xy_ok(const EdtMapSet& s)
{
    if (s.wide) return false;
    for (int i = 0; i < s.n; ++i)
        if (takes_bits(s.m[i]) && !s.m[i].d2) return false;
    return true;
}

// Step 1 of every map of the set once per row, into the maps' d2 buffers.
int launch_row_records(const EdtMapSet& s, hipStream_t st)
{
    static thread_local EdtMapSet r;   // the maps counted in waves (2.3 KiB: off the stack)
    r = s;
    int waves = 0;
    for (int i = 0; i < s.n; ++i) {
        const int per = record_rows_per_wave(s.m[i].occ, s.m[i].nx);
        r.m[i].begin = waves;
        waves += (s.m[i].ny * s.m[i].nz + per - 1) / per;
    }
    r.total = waves;
    hipLaunchKernelGGL(k_row_records, dim3((waves + 3) / 4), dim3(256), 0, st, r);
    return check_launch("k_row_records");
}

// The occupancy bits of the maps of the set that need them, into their d2 buffers.
int launch_map_bits(const EdtMapSet& s, hipStream_t st)
{
    static thread_local EdtMapSet r;
    int blocks = 0;
    r.n = 0;
    for (int i = 0; i < s.n; ++i) {
        if (!takes_bits(s.m[i])) continue;
        const int64_t n = (int64_t)s.m[i].nx * s.m[i].ny * s.m[i].nz + search::misalignment(s.m[i].occ);
        r.m[r.n] = s.m[i];
        r.m[r.n++].begin = blocks;
        blocks += (int)((n + 16 * 256 * search::BITS_U - 1) / (16 * 256 * search::BITS_U));
    }
    if (r.n == 0) return EDT_OK;
    r.total = blocks;
    if (r.n == 1) hipLaunchKernelGGL(k_map_bits<EdtMap>, dim3(blocks), dim3(256), 0, st, r.m[0]);
    else hipLaunchKernelGGL(k_map_bits<EdtMapSet>, dim3(blocks), dim3(256), 0, st, r);
    return check_launch("k_map_bits");
}

// CUs of the current device, 0 on an error.
int cu_count()
{
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess)
        return n;
    set_error("the device's CU count could not be read");
    return 0;
}

// One pass of the search tiles; n = the longest line of the pass.
template <int NMAX, int BAND>
int launch_search_t(const EdtMapSet& s, bool z_pass, int n, hipStream_t st)
{
    // chunks of 4 sites; of 8 beyond 256 positions, where the chunk minima of
    // a z work-group would not fit into the local memory beside its sites, and
    // testing twice the chunks costs the xy pass more than it saves
    // (512 x 512 x 128 frame 84 against 93 us, 512^3 blobs 431 against 436)
    constexpr int C = NMAX <= 256 ? 4 : 8;
    const int nw = (n + BAND - 1) / BAND, np = nw * BAND;
    auto go = [&](auto kernel, DeviceBits& done, size_t lds, const auto& arg, const char* name, int grid) -> int {
        int rc = allow_lds(kernel, done);
        if (rc) return rc;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(64 * nw), lds, st, arg, nw, s.total);
        return check_launch(name);
    };
    static DeviceBits done[4];
    if (z_pass) {
        const size_t lds = (size_t)(np + np / C) * 256;
        if constexpr (NMAX > 256) {
            const int n_cu = cu_count();
            if (!n_cu) return EDT_ERR_HIP;
            const int grid = std::min(s.total, n_cu);
            return s.n == 1 ? go(k_edt_z_stream<NMAX, C, BAND, EdtMap>, done[0], lds, s.m[0], "k_edt_z_stream", grid)
                            : go(k_edt_z_stream<NMAX, C, BAND, EdtMapSet>, done[1], lds, s, "k_edt_z_stream", grid);
        } else {
            return s.n == 1
                       ? go(k_edt_z_search<NMAX, C, BAND, EdtMap>, done[0], lds, s.m[0], "k_edt_z_search", s.total)
                       : go(k_edt_z_search<NMAX, C, BAND, EdtMapSet>, done[1], lds, s, "k_edt_z_search", s.total);
        }
    }
    const size_t lds = (size_t)(np + np / C) * 128;
    return s.n == 1 ? go(k_edt_xy_search<NMAX, C, BAND, EdtMap>, done[2], lds, s.m[0], "k_edt_xy_search", s.total)
                    : go(k_edt_xy_search<NMAX, C, BAND, EdtMapSet>, done[3], lds, s, "k_edt_xy_search", s.total);
}

int launch_search(const EdtMapSet& s, bool z_pass, hipStream_t st)
{
    const int n = z_pass ? s.nz_max : s.ny_max;
    // Bands of 32 rows or 16 slices keep 8 waves per SIMD resident with the
    // local memory of a work-group of 128 or 256 positions (z bands of 32 only
    // 4: 512 x 512 x 128 frame 87 against 76 us).  Launches with fewer waves
    // than that take shorter bands: 64^3 boxes 34 us with bands of 32, 17 with
    // 8; the xy pass of one 256 x 256 x 128 frame 40 us with 32, 36 with 16.
    auto waves = [&](int band) { return (int64_t)s.total * ((n + band - 1) / band); };
    int band = z_pass ? 16 : 32;
    while (band > 8 && waves(band) < 8192) band /= 2;
    if (n <= 64) {
        if (band == 32) return launch_search_t<64, 32>(s, z_pass, n, st);
        return band == 16 ? launch_search_t<64, 16>(s, z_pass, n, st) : launch_search_t<64, 8>(s, z_pass, n, st);
    }
    if (n <= 128) {
        if (band == 32) return launch_search_t<128, 32>(s, z_pass, n, st);
        return band == 16 ? launch_search_t<128, 16>(s, z_pass, n, st) : launch_search_t<128, 8>(s, z_pass, n, st);
    }
    // at most 16 waves per work-group
    if (n <= 256)
        return band == 32 ? launch_search_t<256, 32>(s, z_pass, n, st) : launch_search_t<256, 16>(s, z_pass, n, st);
    return launch_search_t<512, 32>(s, z_pass, n, st);
}

template <int TW, bool WIDE, int NTX>
int launch_xy_w(const EdtMapSet& s, hipStream_t st)
{
    if (TW == 64 && NTX == 512 && !WIDE && search_xy_ok(s)) {
        int rc = launch_map_bits(s, st);
        return rc ? rc : launch_search(s, false, st);
    }
    if (rows_first(s)) {
        int rc = launch_row_records(s, st);
        if (rc) return rc;
        static DeviceBits done_rows;
        rc = allow_lds(k_edt_xy_rows<TW, WIDE, NTX>, done_rows);
        if (rc) return rc;
        hipLaunchKernelGGL((k_edt_xy_rows<TW, WIDE, NTX>), dim3(s.total), dim3(NTX),
                           xy_rows_lds(TW, s.ny_max, NTX), st, s);
        return check_launch("k_edt_xy_rows");
    }
    static DeviceBits done;
    int rc = allow_lds(k_edt_xy<TW, WIDE, NTX>, done);
    if (rc) return rc;
    hipLaunchKernelGGL((k_edt_xy<TW, WIDE, NTX>), dim3(s.total), dim3(NTX), xy_lds(TW, s.ny_max, NTX),
                       st, s);
    return check_launch("k_edt_xy");
}

template <int TW, int NTX>
int launch_xy_tw(const EdtMapSet& s, hipStream_t st)
{
    return s.wide ? launch_xy_w<TW, true, NTX>(s, st) : launch_xy_w<TW, false, NTX>(s, st);
}

template <int TW, bool WIDE, int NTZ>
int launch_z_t(const EdtMapSet& s, hipStream_t st)
{
    if constexpr (TW == 64 && NTZ == 256 && !WIDE) {
        // search tiles: 64 consecutive columns of the xy plane each
        static thread_local EdtMapSet r;
        r = s;
        r.total = 0;
        for (int i = 0; i < s.n; ++i) {
            r.m[i].begin = r.total;
            r.total += (s.m[i].nx * s.m[i].ny + 63) / 64;
        }
        return launch_search(r, true, st);
    } else {
        static DeviceBits done;
        int rc = allow_lds(k_edt_z<TW, WIDE, NTZ>, done);
        if (rc) return rc;
        hipLaunchKernelGGL((k_edt_z<TW, WIDE, NTZ>), dim3(s.total), dim3(NTZ), z_lds(TW, s.nz_max, NTZ), st,
                           s);
        return check_launch("k_edt_z");
    }
}

template <int TW, int NTZ>
int launch_z_tw(const EdtMapSet& s, hipStream_t st)
{
    return s.wide ? launch_z_t<TW, true, NTZ>(s, st) : launch_z_t<TW, false, NTZ>(s, st);
}

// The tiles of every map of the set, ntx column tiles of width tw per row
// of the pass (rows: z slices for xy, y rows for z).
void fill_set(const edt_batch_map_t* maps, int n, int tw, bool z_pass, EdtMapSet& s,
              const int* gates)
{
    s.n = n;
    s.total = 0;
    s.ny_max = s.nz_max = 0;
    s.wide = false;
    for (int i = 0; i < n; ++i) {
        const edt_grid_t& g = maps[i].grid;
        EdtMap& d = s.m[i];
        d.occ = maps[i].occ;
        d.d2 = maps[i].d2;
        d.site = maps[i].site;
        d.nx = g.nx;
        d.ny = g.ny;
        d.nz = g.nz;
        d.ntx = (g.nx + tw - 1) / tw;
        d.begin = s.total;
        d.gate = gates ? gates + i : nullptr;
        s.total += (z_pass ? g.ny : g.nz) * d.ntx;
        s.ny_max = std::max(s.ny_max, g.ny);
        s.nz_max = std::max(s.nz_max, g.nz);
        s.wide = s.wide || needs_wide(&g);
    }
}

}  // namespace

// Every cross product of the dominance test stays below 2^31 when each axis
// has at most 512 voxels; larger grids use 64-bit products.
bool needs_wide(const edt_grid_t* g) { return g->nx > 512 || g->ny > 512 || g->nz > 512; }

bool tile_ok(int pass, int tw, const edt_grid_t* g, int nt)
{
    constexpr size_t LDS_MAX = 160 * 1024 - 8192;
    if (pass == 1) {
        if (tw != 16 && tw != 32 && tw != 64) return false;
        if (nt != 64 && nt != 128 && nt != 256 && !(nt == 512 && tw >= 32)) return false;
        if (tw > nt) return false;
        return xy_lds(tw, g->ny, nt) <= LDS_MAX;
    }
    if (tw != 8 && tw != 16 && tw != 32 && tw != 64) return false;
    if (nt != 64 && nt != 128 && nt != 256 && !(nt == 512 && tw == 64)) return false;
    if (tw > nt) return false;
    return z_lds(tw, g->nz, nt) <= LDS_MAX;
}

EdtTuning default_tuning(const edt_grid_t* g)
{
    // measured on MI355X: 32-wide xy tiles up to 256 rows; up to 512 rows the
    // same tiles with 512 threads (32 rows per band, and each slice staged by
    // half as many work-groups as with 16-wide tiles); 16-wide beyond.  z
    // tiles keep about 32 positions per band
    EdtTuning t;
    t.xy_tw = g->ny <= 512 ? 32 : 16;
    t.xy_nt = g->ny > 256 && g->ny <= 512 ? 512 : 256;
    // with more than 256 slices as well there are tiles enough to balance:
    // 16-wide tiles in 256-thread work-groups (512^3 blobs: 919 against
    // 1006 us for 32 / 512)
    if (g->ny > 256 && g->nz > 256) {
        t.xy_tw = 16;
        t.xy_nt = 256;
    }
    t.z_tw = g->nz <= 128 ? 64 : (g->nz <= 256 ? 32 : 16);
    t.z_nt = 256;
    // the search tiles (64 / 512 for xy, 64 / 256 for z) where they apply
    if (!needs_wide(g)) {
        t.xy_tw = 64;
        t.xy_nt = 512;
        t.z_tw = 64;
        t.z_nt = 256;
    }
    if (!tile_ok(1, t.xy_tw, g, t.xy_nt)) {
        t.xy_tw = 16;
        t.xy_nt = 256;
    }
    if (!tile_ok(2, t.z_tw, g, t.z_nt)) t.z_tw = 8;
    return t;
}

int make_map_sets(const edt_batch_map_t* maps, int n, const EdtTuning& t, EdtMapSet& xy,
                  EdtMapSet& z, const int* gates)
{
    if (!maps || n < 1 || n > EDT_BATCH_MAX) {
        set_error("need 1..%d maps, got %d", EDT_BATCH_MAX, n);
        return EDT_ERR_ARG;
    }
    edt_grid_t big{};
    big.voxel = 1.0f;
    for (int i = 0; i < n; ++i) {
        const edt_grid_t* g = &maps[i].grid;
        int rc = check_grid(g);
        if (rc) return rc;
        if (!maps[i].occ || !maps[i].d2 || !maps[i].site) {
            set_error("map %d: NULL occ, d2 or site", i);
            return EDT_ERR_ARG;
        }
        big.nx = std::max(big.nx, g->nx);
        big.ny = std::max(big.ny, g->ny);
        big.nz = std::max(big.nz, g->nz);
    }
    if (!tile_ok(1, t.xy_tw, &big, t.xy_nt) || !tile_ok(2, t.z_tw, &big, t.z_nt)) {
        set_error("tiles (%d / %d, %d / %d) not valid for maps up to %d x %d x %d", t.xy_tw, t.xy_nt,
                  t.z_tw, t.z_nt, big.nx, big.ny, big.nz);
        return EDT_ERR_UNSUPPORTED;
    }
    fill_set(maps, n, t.xy_tw, false, xy, gates);
    fill_set(maps, n, t.z_tw, true, z, gates);
    return EDT_OK;
}

int launch_edt_xy_set(const EdtMapSet& s, int tw, int nt, hipStream_t st)
{
    if (nt == 512) {
        switch (tw) {
            case 64: return launch_xy_tw<64, 512>(s, st);
            case 32: return launch_xy_tw<32, 512>(s, st);
        }
    } else if (nt == 256) {
        switch (tw) {
            case 64: return launch_xy_tw<64, 256>(s, st);
            case 32: return launch_xy_tw<32, 256>(s, st);
            case 16: return launch_xy_tw<16, 256>(s, st);
        }
    } else if (nt == 128) {
        switch (tw) {
            case 64: return launch_xy_tw<64, 128>(s, st);
            case 32: return launch_xy_tw<32, 128>(s, st);
            case 16: return launch_xy_tw<16, 128>(s, st);
        }
    } else if (nt == 64) {
        switch (tw) {
            case 64: return launch_xy_tw<64, 64>(s, st);
            case 32: return launch_xy_tw<32, 64>(s, st);
            case 16: return launch_xy_tw<16, 64>(s, st);
        }
    }
    set_error("bad xy tile %d / group %d", tw, nt);
    return EDT_ERR_ARG;
}

int launch_edt_z_set(const EdtMapSet& s, int tw, int nt, hipStream_t st)
{
    if (nt == 512 && tw == 64) return launch_z_tw<64, 512>(s, st);
    if (nt == 256) {
        switch (tw) {
            case 64: return launch_z_tw<64, 256>(s, st);
            case 32: return launch_z_tw<32, 256>(s, st);
            case 16: return launch_z_tw<16, 256>(s, st);
            case 8: return launch_z_tw<8, 256>(s, st);
        }
    } else if (nt == 128) {
        switch (tw) {
            case 64: return launch_z_tw<64, 128>(s, st);
            case 32: return launch_z_tw<32, 128>(s, st);
            case 16: return launch_z_tw<16, 128>(s, st);
            case 8: return launch_z_tw<8, 128>(s, st);
        }
    } else if (nt == 64) {
        switch (tw) {
            case 64: return launch_z_tw<64, 64>(s, st);
            case 32: return launch_z_tw<32, 64>(s, st);
            case 16: return launch_z_tw<16, 64>(s, st);
            case 8: return launch_z_tw<8, 64>(s, st);
        }
    }
    set_error("bad z tile %d / group %d", tw, nt);
    return EDT_ERR_ARG;
}

namespace {
edt_batch_map_t one_map(const edt_grid_t* g, const uint8_t* occ, int32_t* d2, int32_t* site)
{
    edt_batch_map_t m{};
    m.grid = *g;
    m.occ = occ;
    m.d2 = d2;
    m.site = site;
    return m;
}
}  // namespace

int launch_edt_xy(const edt_grid_t* g, const uint8_t* occ, int32_t* d2, uint32_t* xy, int tw, int nt,
                  hipStream_t st, const int* gate)
{
    const edt_batch_map_t m = one_map(g, occ, d2, reinterpret_cast<int32_t*>(xy));
    EdtMapSet s;
    fill_set(&m, 1, tw, false, s, gate);
    return launch_edt_xy_set(s, tw, nt, st);
}

int launch_edt_z(const edt_grid_t* g, int32_t* d2, int32_t* site, int tw, int nt, hipStream_t st,
                 const int* gate)
{
    const edt_batch_map_t m = one_map(g, nullptr, d2, site);
    EdtMapSet s;
    fill_set(&m, 1, tw, true, s, gate);
    return launch_edt_z_set(s, tw, nt, st);
}

}  // namespace edtmi
