// Device-wide exclusive scans of int32 counts and small fill kernels.
//
// Tiles of 4,096 values.  Two launches: the sums of all tiles, then the tiles
// themselves, each adding up the sums of the tiles before it (up to SCAN_SUMS
// words from L2) instead of waiting for a scan of the sums by one workgroup.
// Those reads grow with the square of the tiles, so arrays of more than
// SCAN_SUMS tiles take a launch in between that scans their sums.
// Several arrays go through the same launches, and where no
// array has more than SCAN_DIRECT tiles one launch does: a tile then reads the
// values before it again (at most 48 loads per thread, less than a launch).
// Bound by launches below about 10^6 values and by HBM above (4 bytes read
// twice, 4 written).  The scans of a step with
// three launches of 2,048-value tiles per array, and now: 228 and 135 us on the
// 7.2M-triangle star (22.3M row lines, four refinements, 5.8M blocks twice),
// 99 and 43 us with 1,792 triangles, 39 and 18 us in one level of 64^3 cells.
#include "geo_internal.h"

namespace {

constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 16;
constexpr int SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;
constexpr int SCAN_DIRECT = 4;
// ROWS bins of 8,192^2 lines (16,384 tiles) without and with that launch: 236 and
// 207 us; 16,384^2: 1.91 and 0.87 ms (1.13 with three launches of 2,048-value
// tiles); 5,000^2 (6,104 tiles): 86 and 89 us
constexpr int64_t SCAN_SUMS = 8192;

// sum of v over the workgroup (every thread calls it)
__device__ __forceinline__ int64_t block_sum(int64_t v) {
    __shared__ int64_t wsum[SCAN_THREADS / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = v;
    __syncthreads();
    int64_t t = 0;
#pragma unroll
    for (int i = 0; i < SCAN_THREADS / 64; i++) t += wsum[i];
    __syncthreads();
    return t;
}

// exclusive scan across the block (every thread calls it; the wave scan is
// the shared data-parallel one); returns the block total in *total
__device__ __forceinline__ int block_excl_scan(int v, int* total) {
    __shared__ int wsum[SCAN_THREADS / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int incl = wave_incl_scan(v);
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < SCAN_THREADS / 64; i++) {
        if (i < w) base += wsum[i];
        tot += wsum[i];
    }
    __syncthreads();
    *total = tot;
    return base + incl - v;
}

// job of a tile (uniform)
__device__ __forceinline__ int tile_job(const ScanJobs& j, int tile) {
    int q = 0;
    for (int i = 1; i < j.n; i++) q += tile >= j.tile0[i] ? 1 : 0;
    return q;
}

// This thread's values of the tile in[0..n-1] (n may exceed the tile; zero
// past n): value 4 i + c is that of position 1024 i + 4 t + c.  All loads are
// in flight together: 16 bytes each where the tile is whole and aligned, else
// single words with the index clamped instead of a branch per load.
__device__ __forceinline__ void tile_load(const int32_t* in, int64_t n, int v[SCAN_ITEMS]) {
    const int t = threadIdx.x;
    if (n >= SCAN_TILE && (reinterpret_cast<uintptr_t>(in) & 15) == 0) {  // uniform
#pragma unroll
        for (int i = 0; i < SCAN_ITEMS / 4; i++) {
            const int4 x = reinterpret_cast<const int4*>(in)[i * SCAN_THREADS + t];
            v[4 * i] = x.x;
            v[4 * i + 1] = x.y;
            v[4 * i + 2] = x.z;
            v[4 * i + 3] = x.w;
        }
        return;
    }
    if (n <= 0) {  // uniform
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS; k++) v[k] = 0;
        return;
    }
    const int last = n < SCAN_TILE ? (int)n - 1 : SCAN_TILE - 1;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; k++) {
        const int j = 1024 * (k / 4) + 4 * t + (k & 3);
        v[k] = in[j < last ? j : last];
    }
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; k++)
        if (1024 * (k / 4) + 4 * t + (k & 3) > last) v[k] = 0;
}

__device__ __forceinline__ int64_t tile_share(const int32_t* in, int64_t n) {
    int v[SCAN_ITEMS];
    tile_load(in, n, v);
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; k++) s += v[k];
    return s;
}

__global__ void __launch_bounds__(SCAN_THREADS) k_tile_sums(ScanJobs jobs, int64_t* partials) {
    const int q = tile_job(jobs, blockIdx.x);
    const int64_t base = (int64_t)((int)blockIdx.x - jobs.tile0[q]) * SCAN_TILE;
    const int64_t t = block_sum(tile_share(jobs.in[q] + base, jobs.len[q] - base));
    if (threadIdx.x == 0) partials[blockIdx.x] = t;
}

// The tile sums of each array (one workgroup) turned into the sums before each
// tile.  A thread takes SUM_ITEMS tiles in a row.
constexpr int SUM_ITEMS = 16;
__global__ void __launch_bounds__(SCAN_THREADS) k_scan_sums(ScanJobs jobs, int64_t* partials) {
    __shared__ int64_t wsum[SCAN_THREADS / 64];
    const int q = blockIdx.x, t = threadIdx.x, w = t >> 6;
    const int64_t n = (jobs.len[q] + SCAN_TILE - 1) / SCAN_TILE;
    int64_t* p = partials + jobs.tile0[q];
    int64_t carry = 0;
    for (int64_t base = 0; base < n; base += SCAN_THREADS * SUM_ITEMS) {  // uniform
        const int64_t i0 = base + (int64_t)t * SUM_ITEMS;
        int64_t v[SUM_ITEMS], s = 0;
#pragma unroll
        for (int k = 0; k < SUM_ITEMS; k++) v[k] = i0 + k < n ? p[i0 + k] : 0;
#pragma unroll
        for (int k = 0; k < SUM_ITEMS; k++) s += v[k];
        int64_t incl = s;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t u = __shfl_up(incl, o, 64);
            if ((t & 63) >= o) incl += u;
        }
        if ((t & 63) == 63) wsum[w] = incl;
        __syncthreads();
        int64_t ex = carry + incl - s;
#pragma unroll
        for (int i = 0; i < SCAN_THREADS / 64; i++) {
            if (i < w) ex += wsum[i];
            carry += wsum[i];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < SUM_ITEMS; k++) {
            if (i0 + k < n) p[i0 + k] = ex;
            ex += v[k];
        }
    }
}

// The tile passes through LDS so that global reads and writes are coalesced
// (lane-consecutive), while each thread scans SCAN_ITEMS consecutive values.
// The LDS rows are padded by one word per SCAN_ITEMS, so a thread's
// consecutive items fall in distinct banks.  partials == nullptr: the values
// of the tiles before are read themselves; scanned: partials holds the sums
// before each tile.
__global__ void __launch_bounds__(SCAN_THREADS) k_scan_tiles(ScanJobs jobs, const int64_t* partials, int scanned) {
    __shared__ int tile[SCAN_TILE + SCAN_TILE / SCAN_ITEMS];
    const int q = tile_job(jobs, blockIdx.x);
    const int first = jobs.tile0[q], ti = (int)blockIdx.x - first;
    const int32_t* in = jobs.in[q];
    int32_t* out = jobs.out[q];
    const int64_t n = jobs.len[q], base = (int64_t)ti * SCAN_TILE;
    const int t = threadIdx.x;
    auto slot = [](int j) { return j + j / SCAN_ITEMS; };
    int v[SCAN_ITEMS];
    tile_load(in + base, n - base, v);
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; k++) tile[slot(1024 * (k / 4) + 4 * t + (k & 3))] = v[k];
    int64_t before = 0;
    if (scanned)
        before = t == 0 ? partials[first + ti] : 0;
    else if (partials)
        for (int i = t; i < ti; i += SCAN_THREADS) before += partials[first + i];
    else
        for (int i = 0; i < ti; i++) before += tile_share(in + (int64_t)i * SCAN_TILE, SCAN_TILE);
    before = block_sum(before);  // (its barrier also covers the LDS tile)
    int s = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; i++) {
        v[i] = tile[slot(t * SCAN_ITEMS + i)];
        s += v[i];
    }
    int tot;
    int ex = block_excl_scan(s, &tot) + (int)before;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; i++) {
        tile[slot(t * SCAN_ITEMS + i)] = ex;
        ex += v[i];
    }
    __syncthreads();
    if (base + SCAN_TILE <= n && (reinterpret_cast<uintptr_t>(out) & 15) == 0) {  // uniform
#pragma unroll
        for (int i = 0; i < SCAN_ITEMS / 4; i++) {
            const int j = slot(1024 * i + 4 * t);  // four positions of one group
            reinterpret_cast<int4*>(out + base)[i * SCAN_THREADS + t] =
                make_int4(tile[j], tile[j + 1], tile[j + 2], tile[j + 3]);
        }
    } else {
#pragma unroll
        for (int i = 0; i < SCAN_ITEMS; i++) {
            const int j = i * SCAN_THREADS + t;
            if (base + j < n) out[base + j] = tile[slot(j)];
        }
    }
    if (base + SCAN_TILE >= n) {  // the array's last tile: totals, exact in 64 bits
        // the tile's own values summed in 64 bits (their int32 sum may wrap)
        int64_t own = 0;
#pragma unroll
        for (int i = 0; i < SCAN_ITEMS; i++) own += v[i];
        own = block_sum(own);
        if (t == 0) {
            out[n] = (int32_t)(before + own);
            if (jobs.total[q]) *jobs.total[q] = before + own;
        }
    }
}

__global__ void k_fill_i32(int32_t* p, int32_t v, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_fill_u64(uint64_t* p, uint64_t v, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

inline unsigned grid_for(int64_t n, int threads) {
    int64_t g = (n + threads - 1) / threads;
    if (g > 65536) g = 65536;
    if (g < 1) g = 1;
    return (unsigned)g;
}

}  // namespace

size_t geo_scan_partials_bytes(int64_t n) {
    const int64_t ntiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    return sizeof(int64_t) * (size_t)(ntiles > 0 ? ntiles : 1);
}

int geo_scan_jobs(ScanJobs& j, int64_t* partials, hipStream_t s) {
    int64_t tiles = 0, most = 0;
    for (int q = 0; q < j.n; q++) {
        const int64_t nt = j.len[q] > 0 ? (j.len[q] + SCAN_TILE - 1) / SCAN_TILE : 1;
        j.tile0[q] = (int)tiles;
        tiles += nt;
        most = nt > most ? nt : most;
    }
    if (tiles == 0) return GEO_OK;
    const bool direct = most <= SCAN_DIRECT, scanned = most > SCAN_SUMS;
    if (!direct) k_tile_sums<<<(unsigned)tiles, SCAN_THREADS, 0, s>>>(j, partials);
    if (scanned) k_scan_sums<<<(unsigned)j.n, SCAN_THREADS, 0, s>>>(j, partials);
    k_scan_tiles<<<(unsigned)tiles, SCAN_THREADS, 0, s>>>(j, direct ? nullptr : partials, scanned ? 1 : 0);
    GEO_LAUNCH_CHECK();
    return GEO_OK;
}

int geo_scan_exclusive(const int32_t* in, int32_t* out, int64_t n, int64_t* partials, hipStream_t s, int64_t* total) {
    ScanJobs j{};
    j.add(in, out, n, total);
    return geo_scan_jobs(j, partials, s);
}

int geo_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s) {
    if (n <= 0) return GEO_OK;
    k_fill_i32<<<grid_for(n, 256), 256, 0, s>>>(p, v, n);
    GEO_LAUNCH_CHECK();
    return GEO_OK;
}

int geo_fill_u64(uint64_t* p, uint64_t v, int64_t n, hipStream_t s) {
    if (n <= 0) return GEO_OK;
    k_fill_u64<<<grid_for(n, 256), 256, 0, s>>>(p, v, n);
    GEO_LAUNCH_CHECK();
    return GEO_OK;
}
