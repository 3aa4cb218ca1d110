// Solid voxelization of one level (integer gather over the ROWS bins).
//
// The paper flags cells near the surface by local ray casts and fills the
// interior by scan-line propagation inside and across blocks (Algorithms 3-5).
// Here the exact surface events of every row line are already in the ROWS
// bins, so the solid flag of a cell is a local function of its own line:
// parity of the crossings ahead of it on its +x ray, or'ed with the
// on-surface intervals.  No propagation between blocks is needed, so holes in
// the block set of a level cannot leave cells unfilled.
//
// Layout: the 8 children of a block are 8 consecutive blocks, 2 x 2 x 2 in
// space, so a wave takes all 8: one lane per row line of their 8 x 8 lines,
// which produces the 8 flags of its line, four for either block along x.  16
// lanes (a DPP row) hold the 4 x 4 lines of one pair of blocks, from which the
// two 64-bit block masks are assembled (bit t = I + 4 J + 16 K).  Bound by the
// L1's rate of accesses and the latency of offsets and entries, which serve two
// blocks this way and come by loads of 8 and 16 bytes.  On level 0, and where
// 8 blocks are not such a family, 16 lanes take a block.  All
// levels of a step before (4 blocks per wave, loads of 4 bytes), with families,
// and with wider loads too: 514, 358 and 283 us on the 7.2M-triangle star, 405,
// 266 and 188 us on 64 spheres, 150, 122 and 96 us on a 1M-triangle star over
// four levels.
#include "geo_internal.h"

namespace {

// fold entries v[0..3] (those below n) of a line into the parity and surface
// flags of cells x0..x0+W-1
template <int W>
__device__ __forceinline__ void fold_line(const int32_t* v4, int n, int x0, unsigned& par, unsigned& surf) {
#pragma unroll
    for (int i = 0; i < 4; i++) {
        if (i >= n) break;
        const int32_t v = v4[i];
        if (v >= 0) {
            // cells x < v see this crossing ahead: flip those of x0..x0+W-1
            int k = v - x0;
            k = k < 0 ? 0 : (k > W ? W : k);
            par ^= (1u << k) - 1u;
        } else {
            int a = (v & 0x7fff) - x0, b = ((v >> 15) & 0x7fff) - x0;
            a = a < 0 ? 0 : a;
            b = b > W - 1 ? W - 1 : b;
            if (a <= b) surf |= ((1u << (b + 1)) - 1u) & ~((1u << a) - 1u);
        }
    }
}

// flags of cells x0[u]..x0[u]+W-1 of N lines (on[u]), their offsets and then
// their first four entries loaded together
template <int W, int N>
__device__ __forceinline__ void line_flags(const int32_t* off, const int32_t* val, int64_t cap, const bool on[N],
                                           const int64_t line[N], const int x0[N], unsigned f[N]) {
    const int last = entry_limit(cap);
    int e0[N], e1[N];
#pragma unroll
    for (int u = 0; u < N; u++) {
        e0[u] = e1[u] = 0;
        if (on[u]) line_range(off, line[u], last, e0[u], e1[u]);
    }
    int32_t v[N][4];
#pragma unroll
    for (int u = 0; u < N; u++) line_entries(val, e0[u], e1[u], last, v[u]);
#pragma unroll
    for (int u = 0; u < N; u++) {
        unsigned par = 0, surf = 0;
        fold_line<W>(v[u], e1[u] - e0[u], x0[u], par, surf);
        for (int e = e0[u] + 4; e < e1[u] && e > 0; e += 4) {  // lines with more than four entries
            int32_t w[4];
            line_entries(val, e, e1[u], last, w);
            fold_line<W>(w, e1[u] - e, x0[u], par, surf);
        }
        f[u] = (par | surf) & ((1u << W) - 1u);
    }
}

// The 64-bit masks of the two blocks (m0: low nibbles) of a DPP row from the 8
// flags of each lane's line, J = lane & 3, K = lane >> 2 & 3: nibbles joined
// over the four J of a quad, then the four planes K from their quads.  Whole in
// the row's lanes 12..15.
__device__ __forceinline__ void row_masks(unsigned f, int lane, unsigned long long& m0, unsigned long long& m1) {
    const int sh = 4 * (lane & 3);
    unsigned w = ((f & 15u) << sh) | ((f >> 4) << (16 + sh));  // plane K of both blocks, 16 bits each
    w |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)w, 0xb1, 0xf, 0xf, false);  // quad_perm 1,0,3,2
    w |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)w, 0x4e, 0xf, 0xf, false);  // quad_perm 2,3,0,1
    const unsigned k2 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)w, 0x114, 0xf, 0xf, false);  // row_shr:4
    const unsigned k1 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)w, 0x118, 0xf, 0xf, false);  // row_shr:8
    const unsigned k0 = (unsigned)__builtin_amdgcn_update_dpp(0, (int)w, 0x11c, 0xf, 0xf, false);  // row_shr:12
    m0 = ((unsigned long long)((k2 & 0xffffu) | (w << 16)) << 32) | ((k0 & 0xffffu) | (k1 << 16));
    m1 = ((unsigned long long)((k2 >> 16) | (w & 0xffff0000u)) << 32) | ((k0 >> 16) | (k1 & 0xffff0000u));
}

// blocks wb .. wb + 3, 16 lanes each
__device__ __forceinline__ void voxelize4(const DevLevel& d, const int32_t* off, const int32_t* val, int64_t cap,
                                          int64_t wb, uint64_t* solid) {
    const int ny = d.n0[1] << d.level;
    const int lane = threadIdx.x & 63;
    const int64_t b = wb + (lane >> 4);
    const int l = lane & 15;
    const bool on[1] = {b < d.nblocks};
    int c[3] = {0, 0, 0};
    if (on[0])
        for (int a = 0; a < 3; a++) c[a] = d.bcoord[3 * b + a];
    const int64_t line[1] = {(int64_t)(4 * c[1] + (l & 3)) + (int64_t)ny * (4 * c[2] + (l >> 2))};
    const int x0[1] = {4 * c[0]};
    unsigned nib[1];
    line_flags<4, 1>(off, val, cap, on, line, x0, nib);
    unsigned long long m, none;
    row_masks(nib[0], lane, m, none);
    if (l == 15 && b < d.nblocks) solid[b] = m;
}

// Level 0, whose blocks are no families: 4 blocks to a wave, four times the waves
// of the families' kernel (512^3 cells: 78 us, 89 with that; 256^3: 10.5 and 13.7).
__global__ void __launch_bounds__(256) k_voxelize0(DevLevel d, const int32_t* off, const int32_t* val, int64_t cap,
                                                   uint64_t* solid) {
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t wb = wave * 4; wb < d.nblocks; wb += nwaves * 4) voxelize4(d, off, val, cap, wb, solid);
}

constexpr int FAM = 2;  // families of a wave, their loads in flight together
__global__ void __launch_bounds__(256) k_voxelize(DevLevel d, const int32_t* off, const int32_t* val,
                                                  int64_t cap, uint64_t* solid) {
    const int ny = d.n0[1] << d.level;
    const int lane = threadIdx.x & 63;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    for (int64_t wb = wave * 8 * FAM; wb < d.nblocks; wb += nwaves * 8 * FAM) {
        // FAM times 8 blocks' coordinates, lane o's block wb + o; a family: twice
        // the parent's plus the octant bits of o = ox + 2 oy + 4 oz
        int p[FAM][3];
        bool fam[FAM];
#pragma unroll
        for (int u = 0; u < FAM; u++) {
            const int64_t bo = wb + 8 * u + (lane & 7);
            const bool in = bo < d.nblocks;
            int c[3];
#pragma unroll
            for (int a = 0; a < 3; a++) c[a] = in ? d.bcoord[3 * bo + a] : 0;
            bool ok = in;
#pragma unroll
            for (int a = 0; a < 3; a++) {
                p[u][a] = __builtin_amdgcn_readfirstlane(c[a]);
                ok = ok && !(p[u][a] & 1) && c[a] == p[u][a] + (lane >> a & 1);
            }
            fam[u] = __all(ok);  // uniform
        }
        // row r of 16 lanes: the pair of blocks (oy, oz) = (r & 1, r >> 1)
        const int l = lane & 15, r = lane >> 4;
        int64_t line[FAM];
        int x0[FAM];
        unsigned f[FAM];
#pragma unroll
        for (int u = 0; u < FAM; u++) {
            line[u] = (int64_t)(4 * (p[u][1] + (r & 1)) + (l & 3)) + (int64_t)ny * (4 * (p[u][2] + (r >> 1)) + (l >> 2));
            x0[u] = 4 * p[u][0];
        }
        line_flags<8, FAM>(off, val, cap, fam, line, x0, f);
#pragma unroll
        for (int u = 0; u < FAM; u++) {
            const int64_t b = wb + 8 * u;
            if (fam[u]) {  // blocks 2 r and 2 r + 1 of the family
                unsigned long long m0, m1;
                row_masks(f[u], lane, m0, m1);
                if (l == 15) {
                    solid[b + 2 * r] = m0;
                    solid[b + 2 * r + 1] = m1;
                }
            } else {
                voxelize4(d, off, val, cap, b, solid);
                voxelize4(d, off, val, cap, b + 4, solid);
            }
        }
    }
}

__global__ void k_level0(int nbx, int nby, int nbz, int32_t* bcoord) {
    const int64_t n = (int64_t)nbx * nby * nbz;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        bcoord[3 * i] = (int)(i % nbx);
        bcoord[3 * i + 1] = (int)((i / nbx) % nby);
        bcoord[3 * i + 2] = (int)(i / ((int64_t)nbx * nby));
    }
}

}  // namespace

int launch_voxelize(const DevLevel& d, const int32_t* off, const int32_t* val, int64_t cap, uint64_t* solid,
                    hipStream_t s) {
    if (d.nblocks == 0) return GEO_OK;
    const int per_wave = d.level > 0 ? 8 * FAM : 4;
    int64_t waves = ((int64_t)d.nblocks + per_wave - 1) / per_wave;
    int64_t g = (waves * 64 + 255) / 256;
    if (g > 65536) g = 65536;
    kt_record(GEO_KT_VOXELIZE, s, false);
    auto kernel = d.level > 0 ? k_voxelize : k_voxelize0;
    kernel<<<(unsigned)g, 256, 0, s>>>(d, off, val, cap, solid);
    kt_record(GEO_KT_VOXELIZE, s, true);
    GEO_LAUNCH_CHECK();
    return GEO_OK;
}

int launch_level0(const int32_t n0[3], int32_t* bcoord, hipStream_t s) {
    const int nbx = n0[0] / 4, nby = n0[1] / 4, nbz = n0[2] / 4;
    const int64_t n = (int64_t)nbx * nby * nbz;
    int64_t g = (n + 255) / 256;
    if (g > 65536) g = 65536;
    if (g < 1) g = 1;
    k_level0<<<(unsigned)g, 256, 0, s>>>(nbx, nby, nbz, bcoord);
    GEO_LAUNCH_CHECK();
    return GEO_OK;
}
