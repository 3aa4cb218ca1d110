// Refinement flagging of one level (Methodology, "Refinement Flagging and
// Propagation", Eq. 3), block-parallel (the paper's secondary access mode):
//   1-2. 26-neighbour indices through the forest child maps, and in the
//      same pass the class bits: solid, solid-boundary (solid with a fully
//      fluid neighbour) and eligibility (every in-domain neighbour exists:
//      refining keeps the 2:1 balance);
//   3. marks M1 = (solid-boundary and eligible) or next to a solid-boundary
//      block; solid-adjacent class for the fluid ones;
//   4. n_prop synchronous passes (double-buffered, as the paper avoids the
//      read/write race): fluid blocks, and solid blocks in the first pass,
//      join when a neighbour is marked;
//   5. refine = marked and eligible (written by the last pass of step 4, with
//      the refined blocks of each tile counted); children emitted in parent
//      order from those counts, octant o = ox + 2 oy + 4 oz.
#include "geo_internal.h"

namespace {

enum { F_S = 1, F_SB = 2, F_EL = 4 };

__device__ __forceinline__ void nbr_offset(int k, int& dx, int& dy, int& dz) {
    const int kk = k < 13 ? k : k + 1;  // skip the centre of the 3x3x3 cube
    dx = kk % 3 - 1;
    dy = (kk / 3) % 3 - 1;
    dz = kk / 9 - 1;
}

// 26-neighbour indices (forest_lookup values: index, -1 missing, -2 outside
// the domain).  On levels L >= 1 the 26 neighbours have at most 8 distinct
// parents, the 2x2x2 parents from (b-1) >> 1 to (b+1) >> 1 on each axis: the
// first-child indices of those 8 are found by 8 descents of the forest run
// side by side (their dependent loads overlap), and each neighbour is its
// parent's first child plus its octant, with no further load.  The parent of a
// neighbour is a register, chosen by value by the block's parity (an element of
// an array chosen that way would be indexed in scratch); only a solid block reads
// its neighbours' words, all at once.  Latency bound, a level of the
// 1.05M-triangle star on 192 x 200 x 176 cells: 20.4 us with 26 dependent words,
// 14.2 with the parents in 112 bytes of scratch, 12.6 now.
__global__ void k_ref_nbr(DevLevel d, const uint64_t* solid, int32_t* nbr, uint8_t* cls) {
    const int64_t nb = d.nblocks;
    const int L = d.level;
    const int nb0[3] = {d.n0[0] >> 2, d.n0[1] >> 2, d.n0[2] >> 2};
    for (int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < nb; b += (int64_t)gridDim.x * blockDim.x) {
        const int bc[3] = {d.bcoord[3 * b], d.bcoord[3 * b + 1], d.bcoord[3 * b + 2]};
        // class bits from the neighbours' solid words: solid-boundary (solid
        // with a fully fluid neighbour) and eligible (every in-domain
        // neighbour exists)
        int r[26];
        if (L == 0) {  // the dense root grid: no loads
#pragma unroll
            for (int k = 0; k < 26; k++) {
                int dx, dy, dz;
                nbr_offset(k, dx, dy, dz);
                const int n[3] = {bc[0] + dx, bc[1] + dy, bc[2] + dz};
                bool out = false;
#pragma unroll
                for (int a = 0; a < 3; a++)
                    if (n[a] < 0 || n[a] >= nb0[a]) out = true;
                r[k] = out ? -2 : n[0] + nb0[0] * (n[1] + nb0[1] * n[2]);
            }
        } else {
            int p0[3];  // lowest parent coordinate per axis (level L-1)
            for (int a = 0; a < 3; a++) p0[a] = (bc[a] - 1) >> 1;
            int idx[8];
            bool inside[8];
#pragma unroll
            for (int s = 0; s < 8; s++) {
                const int p[3] = {p0[0] + (s & 1), p0[1] + ((s >> 1) & 1), p0[2] + (s >> 2)};
                inside[s] = true;
#pragma unroll
                for (int a = 0; a < 3; a++)
                    if (p[a] < 0 || p[a] >= (nb0[a] << (L - 1))) inside[s] = false;
                idx[s] = inside[s] ? (p[0] >> (L - 1)) + nb0[0] * ((p[1] >> (L - 1)) + nb0[1] * (p[2] >> (L - 1)))
                                   : -1;
            }
            // descend to level L-1, then the parent's first child on level L
            for (int l = 0; l < L; l++) {
                int c[8];
#pragma unroll
                for (int s = 0; s < 8; s++) c[s] = idx[s] >= 0 ? d.child[l][idx[s]] : -1;
                const int sh = L - 2 - l;
#pragma unroll
                for (int s = 0; s < 8; s++) {
                    if (l == L - 1 || c[s] < 0) {
                        idx[s] = c[s];
                    } else {
                        const int p[3] = {p0[0] + (s & 1), p0[1] + ((s >> 1) & 1), p0[2] + (s >> 2)};
                        idx[s] = c[s] + (((p[0] >> sh) & 1) | (((p[1] >> sh) & 1) << 1) | (((p[2] >> sh) & 1) << 2));
                    }
                }
            }
            // the parents seen from the block: per axis the lower one at -1, the
            // upper one at +1, and at 0 the block's own
            int fc[27];
#pragma unroll
            for (int s = 0; s < 8; s++) fc[2 * (s & 1) + 6 * ((s >> 1) & 1) + 18 * (s >> 2)] = idx[s];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const int z = 6 * (q & 1) + 18 * (q >> 1);
                fc[z + 1] = pick2(fc[z], fc[z + 2], bc[0] & 1);
            }
#pragma unroll
            for (int q = 0; q < 6; q++) {
                const int z = q % 3 + 18 * (q / 3);
                fc[z + 3] = pick2(fc[z], fc[z + 6], bc[1] & 1);
            }
#pragma unroll
            for (int q = 0; q < 9; q++) fc[q + 9] = pick2(fc[q], fc[q + 18], bc[2] & 1);
#pragma unroll
            for (int k = 0; k < 26; k++) {
                int dv[3];
                nbr_offset(k, dv[0], dv[1], dv[2]);
                int n[3];
                bool out = false;
#pragma unroll
                for (int a = 0; a < 3; a++) {
                    n[a] = bc[a] + dv[a];
                    if (n[a] < 0 || n[a] >= (nb0[a] << L)) out = true;
                }
                const int f = fc[k < 13 ? k : k + 1];
                r[k] = out ? -2 : f < 0 ? -1 : f + ((n[0] & 1) | ((n[1] & 1) << 1) | ((n[2] & 1) << 2));
            }
        }
        bool elig = true;
#pragma unroll
        for (int k = 0; k < 26; k++) {
            nbr[(int64_t)k * nb + b] = r[k];
            if (r[k] == -1) elig = false;
        }
        uint8_t g = elig ? F_EL : 0;
        if (solid[b] != 0ull) {  // a fluid block's class needs no neighbour
            bool fluid_nbr = false;
#pragma unroll
            for (int k = 0; k < 26; k++) {
                const uint64_t w = solid[r[k] >= 0 ? r[k] : b];  // its own word is not 0
                if (w == 0ull) fluid_nbr = true;
            }
            g |= fluid_nbr ? F_S | F_SB : F_S;
        }
        cls[b] = g;
    }
}

// Whether a neighbour of block b has a bit of a byte array.  Latency bound: all
// 26 indices and then all 26 bytes are loaded at once.  One by one, each
// waiting for the last, the marks of a level took 14.7 us and a propagation
// pass 13.1 us on average (1.05M-triangle star, 192 x 200 x 176 cells), now 7.1
// and 7.0; 10.5 and 7.4 us against 3.1 and 3.6 with 1,792 triangles.
__device__ __forceinline__ bool near_bit(int64_t nb, const int32_t* nbr, int64_t b, const uint8_t* v, unsigned bit) {
    int n[26];
#pragma unroll
    for (int k = 0; k < 26; k++) n[k] = nbr[(int64_t)k * nb + b];
    unsigned any = 0;
#pragma unroll
    for (int k = 0; k < 26; k++) {
        const unsigned x = v[n[k] >= 0 ? n[k] : b];
        any |= n[k] >= 0 ? x : 0u;
    }
    return (any & bit) != 0;
}

__global__ void k_ref_m1(int64_t nb, const int32_t* nbr, const uint8_t* flags, uint8_t* M, uint8_t* bclass) {
    for (int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < nb; b += (int64_t)gridDim.x * blockDim.x) {
        const uint8_t f = flags[b];
        const bool adj = near_bit(nb, nbr, b, flags, F_SB);
        const bool m0 = (f & F_SB) && (f & F_EL);
        const bool m = m0 || adj;
        M[b] = m ? 1 : 0;
        bclass[b] = (f & F_SB) ? 2 : ((f & F_S) ? 1 : ((m && !m0) ? 3 : 0));
    }
}

// One propagation pass; the last one (refine != null) also writes refine =
// marked and eligible, and its tile's refined blocks for the children's places.
// Bound by the latency of the neighbours' marks.
__global__ void __launch_bounds__(256) k_ref_prop(int64_t nb, int passes, const int32_t* nbr, const uint8_t* flags,
                                                  const uint8_t* Min, uint8_t* Mout, int first, uint8_t* refine,
                                                  int32_t* counts) {
    __shared__ int tmp[4];
    int n_ref = 0;
    for (int p = 0; p < passes; p++) {
        const int64_t b = ((int64_t)blockIdx.x * passes + p) * 256 + threadIdx.x;
        if (b >= nb) break;
        uint8_t m = Min[b];
        const uint8_t f = flags[b];
        if (!m && (!(f & F_S) || first)) m = near_bit(nb, nbr, b, Min, 1);
        Mout[b] = m;
        if (refine) {
            const int r = (m && (f & F_EL)) ? 1 : 0;
            refine[b] = (uint8_t)r;
            n_ref += r;
        }
    }
    if (!refine) return;
    n_ref = wg_sum256(n_ref, tmp);
    if (threadIdx.x == 0) counts[blockIdx.x] = n_ref;
}

// without propagation passes: refine and the tiles' counts from the marks
__global__ void __launch_bounds__(256) k_ref_final(int64_t nb, int passes, const uint8_t* flags, const uint8_t* M,
                                                   uint8_t* refine, int32_t* counts) {
    __shared__ int tmp[4];
    int n_ref = 0;
    for (int p = 0; p < passes; p++) {
        const int64_t b = ((int64_t)blockIdx.x * passes + p) * 256 + threadIdx.x;
        if (b >= nb) break;
        const int r = (M[b] && (flags[b] & F_EL)) ? 1 : 0;
        refine[b] = (uint8_t)r;
        n_ref += r;
    }
    n_ref = wg_sum256(n_ref, tmp);
    if (threadIdx.x == 0) counts[blockIdx.x] = n_ref;
}

// The children, tile by tile: 6.3 us a level where a star of 1.05M triangles on
// 192 x 200 x 176 cells is refined, launch and latency bound (with a scan of its
// own, two launches and 9.6 us more, and a lane per block writing its 24 words
// apart, 7.0 us).
__global__ void __launch_bounds__(256) k_ref_emit(int64_t nb, const int32_t* bcoord, const uint8_t* refine,
                                                  const int32_t* counts, int passes, int32_t* child_map,
                                                  int32_t* child_bcoord, int64_t* d_nchild) {
    emit_children<3>(nb, bcoord, refine, counts, passes, child_map, child_bcoord, d_nchild);
}

inline unsigned grid_for(int64_t n) {
    int64_t g = (n + 255) / 256;
    if (g > 65536) g = 65536;
    if (g < 1) g = 1;
    return (unsigned)g;
}

inline size_t al(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

size_t geo_refine_ws_bytes(int64_t nb) {
    return al(sizeof(int32_t) * 26 * (size_t)nb) + 3 * al((size_t)nb) + al(sizeof(int32_t) * child_tiles(nb));
}

int launch_refine(const DevLevel& d, const uint64_t* solid, int n_prop, uint8_t* bclass, uint8_t* refine,
                  int32_t* child_map, int32_t* child_bcoord, int64_t* d_nchild, void* ws, size_t ws_bytes,
                  hipStream_t s) {
    const int64_t nb = d.nblocks;
    if (ws_bytes < geo_refine_ws_bytes(nb)) return GEO_ERR_WORKSPACE;
    char* p = static_cast<char*>(ws);
    int32_t* nbr = reinterpret_cast<int32_t*>(p);
    p += al(sizeof(int32_t) * 26 * (size_t)nb);
    uint8_t* cls = reinterpret_cast<uint8_t*>(p);
    p += al((size_t)nb);
    uint8_t* M = reinterpret_cast<uint8_t*>(p);
    p += al((size_t)nb);
    uint8_t* Mn = reinterpret_cast<uint8_t*>(p);
    p += al((size_t)nb);
    int32_t* counts = reinterpret_cast<int32_t*>(p);

    if (nb == 0) {
        int rc = geo_fill_u64(reinterpret_cast<uint64_t*>(d_nchild), 0, 1, s);
        return rc;
    }
    const unsigned g = grid_for(nb), tiles = child_tiles(nb);
    const int passes = child_passes(nb);
    k_ref_nbr<<<g, 256, 0, s>>>(d, solid, nbr, cls);
    k_ref_m1<<<g, 256, 0, s>>>(nb, nbr, cls, M, bclass);
    for (int k = 1; k <= n_prop; k++) {
        const bool last = k == n_prop;
        k_ref_prop<<<tiles, 256, 0, s>>>(nb, passes, nbr, cls, M, Mn, k == 1 ? 1 : 0, last ? refine : nullptr,
                                         last ? counts : nullptr);
        uint8_t* t = M;
        M = Mn;
        Mn = t;
    }
    if (n_prop == 0) k_ref_final<<<tiles, 256, 0, s>>>(nb, passes, cls, M, refine, counts);
    k_ref_emit<<<tiles, 256, 0, s>>>(nb, d.bcoord, refine, counts, passes, child_map, child_bcoord, d_nchild);
    GEO_LAUNCH_CHECK();
    return GEO_OK;
}
