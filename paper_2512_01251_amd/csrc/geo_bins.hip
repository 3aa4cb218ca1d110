// Spatial binning on gfx950 (Methodology, "Spatial Binning").
//
// ROWS bins hold, per x-row line of a level, the exact surface events along
// the line (parity crossings and on-surface intervals); they are built from
// the triangles: for each row line inside a triangle's yz bounding box it is
// decided exactly whether the line meets it, and where along the line.  LINKS
// bins hold, per block, the triangles overlapping the block box widened by half
// a cell on every side, the reach of its links (Algorithm 2 widens by a cell).
//
// Both are counting sorts without a global sort: pass 1 appends (key, value)
// pairs with one atomic per wave and counts per key, an exclusive scan turns
// counts into offsets, and a scatter pass places the pairs.
#include <type_traits>

#include "geo_internal.h"

namespace {

// ------------------------------------------------------------------------
// Append of (key, value) pairs.  Each workgroup is one wave; pairs are staged
// in an LDS buffer and flushed with one global reservation per flush (a
// global counter touched once per wave-iteration would serialise at L2).
// Reservations on one counter complete one every 8.7 ns (64 spheres: 21,000
// of them were 0.18 of the LINKS pass's 0.24 ms), so there are two: even
// workgroups fill the pair array upwards from its start, odd ones downwards
// from its end, and any split of the pairs between them fits.
// The per-key counts are incremented at flush time, and the count a pair
// finds is its rank among its key's pairs, kept beside it: the scatter then
// places it without atomics.
// ------------------------------------------------------------------------
constexpr int APP_BUF = 512;
constexpr int APP_TAB_BITS = 9, APP_TAB = 1 << APP_TAB_BITS;

// Group: pairs whose keys repeat within a flush (link bins: neighbouring
// triangles share blocks) take their ranks with one atomic per key and 256
// pairs (atomics on one address serialise); else one atomic per pair (row bins:
// keys mostly distinct).
template <bool Group>
struct Appender {
    int2* buf;       // LDS [APP_BUF]
    int n;           // pairs staged (identical in every lane)
    const BinWork& w;
    unsigned* tab;   // LDS [APP_TAB] (Group)

    // array position of the i-th pair of a flush, or -1 past the capacity
    __device__ __forceinline__ int64_t place(unsigned long long base, int i) const {
        const unsigned long long k = base + (unsigned long long)i;
        if (k >= (unsigned long long)w.cap) return -1;
        return (blockIdx.x & 1) ? w.cap - 1 - (int64_t)k : (int64_t)k;
    }

    __device__ __forceinline__ void flush() {
        if (n == 0) return;
        __syncthreads();
        unsigned long long base = 0;
        if (threadIdx.x == 0) base = atomicAdd((blockIdx.x & 1) ? &w.ctl->down : &w.ctl->up, (unsigned long long)n);
        base = __shfl(base, 0, 64);
        if constexpr (Group) {
            // 256 pairs at a time, four of a lane.  Pairs with the same key meet in
            // a slot of an LDS table (open addressing, never more than half full),
            // which counts them and holds the number of the first, whose key it is
            // and whose lane then takes the slot's ranks with one atomic.  The
            // whole LINKS call with groups found by ballots within rows of 64
            // pairs, and with the table: 803 and 724 us on the 7.2M-triangle star,
            // 200 and 186 us on 64 spheres, 313 and 124 us on a 40,000-triangle
            // cylinder, 82 and 70 us on the 112k star.
            const int lane = threadIdx.x;
            constexpr unsigned EMPTY = ~0u;
            for (int i0 = 0; i0 < n; i0 += 256) {
#pragma unroll
                for (int k = 0; k < APP_TAB / 64; k++) tab[64 * k + lane] = EMPTY;
                __syncthreads();
                int2 p[4];
                unsigned at[4];  // slot | rank in it << 16
                bool head[4];    // the slot's first
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    const int i = 64 * u + lane;
                    p[u] = i0 + i < n ? buf[i0 + i] : make_int2(-1, 0);
                    at[u] = 0;
                    head[u] = false;
                }
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    if (p[u].x < 0) continue;
                    unsigned s = ((unsigned)p[u].x * 2654435761u) >> (32 - APP_TAB_BITS);
                    while (true) {
                        unsigned e = __hip_atomic_load(&tab[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        if (e == EMPTY) e = atomicCAS(&tab[s], EMPTY, (unsigned)(64 * u + lane) << 16 | 1u);
                        if (e == EMPTY) {
                            at[u] = s;
                            head[u] = true;
                            break;
                        }
                        if (buf[i0 + (e >> 16)].x == p[u].x) {
                            at[u] = s | (atomicAdd(&tab[s], 1u) & 0xffffu) << 16;
                            break;
                        }
                        s = (s + 1) & (APP_TAB - 1);
                    }
                }
                __syncthreads();
                int r[4];
#pragma unroll
                for (int u = 0; u < 4; u++) r[u] = head[u] ? atomicAdd(&w.cnt[p[u].x], (int)(tab[at[u]] & 0xffffu)) : 0;
                __syncthreads();
#pragma unroll
                for (int u = 0; u < 4; u++)
                    if (head[u]) tab[at[u]] = (unsigned)r[u];
                __syncthreads();
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    const int64_t pos = place(base, i0 + 64 * u + lane);
                    if (p[u].x >= 0 && pos >= 0) {
                        w.pairs[pos] = p[u];
                        w.rank[pos] = (int)tab[at[u] & (APP_TAB - 1)] + (int)(at[u] >> 16);
                    }
                }
                __syncthreads();
            }
        } else {
            // four returning atomics in flight per lane before their results are used
            for (int i0 = threadIdx.x; i0 < n; i0 += 256) {
                int2 p[4];
                int r[4];
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    const int i = i0 + 64 * u;
                    p[u] = i < n ? buf[i] : make_int2(-1, 0);
                }
#pragma unroll
                for (int u = 0; u < 4; u++) r[u] = p[u].x >= 0 ? atomicAdd(&w.cnt[p[u].x], 1) : 0;
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    const int64_t pos = place(base, i0 + 64 * u);
                    if (p[u].x >= 0 && pos >= 0) {
                        w.pairs[pos] = p[u];
                        w.rank[pos] = r[u];
                    }
                }
            }
        }
        __syncthreads();
        n = 0;
    }
    // returns the number of pairs added (identical in every lane)
    __device__ __forceinline__ int add(bool has, int key, int32_t val) {
        const unsigned long long mask = __ballot(has);
        if (mask == 0ull) return 0;
        const int k = __popcll(mask);
        if (n + k > APP_BUF) flush();
        if (has) {
            const int lane = __lane_id();
            buf[n + __popcll(mask & ((1ull << lane) - 1ull))] = make_int2(key, val);
        }
        n += k;
        return k;
    }
};

using RowAppender = Appender<false>;

// ------------------------------------------------------------------------
// per-triangle local frame for the row pass
// ------------------------------------------------------------------------
template <typename R>
struct RowTri {
    R v[3][3];    // local coordinates (level-L cell units, centres at integers)
    R delta;      // bound on |v - exact| (0 when exact)
    int o[3];     // integer origin of the local frame
    int tri;      // triangle id; bit 31: b and c swapped (the yz area is negative)
};

// exact scaled coordinate X = v 2^L - 1/2 of vertex vid, axis a, in float64
__device__ __forceinline__ double scaled64(const DevMesh& m, int vid, int a, double s) {
    return load_coord(m, vid, a) * s - 0.5;
}

// exact float64 local coordinates of T (reloaded from memory)
template <typename R>
__device__ __forceinline__ void local64(const DevMesh& m, const RowTri<R>& T, double s, double v[3][3]) {
    const int64_t t = 3 * (int64_t)(T.tri & 0x7fffffff);
    const int sw = T.tri < 0 ? 1 : 0;
    for (int i = 0; i < 3; i++) {
        const int vid = m.tris[t + (i == 0 ? 0 : (i - 1) ^ sw) + (i == 0 ? 0 : 1)];
        for (int a = 0; a < 3; a++) v[i][a] = scaled64(m, vid, a, s) - (double)T.o[a];
    }
}

struct Stats {
    unsigned fb = 0, ex = 0;
};

// the rows pass counts into slots of 128 bytes, like the q kernel: atomics of
// all its workgroups on the caller's counters complete one every 8.7 ns
template <typename R>
__device__ __forceinline__ void row_stats(unsigned long long* slots, const Stats& st) {
    if (!slots) return;
    unsigned long long* s = slots + (blockIdx.x % ROW_SLOTS) * ROW_SLOT_WORDS;
    const unsigned fb = (unsigned)wave_incl_scan((int)st.fb), ex = (unsigned)wave_incl_scan((int)st.ex);
    if (threadIdx.x != 63) return;
    if (std::is_same<R, float>::value && fb) atomicAdd(&s[0], (unsigned long long)fb);
    if (ex) atomicAdd(&s[1], (unsigned long long)ex);
}

// exact sign of orient2d in the (y,z) plane of local points p, q and (py, pz)
template <typename R>
__device__ __forceinline__ int chain_o2_yz(const DevMesh& m, const RowTri<R>& T, double s, int i, int j,
                                           int py, int pz, Stats& st) {
    int r = orient2d_filter<R>(T.v[i][1], T.v[i][2], T.v[j][1], T.v[j][2], (R)py, (R)pz, T.delta);
    if (r != 0) return r;
    double v[3][3];
    if constexpr (std::is_same<R, float>::value) {
        st.fb++;
        local64(m, T, s, v);
        r = orient2d_filter<double>(v[i][1], v[i][2], v[j][1], v[j][2], (double)py, (double)pz, 0.0);
        if (r != 0) return r;
    } else {
        local64(m, T, s, v);
    }
    st.ex++;
    return orient2d_exact(v[i][1], v[i][2], v[j][1], v[j][2], (double)py, (double)pz);
}

// exact sign of orient3d(v0, v1, v2, P) with local P = (px, py, pz)
template <typename R>
__device__ __forceinline__ int chain_o3(const DevMesh& m, const RowTri<R>& T, double s, int px, int py,
                                        int pz, Stats& st) {
    R P[3] = {(R)px, (R)py, (R)pz};
    int r = orient3d_filter<R>(T.v[0], T.v[1], T.v[2], P, T.delta);
    if (r != 0) return r;
    double v[3][3];
    double P64[3] = {(double)px, (double)py, (double)pz};
    if constexpr (std::is_same<R, float>::value) {
        st.fb++;
        local64(m, T, s, v);
        r = orient3d_filter<double>(v[0], v[1], v[2], P64, 0.0);
        if (r != 0) return r;
    } else {
        local64(m, T, s, v);
    }
    st.ex++;
    return orient3d_exact(v[0], v[1], v[2], P64);
}

// exact sign of orient2d on axes (a0, a1) of the three local vertices
template <typename R>
__device__ __forceinline__ int chain_area(const DevMesh& m, const RowTri<R>& T, double s, int a0, int a1,
                                          Stats& st) {
    int r = orient2d_filter<R>(T.v[0][a0], T.v[0][a1], T.v[1][a0], T.v[1][a1], T.v[2][a0], T.v[2][a1],
                               T.delta);
    if (r != 0) return r;
    double v[3][3];
    local64(m, T, s, v);
    if constexpr (std::is_same<R, float>::value) {
        st.fb++;
        r = orient2d_filter<double>(v[0][a0], v[0][a1], v[1][a0], v[1][a1], v[2][a0], v[2][a1], 0.0);
        if (r != 0) return r;
    }
    st.ex++;
    return orient2d_exact(v[0][a0], v[0][a1], v[1][a0], v[1][a1], v[2][a0], v[2][a1]);
}

// exact sign of orient2d on axes (a0, a1) of local vertices i, j and point (p0, p1)
template <typename R>
__device__ __forceinline__ int chain_o2_axes(const DevMesh& m, const RowTri<R>& T, double s, int i, int j,
                                             int a0, int a1, int p0, int p1, Stats& st) {
    int r = orient2d_filter<R>(T.v[i][a0], T.v[i][a1], T.v[j][a0], T.v[j][a1], (R)p0, (R)p1, T.delta);
    if (r != 0) return r;
    double v[3][3];
    local64(m, T, s, v);
    if constexpr (std::is_same<R, float>::value) {
        st.fb++;
        r = orient2d_filter<double>(v[i][a0], v[i][a1], v[j][a0], v[j][a1], (double)p0, (double)p1, 0.0);
        if (r != 0) return r;
    }
    st.ex++;
    return orient2d_exact(v[i][a0], v[i][a1], v[j][a0], v[j][a1], (double)p0, (double)p1);
}

// Simulation-of-simplicity sign of the yz edge function of u->w at a point
// where it vanishes exactly: the point is moved to (y + e, z + e^2), so
// E changes by -(w_z - u_z) e + (w_y - u_y) e^2.
template <typename R>
__device__ __forceinline__ int sos_tie(const DevMesh& m, const RowTri<R>& T, double s, int i, int j) {
    double v[3][3];
    local64(m, T, s, v);
    const double dz = v[j][2] - v[i][2], dy = v[j][1] - v[i][1];  // exact comparisons via signs
    if (v[j][2] != v[i][2]) return dz > 0 ? -1 : 1;
    if (v[j][1] != v[i][1]) return dy > 0 ? 1 : -1;
    return 0;
}

// vertex ids and coordinates of one triangle, loaded once for every level
struct TriLoad {
    int id[3];
    double x[3][3];
};

__device__ __forceinline__ void tri_load(const DevMesh& m, int64_t t, TriLoad& tl) {
    load_tri(m, t, tl.id);
    for (int i = 0; i < 3; i++) load_vert(m, tl.id[i], tl.x[i]);
}

// Row lines of level L inside the triangle's yz box: [jlo, jhi] x [klo, khi]
// (empty when the low end is above the high one).  X: scaled coordinates.
struct RowBox {
    int jlo, jhi, klo, khi;
    __device__ __forceinline__ bool any() const { return jlo <= jhi && klo <= khi; }
};
__device__ __forceinline__ RowBox row_box(const TriLoad& tl, double s, int ny, int nz) {
    double y[3], z[3];  // the same float64 operations as scaled64
    for (int i = 0; i < 3; i++) {
        y[i] = tl.x[i][1] * s - 0.5;
        z[i] = tl.x[i][2] * s - 0.5;
    }
    const double ymin = fmin(y[0], fmin(y[1], y[2])), ymax = fmax(y[0], fmax(y[1], y[2]));
    const double zmin = fmin(z[0], fmin(z[1], z[2])), zmax = fmax(z[0], fmax(z[1], z[2]));
    return {(int)fmax(ceil(ymin), 0.0), (int)fmin(floor(ymax), (double)(ny - 1)), (int)fmax(ceil(zmin), 0.0),
            (int)fmin(floor(zmax), (double)(nz - 1))};
}

// The local frame of a level (s = 2^L) of a triangle with lines in box b
template <typename R>
__device__ void row_frame(const TriLoad& tl, int tri, double s, const RowBox& b, bool f32_verts, RowTri<R>& T) {
    double X[3][3];  // the same float64 operations as scaled64
    for (int i = 0; i < 3; i++)
        for (int a = 0; a < 3; a++) X[i][a] = tl.x[i][a] * s - 0.5;
    // origin: x from vertex 0, y/z from the first line; fall back to 0 on an
    // axis where the translation would not be exact in float64.  Float32
    // vertices within the coordinate contract (0 or [1/4, n0], n0 2^L <=
    // 2^15) need no check: X and X - o span at most 2^14 .. 2^-25, 40 bits.
    int o[3] = {(int)floor(X[0][0]), b.jlo, b.klo};
    for (int a = 0; a < 3 && !f32_verts; a++) {
        bool exact = true;
        for (int i = 0; i < 3; i++) {
            // Knuth's two-sum error of X - o: zero iff the difference is exact
            const double sum = X[i][a] - (double)o[a];
            const double bb = sum - X[i][a];
            const double err = (X[i][a] - (sum - bb)) + (-(double)o[a] - bb);
            if (err != 0.0) exact = false;
        }
        if (!exact) o[a] = 0;
    }
    R delta = 0;
    for (int i = 0; i < 3; i++) {
        for (int a = 0; a < 3; a++) {
            const double x = X[i][a] - (double)o[a];
            T.v[i][a] = (R)x;
            const double err = fabs((double)T.v[i][a] - x);
            // round the bound up when stored in float
            if ((R)err < err) delta = geo_max(delta, (R)(err * (1.0 + 1e-6)));
            else delta = geo_max(delta, (R)err);
        }
    }
    T.delta = delta;
    T.tri = tri;
    for (int a = 0; a < 3; a++) T.o[a] = o[a];
}

template <typename R>
__device__ __forceinline__ void swap_bc(RowTri<R>& T) {
    for (int a = 0; a < 3; a++) {
        R tmp = T.v[1][a];
        T.v[1][a] = T.v[2][a];
        T.v[2][a] = tmp;
    }
    T.tri ^= (int)0x80000000u;
}

// how the lines meet the triangle: mode 1, proper yz projection (made
// counter-clockwise here); mode 2, edge-on (drop = the axis besides x of a
// plane with non-zero area, areaSign its sign); mode 0, zero area
struct RowMode {
    int mode, drop, areaSign;
};
template <typename R>
__device__ __forceinline__ RowMode row_mode(const DevMesh& m, RowTri<R>& T, double s, Stats& st) {
    const int ayz = chain_area<R>(m, T, s, 1, 2, st);
    if (ayz < 0) swap_bc<R>(T);
    if (ayz != 0) return {1, 0, 0};
    // edge-on or degenerate: find a plane (x,y) or (x,z) with non-zero area
    const int axy = chain_area<R>(m, T, s, 0, 1, st);
    if (axy != 0) return {2, 1, axy};
    const int axz = chain_area<R>(m, T, s, 0, 2, st);
    return {axz != 0 ? 2 : 0, 2, axz};
}

// events of one (triangle, line) pair; e0: parity event or none, e1: surface interval or none
template <typename R>
__device__ void row_events(const DevMesh& m, const RowTri<R>& T, double s, int mode, int drop, int areaSign,
                           int j, int k, int nx, Stats& st, bool& has0, int32_t& e0, bool& has1, int32_t& e1) {
    has0 = has1 = false;
    const int py = j - T.o[1], pz = k - T.o[2];
    R xmn = geo_min(T.v[0][0], geo_min(T.v[1][0], T.v[2][0])) - T.delta;
    R xmx = geo_max(T.v[0][0], geo_max(T.v[1][0], T.v[2][0])) + T.delta;
    if (mode == 1) {
        // proper yz projection (counter-clockwise after set-up)
        int e[3];
        for (int i = 0; i < 3; i++) {
            e[i] = chain_o2_yz<R>(m, T, s, i, (i + 1) % 3, py, pz, st);
            if (e[i] < 0) return;
        }
        bool sos_in = true;
        for (int i = 0; i < 3; i++)
            if (e[i] == 0 && sos_tie<R>(m, T, s, i, (i + 1) % 3) <= 0) sos_in = false;
        // crossing position: smallest integer c with orient3d(T, (c, py, pz)) <= 0
        // (x_hit <= c); orient3d is n_x (x_hit - x) with n_x > 0.
        const R e1x = T.v[1][0] - T.v[0][0], e1y = T.v[1][1] - T.v[0][1], e1z = T.v[1][2] - T.v[0][2];
        const R e2x = T.v[2][0] - T.v[0][0], e2y = T.v[2][1] - T.v[0][1], e2z = T.v[2][2] - T.v[0][2];
        const R nx_ = e1y * e2z - e1z * e2y, ny_ = e1z * e2x - e1x * e2z, nz_ = e1x * e2y - e1y * e2x;
        const int lo = (int)ceil((double)xmn), hi = (int)ceil((double)xmx);
        R xs = T.v[0][0] - (ny_ * ((R)py - T.v[0][1]) + nz_ * ((R)pz - T.v[0][2])) / nx_;
        int c;
        if (!(xs == xs) || xs < (R)lo) c = lo;
        else if (xs > (R)hi) c = hi;
        else c = (int)ceil((double)xs);
        int sc = chain_o3<R>(m, T, s, c, py, pz, st);
        if (sc > 0) {
            do {
                c++;
                sc = chain_o3<R>(m, T, s, c, py, pz, st);
            } while (sc > 0 && c < hi + 1);
        } else {
            while (c > lo) {
                const int sp = chain_o3<R>(m, T, s, c - 1, py, pz, st);
                if (sp > 0) break;
                c--;
                sc = sp;
            }
        }
        const int g = c + T.o[0];  // global index of the first centre at or right of the crossing
        if (sos_in && g >= 1) {
            has0 = true;
            e0 = g < nx ? g : nx;
        }
        if (sc == 0 && g >= 0 && g < nx) {
            has1 = true;
            e1 = row_surf_entry(g, g);
        }
        return;
    }
    // mode 2: edge-on triangle (zero yz area, non-degenerate).  The line meets
    // it only if the line point is on the projected segment; then every
    // centre of the line inside the closed triangle is on the surface.
    {
        // longest projected edge (any edge with distinct yz endpoints works)
        int bi = 0;
        R best = -1;
        for (int i = 0; i < 3; i++) {
            const int jn = (i + 1) % 3;
            const R l = geo_fabs(T.v[jn][1] - T.v[i][1]) + geo_fabs(T.v[jn][2] - T.v[i][2]);
            if (l > best) { best = l; bi = i; }
        }
        if (chain_o2_yz<R>(m, T, s, bi, (bi + 1) % 3, py, pz, st) != 0) return;
        const int pw = drop == 1 ? py : pz;  // coordinate kept beside x
        bool found = false;
        int first = 0, last = 0;  // local indices; may be negative
        const int lo = (int)ceil((double)xmn), hi = (int)floor((double)xmx);
        for (int c = lo; c <= hi; c++) {
            bool in = true;
            for (int i = 0; i < 3 && in; i++) {
                const int r = chain_o2_axes<R>(m, T, s, i, (i + 1) % 3, 0, drop, c, pw, st);
                if (r * areaSign < 0) in = false;
            }
            if (in) {
                if (!found) first = c;
                found = true;
                last = c;
            } else if (found) {
                break;  // convex: the inside centres are contiguous
            }
        }
        if (found) {
            int gl = first + T.o[0], gh = last + T.o[0];
            gl = gl < 0 ? 0 : gl;
            gh = gh > nx - 1 ? nx - 1 : gh;
            if (gl <= gh) {
                has1 = true;
                e1 = row_surf_entry(gl, gh);
            }
        }
    }
}

// ------------------------------------------------------------------------
// ROWS pass: the levels' keys are consecutive ranges of one key space.
//
// A wave takes a batch of up to 64 triangles.  First every lane finds, for its
// triangle and each level, whether it has row lines there at all; the
// (triangle, level) items that have are set up 64 at a time, one per lane (a
// fine triangle has lines on one level or two of five), and kept in LDS; then
// their (item, line) pairs are numbered through and every lane takes one pair,
// whatever triangle it is of.  Bound by VALU work and its latency: the lines
// per item vary from one to hundreds, and a lane that walked the lines of its
// own triangle left the others idle.  An item with more than ROW_BIG lines is
// cut into pieces that a second launch spreads over the chip (a CAD mesh has a
// dozen triangles of 10^5 lines; overflow of that list is done in place).
// Before (one lane per triangle, its lines in turn) and now, float32 form:
// 0.61 and 0.42 ms on 7.2M triangles over levels 0..4, 0.16 and 0.10 ms on 112k
// over 0..3, 127 and 22 us on 1,792 over 0..2, 6.4 and 0.08 ms on a 1,024-
// triangle cylinder over 0..3; float64 form 0.28 and 0.19 ms on 1.02M.
// ------------------------------------------------------------------------
constexpr int ROW_BIG = 128;          // lines of an item done by its own wave
constexpr int ROW_PIECES = 64;        // most pieces of an item

template <typename R>
struct RowItems {  // field-major: lane i writes item i, any lane reads any item
    R v[9][64], delta[64];
    int o[3][64], tri[64];
    int jlo[64], klo[64], nj[64];
    int base[64];  // first key of the item's level
    int meta[64];  // level | mode << 4 | drop << 6 | (areaSign + 1) << 8
    int pre[64];   // number of the item's first pair
};

template <typename R>
__device__ __forceinline__ void item_store(RowItems<R>& I, int i, const RowTri<R>& T, const RowBox& b, int base, int L,
                                           const RowMode& md, int pre) {
    for (int k = 0; k < 9; k++) I.v[k][i] = T.v[k / 3][k % 3];
    I.delta[i] = T.delta;
    for (int a = 0; a < 3; a++) I.o[a][i] = T.o[a];
    I.tri[i] = T.tri;
    I.jlo[i] = b.jlo;
    I.klo[i] = b.klo;
    I.nj[i] = b.jhi - b.jlo + 1;
    I.base[i] = base;
    I.meta[i] = L | md.mode << 4 | md.drop << 6 | (md.areaSign + 1) << 8;
    I.pre[i] = pre;
}

// events of line `line` (j fastest) of the item, appended by the whole wave
template <typename R>
__device__ __forceinline__ void line_events(const DevMesh& m, const int n0[3], bool on, const RowTri<R>& T, int L,
                                            const RowMode& md, int jlo, int klo, int nj, int base, int line,
                                            RowAppender& app, Stats& st) {
    bool h0 = false, h1 = false;
    int32_t e0 = 0, e1 = 0;
    int key = 0;
    if (on) {
        const unsigned q = (unsigned)line / (unsigned)nj;
        const int j = jlo + (line - (int)q * nj), k = klo + (int)q;
        key = base + j + (n0[1] << L) * k;
        row_events<R>(m, T, ldexp(1.0, L), md.mode, md.drop, md.areaSign, j, k, n0[0] << L, st, h0, e0, h1, e1);
    }
    app.add(h0, key, e0);
    app.add(h1, key, e1);
}

template <typename R>
__device__ __forceinline__ void item_events(const DevMesh& m, const int n0[3], bool on, const RowItems<R>& I, int i,
                                            int line, RowAppender& app, Stats& st) {
    RowTri<R> P;
    for (int k = 0; k < 9; k++) P.v[k / 3][k % 3] = I.v[k][i];
    P.delta = I.delta[i];
    for (int a = 0; a < 3; a++) P.o[a] = I.o[a][i];
    P.tri = I.tri[i];
    const int meta = I.meta[i];
    line_events<R>(m, n0, on, P, meta & 15, {meta >> 4 & 3, meta >> 6 & 3, (meta >> 8) - 1}, I.jlo[i], I.klo[i], I.nj[i],
                   I.base[i], line, app, st);
}

// Pieces of an item with n lines: written to the list (triangle, level index,
// first line, lines) by its lane.  Returns whether the list took them.
__device__ __forceinline__ bool list_item(const BinWork& w, bool big, int tri, int l, int n) {
    const int want = big ? ((n + ROW_PIECES - 1) / ROW_PIECES + 63) & ~63 : 1;
    const int piece = want < ROW_BIG ? ROW_BIG : want;
    const int k = big ? (n + piece - 1) / piece : 0;
    const int incl = wave_incl_scan(k), total = __shfl(incl, 63, 64);
    // a full list is not added to any more, so that its counter cannot wrap
    int at = BIN_LIST_CAP;
    if (threadIdx.x == 0 && __hip_atomic_load(&w.ctl->list_n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < BIN_LIST_CAP)
        at = atomicAdd(&w.ctl->list_n, total);
    at = __shfl(at, 0, 64);
    at += incl - k;
    const bool taken = big && at + k <= BIN_LIST_CAP;
    for (int i = 0; i < k; i++)  // a refused item leaves empty pieces
        if (at + i < BIN_LIST_CAP)
            w.list[at + i] = make_int4(tri, l, i * piece, !taken ? 0 : (n - i * piece < piece ? n - i * piece : piece));
    return taken;
}

template <typename R>
__device__ __forceinline__ void rows_levels_body(const DevMesh& m, const DevLevel& d, const RowLevels& rl, int tpw,
                                                 const BinWork& w) {
    __shared__ int2 sbuf[APP_BUF];
    __shared__ RowItems<R> I;
    __shared__ uint16_t items[64 * GEO_MAX_LEVELS];  // lane | level index << 6
    __shared__ int mark[64];
    __shared__ int sbase[GEO_MAX_LEVELS];
    const int lane = threadIdx.x;
    if (lane < GEO_MAX_LEVELS) sbase[lane] = rl.base[lane];
    RowAppender app{sbuf, 0, w, nullptr};
    Stats st;
    const bool f32v = m.vdtype == GEO_F32;
    const int64_t stride = (int64_t)gridDim.x * tpw;
    for (int64_t base = (int64_t)blockIdx.x * tpw; base < m.nt; base += stride) {
        const int64_t t = base + lane;
        TriLoad tl{};
        const bool live = lane < tpw && t < m.nt;
        if (live) tri_load(m, t, tl);
        int nitems = 0;
        __syncthreads();
        for (int l = 0; l < rl.nlev; l++) {
            const int L = rl.lmin + l;
            const bool has = live && row_box(tl, ldexp(1.0, L), d.n0[1] << L, d.n0[2] << L).any();
            const unsigned long long bal = __ballot(has);
            if (has) items[nitems + __popcll(bal & ((1ull << lane) - 1ull))] = (uint16_t)(lane | l << 6);
            nitems += __popcll(bal);
        }
        __syncthreads();
        for (int c = 0; c < nitems; c += 64) {  // uniform
            const bool valid = c + lane < nitems;
            const int code = valid ? items[c + lane] : lane;
            const int src = code & 63, l = code >> 6, L = rl.lmin + l;
            TriLoad ti;
            for (int i = 0; i < 3; i++)
                for (int a = 0; a < 3; a++) ti.x[i][a] = __shfl(tl.x[i][a], src, 64);
            const int tri = (int)base + src;
            RowBox b{0, -1, 0, -1};
            RowMode md{0, 0, 0};
            RowTri<R> T;
            int n = 0;
            if (valid) {
                const double s = ldexp(1.0, L);
                b = row_box(ti, s, d.n0[1] << L, d.n0[2] << L);
                row_frame<R>(ti, tri, s, b, f32v, T);
                md = row_mode<R>(m, T, s, st);
                if (md.mode) n = (b.jhi - b.jlo + 1) * (b.khi - b.klo + 1);
            }
            // large items: to the list, or (refused) below by the whole wave
            int nbig = n > ROW_BIG ? n : 0;
            if (__any(nbig > 0) && list_item(w, nbig > 0, tri, l, nbig)) nbig = 0;
            if (n > ROW_BIG) n = 0;
            const int incl = wave_incl_scan(n), total = __shfl(incl, 63, 64);
            __syncthreads();
            if (n > 0 || nbig > 0) item_store<R>(I, lane, T, b, sbase[l], L, md, incl - n);
            for (int done = 0; done < total; done += 64) {  // uniform
                // item of each pair: its number where the item's pairs start
                // (or the chunk does), carried on by a prefix maximum
                mark[lane] = 0;
                __syncthreads();
                if (n > 0 && incl > done && incl - n < done + 64)
                    mark[incl - n > done ? incl - n - done : 0] = lane;
                __syncthreads();
                const int i = wave_incl_max(mark[lane]);
                item_events<R>(m, d.n0, done + lane < total, I, i, done + lane - I.pre[i], app, st);
            }
            unsigned long long rest = __ballot(nbig > 0);
            if (rest) __syncthreads();
            while (rest) {  // uniform
                const int i = __ffsll(rest) - 1;
                rest &= rest - 1;
                const int nl = __shfl(nbig, i, 64);
                for (int q = 0; q < nl; q += 64) item_events<R>(m, d.n0, q + lane < nl, I, i, q + lane, app, st);
            }
        }
    }
    app.flush();
    row_stats<R>(w.slots, st);
}

// float32 form: 3 waves per SIMD; the float64 form keeps its registers (a cap
// spills it heavily)
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3, 8)))
k_rows_levels_f32(DevMesh m, DevLevel d, RowLevels rl, int tpw, BinWork w) {
    rows_levels_body<float>(m, d, rl, tpw, w);
}

__global__ void __launch_bounds__(64) k_rows_levels_f64(DevMesh m, DevLevel d, RowLevels rl, int tpw, BinWork w) {
    rows_levels_body<double>(m, d, rl, tpw, w);
}

// the listed pieces of large items, one wave per piece, lanes over its lines
template <typename R>
__global__ void __launch_bounds__(64) k_rows_pieces(DevMesh m, DevLevel d, RowLevels rl, BinWork w) {
    __shared__ int2 sbuf[APP_BUF];
    const int lane = threadIdx.x;
    int np = w.ctl->list_n;
    if (np < 0 || np > BIN_LIST_CAP) np = BIN_LIST_CAP;
    if ((int)blockIdx.x >= np) return;
    RowAppender app{sbuf, 0, w, nullptr};
    Stats st;
    for (int e = blockIdx.x; e < np; e += gridDim.x) {
        const int4 p = w.list[e];
        if (p.w <= 0) continue;  // uniform
        const int l = p.y, L = rl.lmin + l;
        const double s = ldexp(1.0, L);
        TriLoad tl;
        tri_load(m, p.x, tl);
        const RowBox b = row_box(tl, s, d.n0[1] << L, d.n0[2] << L);
        RowTri<R> T;
        row_frame<R>(tl, p.x, s, b, m.vdtype == GEO_F32, T);
        Stats again;  // counted where the item was listed
        const RowMode md = row_mode<R>(m, T, s, again);
        for (int i = 0; i < p.w; i += 64)  // uniform
            line_events<R>(m, d.n0, i + lane < p.w, T, L, md, b.jlo, b.klo, b.jhi - b.jlo + 1, rl.base[l],
                           p.z + i + lane, app, st);
    }
    app.flush();
    row_stats<R>(w.slots, st);
}

// zero the counters, the statistics slots and the key counts
__global__ void k_bins_zero(BinWork w, int64_t nkeys) {
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, n = (int64_t)gridDim.x * blockDim.x;
    if (i0 == 0) {
        w.ctl->up = w.ctl->down = 0;
        w.ctl->list_n = 0;
    }
    if (w.slots && blockIdx.x == 0)
        for (int i = threadIdx.x; i < ROW_SLOTS * ROW_SLOT_WORDS; i += blockDim.x) w.slots[i] = 0ull;
    for (int64_t i = i0; i < nkeys; i += n) w.cnt[i] = 0;
}

// staged pairs are the first `up` and the last `down` of the array
struct BinPairs {
    int64_t up, n;
};
__device__ __forceinline__ BinPairs staged_pairs(const BinWork& w) {
    const unsigned long long c = (unsigned long long)w.cap, up = w.ctl->up, down = w.ctl->down;
    const int64_t u = (int64_t)(up < c ? up : c);
    return {u, u + (int64_t)(down < c ? down : c)};
}

// place the pairs of every level: the level of a pair is found from its key;
// the statistics slots are added to the caller's counters
__global__ void k_rows_levels_scatter(BinWork w, RowLevels rl, uint64_t* stats) {
    __shared__ int sbase[GEO_MAX_LEVELS + 1];
    __shared__ const int32_t* soff[GEO_MAX_LEVELS];
    __shared__ int32_t* sval[GEO_MAX_LEVELS];
    __shared__ int64_t scap[GEO_MAX_LEVELS];
    if (threadIdx.x < GEO_MAX_LEVELS + 1) sbase[threadIdx.x] = rl.base[threadIdx.x];
    if (threadIdx.x < GEO_MAX_LEVELS) {
        soff[threadIdx.x] = rl.off[threadIdx.x];
        sval[threadIdx.x] = rl.val[threadIdx.x];
        scap[threadIdx.x] = rl.cap[threadIdx.x];
    }
    __syncthreads();
    if (w.slots && blockIdx.x == 0 && threadIdx.x < ROW_SLOTS) {
        const unsigned long long fb = w.slots[threadIdx.x * ROW_SLOT_WORDS],
                                 ex = w.slots[threadIdx.x * ROW_SLOT_WORDS + 1];
        if (fb) atomicAdd((unsigned long long*)&stats[GEO_STAT_F32_TO_F64], fb);
        if (ex) atomicAdd((unsigned long long*)&stats[GEO_STAT_EXACT], ex);
    }
    const BinPairs bp = staged_pairs(w);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < bp.n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t at = i < bp.up ? i : w.cap - 1 - (i - bp.up);
        const int2 p = w.pairs[at];
        int l = 0;
        for (int q = 1; q < rl.nlev; q++) l += p.x >= sbase[q] ? 1 : 0;
        const int64_t pos = (int64_t)soff[l][p.x - sbase[l]] + w.rank[at];
        if (pos >= 0 && pos < scap[l]) sval[l][pos] = p.y;
    }
}

// ------------------------------------------------------------------------
// LINKS: triangle / widened block box overlap (separating axes, with outward
// margins so that rounding can only add candidates)
// ------------------------------------------------------------------------

// Triangles of a wave's batch, with the quantities of the separating-axis test
// (V: the vertices' own type).  Field-major in LDS: lane i writes triangle i,
// any lane reads any triangle.
template <typename V>
struct LinkItems {
    V v[9][64];
    double n[3][64];                // e0 x e1 (rounded; any vector is a valid separating axis)
    double nvmin[64], nvmax[64];    // min / max over the vertices of n . v
    double nrad[64];                // radius of the block's reach along n, with its margins
    int lo[3][64];                  // candidate blocks: lo + (0..sx-1, 0..sy-1, ..)
    int sx[64], sy[64];
    int ix[64], iy[64];             // ceil(2^20 / sx), ceil(2^20 / sy)
    int pre[64];                    // number of the triangle's first pair
};

// Conservative triangle / cube overlap (centre c, half side hs): separating
// axes are the box normals, the triangle normal and the nine edge crosses,
// each with a margin that covers the rounding of the test.  The box normals
// are the candidate range itself (the caller enumerates exactly the blocks
// whose widened box meets the triangle's bounding box); stage one takes the
// triangle normal, stage two the edges.
template <typename V>
__device__ __forceinline__ bool tri_box_stage1(const double c[3], const LinkItems<V>& I, int i) {
    // the normal axis: projections n . v_i - n . c against the box radius; the
    // margin bounds the rounding of the dot products (4.5 u each side)
    const double p0 = I.n[0][i] * c[0], p1 = I.n[1][i] * c[1], p2 = I.n[2][i] * c[2];
    const double nc = p0 + p1 + p2;
    const double rn = I.nrad[i] + 5e-16 * (fabs(p0) + fabs(p1) + fabs(p2));
    return !(I.nvmin[i] - nc > rn || I.nvmax[i] - nc < -rn);
}

// The nine edge axes in float.  The vertices relative to the centre,
// w = v - c, are formed in double and rounded once; |w| is at most the
// triangle's extent plus the box's, so each projection x1 w1 + x2 w2 carries
// an absolute error below 4u (|x1| + |x2|) max|w| (u = 2^-24: the roundings
// of w, of the edge components and of the two products and the sum).  The
// radius is widened by 1e-6 max|w| (|x1| + |x2|), more than twice that, and
// by a relative 1e-5 for its own rounding, so an axis is only taken as
// separating where it separates the exact figures; the 1e-30 floor covers
// products that underflow.
template <typename V>
__device__ __forceinline__ bool tri_box_stage2(const double c[3], double hs, const LinkItems<V>& I, int i) {
    double v[3][3];
    float w[3][3];
    float wmax = 0.0f;
    for (int k = 0; k < 3; k++)
        for (int a = 0; a < 3; a++) {
            v[k][a] = (double)I.v[3 * k + a][i];
            w[k][a] = (float)(v[k][a] - c[a]);
            wmax = fmaxf(wmax, fabsf(w[k][a]));
        }
    const float hsf = (float)hs * (1.0f + 1e-5f) + 1e-6f * wmax + 1e-30f;
    // axis = e_box(a) x e(k), nonzero in components b1 = a+1 and b2 = a+2
    bool hit = true;
    for (int k = 0; k < 3; k++) {
        float e[3];
        for (int a = 0; a < 3; a++) e[a] = (float)(v[(k + 1) % 3][a] - v[k][a]);
        for (int a = 0; a < 3; a++) {
            const int b1 = (a + 1) % 3, b2 = (a + 2) % 3;
            const float x1 = -e[b2], x2 = e[b1];
            const float p0 = x1 * w[0][b1] + x2 * w[0][b2];
            const float p1 = x1 * w[1][b1] + x2 * w[1][b2];
            const float p2 = x1 * w[2][b1] + x2 * w[2][b2];
            const float r = hsf * (fabsf(x1) + fabsf(x2));
            const float mn = fminf(p0, fminf(p1, p2)), mx = fmaxf(p0, fmaxf(p1, p2));
            hit &= !(mn > r || mx < -r);
        }
    }
    return hit;
}

// The LINKS pass.  A wave takes a batch of up to 64 triangles, one per lane for
// the set-up (kept in LDS); their (triangle, candidate block) pairs are then
// numbered through and every lane takes LINKS_U pairs at a time, whatever
// triangle they are of, so that their forest descents overlap.  Bound by VALU
// work and by the latency of the descents.  A triangle with more than LINK_BIG
// candidates is cut into pieces for a second launch, as in the ROWS pass.
// Before (one lane per triangle, its candidates in turn) and now, both launches:
// 0.81 and 0.54 ms on 7.2M triangles (24.3M entries), 160 and 50 us on 112k, 100
// and 19 us on 1,792, 3.31 and 0.065 ms on a 1,024-triangle cylinder.  Two
// counters instead of one and buffers of 512 instead of 1,024 pairs are 0.15 ms
// of the first.
constexpr int LINKS_U = 4;
// (at most 1,024: ix and iy divide exactly.  The call with 128, 256 and 512: 95,
// 48 and 48 us on an icosphere of 5,120 triangles over 0.97M blocks, 263, 139 and
// 139 us on a cylinder of 40,000, 68, 85 and 123 us on one of 1,024)
constexpr int LINK_BIG = 256;
constexpr int LINK_PIECES = 64;    // most pieces of a triangle
constexpr int64_t LINK_PIECE_MAX = 1 << 30;

using LinkAppender = Appender<true>;

struct LinkGrid {  // block geometry of the level
    int L, nb[3], nb0[3];
    double h, bw, ibw, hs;
};
__device__ __forceinline__ LinkGrid link_grid(const DevLevel& d) {
    LinkGrid g;
    g.L = d.level;
    g.h = ldexp(1.0, -g.L);
    g.bw = 4.0 * g.h;
    g.ibw = ldexp(1.0, g.L - 2);  // 1 / bw, exact
    // half side of the box [4bh - h/2, 4(b+1)h + h/2] that the block's links reach
    g.hs = (0.5 * g.bw + 0.5 * g.h) * (1.0 + 1e-9);
    for (int a = 0; a < 3; a++) {
        g.nb0[a] = d.n0[a] >> 2;
        g.nb[a] = g.nb0[a] << g.L;
    }
    return g;
}

// Set-up of triangle t as item i: its candidate range and the data of the
// tests.  Returns the number of candidates (0 for zero area).
template <typename V>
__device__ __forceinline__ int64_t link_setup(const DevMesh& m, int64_t t, const LinkGrid& g, LinkItems<V>& I, int i) {
    double v[3][3];
    int vid[3];
    load_tri(m, t, vid);
    for (int k = 0; k < 3; k++) {
        V x[3];
        __builtin_memcpy(x, static_cast<const V*>(m.verts) + 3 * (int64_t)vid[k], sizeof(x));
        for (int a = 0; a < 3; a++) {
            I.v[3 * k + a][i] = x[a];
            v[k][a] = (double)x[a];
        }
    }
    // zero-area triangles never meet a segment: exact test (all three
    // coordinate-plane projections have zero area)
    if (orient2d_filter<double>(v[0][1], v[0][2], v[1][1], v[1][2], v[2][1], v[2][2], 0.0) == 0 &&
        orient2d_filter<double>(v[0][2], v[0][0], v[1][2], v[1][0], v[2][2], v[2][0], 0.0) == 0 &&
        orient2d_filter<double>(v[0][0], v[0][1], v[1][0], v[1][1], v[2][0], v[2][1], 0.0) == 0 &&
        orient2d_exact(v[0][1], v[0][2], v[1][1], v[1][2], v[2][1], v[2][2]) == 0 &&
        orient2d_exact(v[0][2], v[0][0], v[1][2], v[1][0], v[2][2], v[2][0]) == 0 &&
        orient2d_exact(v[0][0], v[0][1], v[1][0], v[1][1], v[2][0], v[2][1]) == 0)
        return 0;
    double e0[3], e1[3], n[3];
    for (int a = 0; a < 3; a++) {
        e0[a] = v[1][a] - v[0][a];
        e1[a] = v[2][a] - v[1][a];
    }
    n[0] = e0[1] * e1[2] - e0[2] * e1[1];
    n[1] = e0[2] * e1[0] - e0[0] * e1[2];
    n[2] = e0[0] * e1[1] - e0[1] * e1[0];
    double nvmin = 1e300, nvmax = -1e300, nvabs = 0.0;
    for (int k = 0; k < 3; k++) {
        const double p = n[0] * v[k][0] + n[1] * v[k][1] + n[2] * v[k][2];
        nvmin = fmin(nvmin, p);
        nvmax = fmax(nvmax, p);
        nvabs = fmax(nvabs, fabs(n[0] * v[k][0]) + fabs(n[1] * v[k][1]) + fabs(n[2] * v[k][2]));
    }
    const double n1 = fabs(n[0]) + fabs(n[1]) + fabs(n[2]);
    I.nvmin[i] = nvmin;
    I.nvmax[i] = nvmax;
    I.nrad[i] = g.hs * n1 * (1.0 + 1e-9) + 1e-12 * n1 + 5e-16 * nvabs;
    int sz[3];
    for (int a = 0; a < 3; a++) {
        I.n[a][i] = n[a];
        const double mn = fmin(v[0][a], fmin(v[1][a], v[2][a])), mx = fmax(v[0][a], fmax(v[1][a], v[2][a]));
        // block b's links reach [4bh - h/2, 4bh + 4.5h]: it meets
        // [mn, mx] iff (mn - 4.5h) / bw <= b <= (mx + h/2) / bw (the
        // roundings are monotone and bw is a power of two; the 1e-7
        // only widens the range)
        int lo = (int)ceil((mn - 4.5 * g.h) * g.ibw - 1e-7);
        int hi = (int)floor((mx + 0.5 * g.h) * g.ibw + 1e-7);
        lo = lo < 0 ? 0 : lo;
        hi = hi > g.nb[a] - 1 ? g.nb[a] - 1 : hi;
        I.lo[a][i] = lo;
        sz[a] = hi - lo + 1;
    }
    if (sz[0] <= 0 || sz[1] <= 0 || sz[2] <= 0) return 0;
    I.sx[i] = sz[0];
    I.sy[i] = sz[1];
    I.ix[i] = (1048575 + sz[0]) / sz[0];
    I.iy[i] = (1048575 + sz[1]) / sz[1];
    return (int64_t)sz[0] * sz[1] * sz[2];
}

// LINKS_U pairs per lane (item i[u], candidate block b[u], on[u]) through both
// tests and down the forest; the blocks found are appended
template <typename V>
__device__ __forceinline__ void link_pairs(const DevLevel& d, const LinkGrid& g, const LinkItems<V>& I,
                                           const bool on[LINKS_U], const int i[LINKS_U], const int b[LINKS_U][3],
                                           const int32_t tri[LINKS_U], LinkAppender& app) {
    int idx[LINKS_U];
#pragma unroll
    for (int u = 0; u < LINKS_U; u++) {
        idx[u] = -1;
        if (on[u]) {
            const double c[3] = {(b[u][0] + 0.5) * g.bw, (b[u][1] + 0.5) * g.bw, (b[u][2] + 0.5) * g.bw};
            if (tri_box_stage1<V>(c, I, i[u]) && tri_box_stage2<V>(c, g.hs, I, i[u]))
                idx[u] = (b[u][0] >> g.L) + g.nb0[0] * ((b[u][1] >> g.L) + g.nb0[1] * (b[u][2] >> g.L));
        }
    }
    for (int l = 0; l < g.L; l++) {
        int ch[LINKS_U];
        const int sh = g.L - 1 - l;
#pragma unroll
        for (int u = 0; u < LINKS_U; u++) ch[u] = idx[u] >= 0 ? d.child[l][idx[u]] : -1;
#pragma unroll
        for (int u = 0; u < LINKS_U; u++)
            idx[u] = ch[u] < 0 ? -1
                               : ch[u] + (((b[u][0] >> sh) & 1) | (((b[u][1] >> sh) & 1) << 1) |
                                          (((b[u][2] >> sh) & 1) << 2));
    }
#pragma unroll
    for (int u = 0; u < LINKS_U; u++) app.add(idx[u] >= 0, idx[u], tri[u]);
}

// candidates first .. first + count - 1 of item i (its candidate box by
// divisions), by the whole wave
template <typename V>
__device__ void link_range(const DevLevel& d, const LinkGrid& g, const LinkItems<V>& I, int i, int32_t t, int64_t first,
                           int64_t count, LinkAppender& app) {
    // a lane's candidate by division once, then 64 further on each time by carries
    const int lane = threadIdx.x;
    const int sx = I.sx[i], sy = I.sy[i], dx = 64 % sx, dy = 64 / sx % sy, dz = 64 / sx / sy;
    int x, y, z;
    if (first + lane <= UINT32_MAX) {
        const unsigned c = (unsigned)(first + lane), r = c / (unsigned)sx;
        x = (int)(c - r * (unsigned)sx);
        z = (int)(r / (unsigned)sy);
        y = (int)(r - (unsigned)z * (unsigned)sy);
    } else {
        const int64_t c = first + lane, r = c / sx;
        x = (int)(c - r * sx);
        y = (int)(r % sy);
        z = (int)(r / sy);
    }
    for (int64_t q0 = 0; q0 < count; q0 += 64 * LINKS_U) {  // uniform
        bool on[LINKS_U];
        int item[LINKS_U], b[LINKS_U][3];
        int32_t tri[LINKS_U];
#pragma unroll
        for (int u = 0; u < LINKS_U; u++) {
            on[u] = q0 + 64 * u + lane < count;
            item[u] = i;
            tri[u] = t;
            b[u][0] = I.lo[0][i] + x;
            b[u][1] = I.lo[1][i] + y;
            b[u][2] = I.lo[2][i] + z;
            x += dx;
            y += dy;
            z += dz;
            if (x >= sx) {
                x -= sx;
                y++;
            }
            if (y >= sy) {
                y -= sy;
                z++;
            }
        }
        link_pairs<V>(d, g, I, on, item, b, tri, app);
    }
}

// pieces of a large triangle to the list (triangle, first candidate in 64
// bits, count); returns whether the list took them
__device__ __forceinline__ bool list_links(const BinWork& w, int64_t n, int32_t tri) {
    constexpr int64_t step = 64 * LINKS_U;  // what a wave takes at a time
    const int64_t want = ((n + LINK_PIECES - 1) / LINK_PIECES + step - 1) & ~(step - 1);
    const bool big = n > 0 && want <= LINK_PIECE_MAX;
    const int k = big ? (int)((n + want - 1) / want) : 0;
    const int incl = wave_incl_scan(k), total = __shfl(incl, 63, 64);
    // a full list is not added to any more, so that its counter cannot wrap
    int at = BIN_LIST_CAP;
    if (threadIdx.x == 0 && __hip_atomic_load(&w.ctl->list_n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < BIN_LIST_CAP)
        at = atomicAdd(&w.ctl->list_n, total);
    at = __shfl(at, 0, 64) + incl - k;
    const bool taken = big && at + k <= BIN_LIST_CAP;
    for (int q = 0; q < k; q++) {  // a refused triangle leaves empty pieces
        const int64_t first = q * want;
        const int count = taken ? (int)(n - first < want ? n - first : want) : 0;
        if (at + q < BIN_LIST_CAP) w.list[at + q] = make_int4(tri, (int)(uint32_t)first, (int)(first >> 32), count);
    }
    return taken;
}

template <typename V>
__global__ void __launch_bounds__(64) k_links_pass1(DevMesh m, DevLevel d, int tpw, BinWork w) {
    __shared__ int2 sbuf[APP_BUF];
    __shared__ LinkItems<V> I;
    __shared__ int mark[64 * LINKS_U];
    __shared__ unsigned stab[APP_TAB];
    const int lane = threadIdx.x;
    LinkAppender app{sbuf, 0, w, stab};
    const LinkGrid g = link_grid(d);
    const int64_t stride = (int64_t)gridDim.x * tpw;
    for (int64_t base = (int64_t)blockIdx.x * tpw; base < m.nt; base += stride) {
        const int64_t t = base + lane;
        int64_t nall = 0;
        __syncthreads();
        if (lane < tpw && t < m.nt) nall = link_setup<V>(m, t, g, I, lane);
        int64_t nbig = nall > LINK_BIG ? nall : 0;
        if (__any(nbig > 0) && list_links(w, nbig, (int32_t)t)) nbig = 0;
        const int n = nall > LINK_BIG ? 0 : (int)nall;
        const int incl = wave_incl_scan(n), total = __shfl(incl, 63, 64);
        I.pre[lane] = incl - n;
        for (int done = 0; done < total; done += 64 * LINKS_U) {  // uniform
            // triangle of each pair: its number where its pairs start (or the
            // chunk does), carried on by a prefix maximum
#pragma unroll
            for (int u = 0; u < LINKS_U; u++) mark[64 * u + lane] = 0;
            __syncthreads();
            if (n > 0 && incl > done && incl - n < done + 64 * LINKS_U)
                mark[incl - n > done ? incl - n - done : 0] = lane;
            __syncthreads();
            bool on[LINKS_U];
            int item[LINKS_U], b[LINKS_U][3];
            int32_t tri[LINKS_U];
            int last = 0;
#pragma unroll
            for (int u = 0; u < LINKS_U; u++) {
                const int own = wave_incl_max(mark[64 * u + lane]);
                const int i = own > last ? own : last;
                last = __shfl(i, 63, 64);
                const int p = done + 64 * u + lane;
                on[u] = p < total;
                item[u] = i;
                tri[u] = (int32_t)base + i;
                // candidate c = x + sx (y + sy z), c < LINK_BIG
                const int c = on[u] ? p - I.pre[i] : 0;
                const int r = (c * I.ix[i]) >> 20, z = (r * I.iy[i]) >> 20;
                b[u][0] = I.lo[0][i] + c - r * I.sx[i];
                b[u][1] = I.lo[1][i] + r - z * I.sy[i];
                b[u][2] = I.lo[2][i] + z;
            }
            link_pairs<V>(d, g, I, on, item, b, tri, app);
        }
        unsigned long long rest = __ballot(nbig > 0);  // refused by the list: by the whole wave
        if (rest) __syncthreads();
        while (rest) {  // uniform
            const int i = __ffsll(rest) - 1;
            rest &= rest - 1;
            link_range<V>(d, g, I, i, (int32_t)base + i, 0, __shfl((long long)nbig, i, 64), app);
        }
    }
    app.flush();
}

// the listed pieces of large triangles, one wave per piece
template <typename V>
__global__ void __launch_bounds__(64) k_links_pieces(DevMesh m, DevLevel d, BinWork w) {
    __shared__ int2 sbuf[APP_BUF];
    __shared__ LinkItems<V> I;
    __shared__ unsigned stab[APP_TAB];
    int np = w.ctl->list_n;
    if (np < 0 || np > BIN_LIST_CAP) np = BIN_LIST_CAP;
    if ((int)blockIdx.x >= np) return;
    LinkAppender app{sbuf, 0, w, stab};
    const LinkGrid g = link_grid(d);
    for (int e = blockIdx.x; e < np; e += gridDim.x) {
        const int4 p = w.list[e];
        if (p.w <= 0) continue;  // uniform
        __syncthreads();
        if (threadIdx.x == 0) link_setup<V>(m, p.x, g, I, 0);
        __syncthreads();
        link_range<V>(d, g, I, 0, p.x, (int64_t)(((uint64_t)(uint32_t)p.z << 32) | (uint32_t)p.y), p.w, app);
    }
    app.flush();
}

__global__ void k_bins_scatter(BinWork w, const int32_t* off, int32_t* val) {
    const BinPairs bp = staged_pairs(w);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < bp.n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t at = i < bp.up ? i : w.cap - 1 - (i - bp.up);
        const int2 p = w.pairs[at];
        const int64_t pos = (int64_t)off[p.x] + w.rank[at];
        if (pos >= 0 && pos < w.cap) val[pos] = p.y;
    }
}

__global__ void k_check_mesh(DevMesh m, DevLevel d, uint64_t* stats) {
    // one vertex per thread, its three coordinates in turn (no index division)
    unsigned bad = 0;
    const double top[3] = {(double)d.n0[0], (double)d.n0[1], (double)d.n0[2]};
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < m.nv; v += (int64_t)gridDim.x * blockDim.x) {
        double xs[3];
        load_vert(m, (int)v, xs);
        for (int a = 0; a < 3; a++) {
            const double x = xs[a];
            const bool ok = x == 0.0 || (x >= 0.25 && x <= top[a]);
            bad += ok ? 0u : 1u;
        }
    }
    wave_count(&stats[GEO_STAT_CONTRACT], bad);
}

inline unsigned grid_for(int64_t n, int threads, int64_t maxg = 1 << 16) {
    int64_t g = (n + threads - 1) / threads;
    if (g > maxg) g = maxg;
    if (g < 1) g = 1;
    return (unsigned)g;
}

}  // namespace

int launch_rows_levels(const DevMesh& m, const DevLevel& d, int precision, const RowLevels& rl, const BinWork& w,
                       hipStream_t s) {
    if (m.nt == 0) return GEO_OK;
    const bool f32 = precision == GEO_PREC_F32_FALLBACK;
    // triangles per wave: 64, fewer where that would leave the chip idle (below
    // 4,096 waves; 112k triangles: 86 us, 136 with 2,048 waves, 0.16 ms with 64
    // each), but 4 at least (1,792 triangles: 22 us, 29 with 2)
    const int64_t per = (m.nt + 4095) / 4096;
    const int tpw = per < 4 ? 4 : (per > 64 ? 64 : (int)per);
    // grid caps: float32 form 16,384 (0.42 ms on 7.2M triangles over levels
    // 0..4; 0.43 at 8,192, 0.50 at 32,768), float64 form 8,192 (0.19 ms on 1M
    // triangles over levels 0..3, 0.22 at 2,048)
    const unsigned g = grid_for(m.nt, tpw, f32 ? 16384 : 8192);
    kt_record(GEO_KT_ROWS, s, false);
    auto pass = f32 ? k_rows_levels_f32 : k_rows_levels_f64;
    pass<<<g, 64, 0, s>>>(m, d, rl, tpw, w);
    auto pieces = f32 ? k_rows_pieces<float> : k_rows_pieces<double>;
    pieces<<<2048, 64, 0, s>>>(m, d, rl, w);
    kt_record(GEO_KT_ROWS, s, true);
    GEO_LAUNCH_CHECK();
    return GEO_OK;
}

int launch_bins_zero(const BinWork& w, int64_t nkeys, hipStream_t s) {
    k_bins_zero<<<grid_for(nkeys, 256, 16384), 256, 0, s>>>(w, nkeys);
    GEO_LAUNCH_CHECK();
    return GEO_OK;
}

int launch_rows_levels_scatter(const RowLevels& rl, const BinWork& w, uint64_t* d_stats, hipStream_t s) {
    if (w.cap <= 0 && !w.slots) return GEO_OK;
    k_rows_levels_scatter<<<grid_for(w.cap, 256, 8192), 256, 0, s>>>(w, rl, d_stats);
    GEO_LAUNCH_CHECK();
    return GEO_OK;
}

int launch_links_pass1(const DevMesh& m, const DevLevel& d, const BinWork& w, hipStream_t s) {
    if (m.nt == 0) return GEO_OK;
    // triangles per wave, as in the ROWS pass; but half as many waves where the
    // blocks are few, so that a triangle has few candidates and the waves'
    // reservations would take most of the time (the call with 20k triangles of 8
    // spheres over 40k blocks 52 us with 4,096 waves, 34 with half; 112k of a star
    // over 1.48M blocks 94 and 118 us)
    const int64_t waves = d.nblocks < 4 * (int64_t)m.nt ? 2048 : 4096;
    const int64_t per = (m.nt + waves - 1) / waves;
    const int tpw = per < 4 ? 4 : (per > 64 ? 64 : (int)per);
    const bool f32 = m.vdtype == GEO_F32;
    kt_record(GEO_KT_LINKS_BINS, s, false);
    auto pass = f32 ? k_links_pass1<float> : k_links_pass1<double>;
    // (7.2M triangles: 0.64 ms; 0.68 with at most 8,192 workgroups)
    pass<<<grid_for(m.nt, tpw, 16384), 64, 0, s>>>(m, d, tpw, w);
    auto pieces = f32 ? k_links_pieces<float> : k_links_pieces<double>;
    pieces<<<2048, 64, 0, s>>>(m, d, w);
    kt_record(GEO_KT_LINKS_BINS, s, true);
    GEO_LAUNCH_CHECK();
    return GEO_OK;
}

int launch_bins_scatter(const BinWork& w, const int32_t* off, int32_t* val, hipStream_t s) {
    if (w.cap <= 0) return GEO_OK;
    k_bins_scatter<<<grid_for(w.cap, 256, 8192), 256, 0, s>>>(w, off, val);
    GEO_LAUNCH_CHECK();
    return GEO_OK;
}

int launch_check_mesh(const DevMesh& m, const DevLevel& d, uint64_t* d_stats, hipStream_t s) {
    if (!d_stats || m.nv == 0) return GEO_OK;
    k_check_mesh<<<grid_for(m.nv, 256, 4096), 256, 0, s>>>(m, d, d_stats);
    GEO_LAUNCH_CHECK();
    return GEO_OK;
}
