// Backward of the cut-link lengths q with respect to the mesh vertices.
//
// q = n.(a - x) / (n.d) for the hit triangle (a, b, c), n = (b-a) x (c-a),
// d = h c_k.  Moving vertex v_j by dv moves the surface at the hit point by
// lambda_j dv (barycentric coordinate of the hit point), and the hit slides
// along d until n.(dq d) = n.(lambda_j dv), so dq/dv_j = lambda_j n / (n.d).
// One thread per link; float64 arithmetic.  For a fixed triangle n is fixed, so
// a link only adds three numbers g lambda_j / (n.d) to its triangle, in an LDS
// table; the triangles of a run of links (neighbours in the table come from
// neighbouring cells and hit the same few) then add n times their sums to
// their vertices, in the same table, and each distinct vertex of the run takes
// one float32 atomic add per component in HBM.  The sums in LDS are float64
// (its float32 atomics are slower).  What bounds it: latency, of the vertex
// gathers and the LDS atomics, so the table is small (14 KB), and the atomics
// in HBM (19 per ns), so it is kept over a run of up to BW_RUN links.  Before (nine
// sums per link, by segmented prefix sums over the wave and an LDS table of
// vertices per 256 links) and now: 543 and 244 us for 14.5M links on a
// 448k-triangle star, 2.66 and 1.28 ms for 58M on the 7.2M star.  Measured on the
// first beside this form at 300 us (its gathers by single words): two tables in
// 28 KB 360 us, two replicas of the sums 435, runs of 1,024 330, 4,096 315.
#include "geo_internal.h"

namespace {

constexpr int BW_THREADS = 256;
constexpr int BW_SLOTS = 512;
constexpr int BW_RUN = 2048;           // links per workgroup, at most
// with fewer than BW_FINE links per triangle of the mesh the triangles of a run
// fill the table after a round or two, so a longer run merges nothing more: runs
// of two rounds
constexpr int BW_FINE = 8, BW_RUN_FINE = 2 * BW_THREADS;
// from BW_DENSE links per triangle on all workgroups add to few vertices, whose
// atomics in HBM serialise: half as many workgroups (0.79M links on 300
// triangles: 35 us, 49 with 2,048)
constexpr int BW_DENSE = 64;
// places that a vertex is looked for in the table (4, 8, 16, 48: 179, 178, 181
// and 211 us for 0.85M links on 2M triangles; 69, 68, 68 and 117 on 448k)
constexpr int BW_PROBES = 8;

__device__ __forceinline__ unsigned bw_hash(int v) { return ((unsigned)v * 2654435761u) >> 23; }

struct BwTable {
    int key[BW_SLOTS];
    double sum[3][BW_SLOTS];
    int count;  // distinct keys
    __device__ __forceinline__ int taken() const {
        return __hip_atomic_load(&count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ __forceinline__ void clear() {
        for (int i = threadIdx.x; i < BW_SLOTS; i += BW_THREADS) {
            key[i] = -1;
            sum[0][i] = sum[1][i] = sum[2][i] = 0.0;
        }
        if (threadIdx.x == 0) count = 0;
    }
    // slot of key v, taken if need be (the callers leave one free)
    __device__ __forceinline__ int slot(int v) {
        unsigned s = bw_hash(v);
        while (true) {
            // most keys are there already: a plain read, which lanes share
            int prev = __hip_atomic_load(&key[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (prev == -1) {
                prev = atomicCAS(&key[s], -1, v);
                if (prev == -1) {
                    atomicAdd(&count, 1);
                    return (int)s;
                }
            }
            if (prev == v) return (int)s;
            s = (s + 1) & (BW_SLOTS - 1);
        }
    }
    // the same, or -1 when the first BW_PROBES slots from its place on are all
    // others' (a table so filled does not keep a count)
    __device__ __forceinline__ int near_slot(int v) {
        unsigned s = bw_hash(v);
        for (int k = 0; k < BW_PROBES; k++) {
            int prev = __hip_atomic_load(&key[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (prev == -1) prev = atomicCAS(&key[s], -1, v);
            if (prev == -1 || prev == v) return (int)s;
            s = (s + 1) & (BW_SLOTS - 1);
        }
        return -1;
    }
    __device__ __forceinline__ void add(int s, double x, double y, double z) {
        atomicAdd(&sum[0][s], x);
        atomicAdd(&sum[1][s], y);
        atomicAdd(&sum[2][s], z);
    }
};

struct BwTri {
    int v[3];
    double P[3][3], n[3];
    // (without contraction: n is exactly zero where two vertices coincide)
    __device__ __forceinline__ void load(const DevMesh& m, int tri) {
#pragma clang fp contract(off)
        load_tri(m, tri, v);
        for (int j = 0; j < 3; j++) load_vert(m, v[j], P[j]);
        const double e1[3] = {P[1][0] - P[0][0], P[1][1] - P[0][1], P[1][2] - P[0][2]};
        const double e2[3] = {P[2][0] - P[0][0], P[2][1] - P[0][1], P[2][2] - P[0][2]};
        n[0] = e1[1] * e2[2] - e1[2] * e2[1];
        n[1] = e1[2] * e2[0] - e1[0] * e2[2];
        n[2] = e1[0] * e2[1] - e1[1] * e2[0];
    }
};

// (8 waves per SIMD: 64 VGPRs; with the compiler's own 68 and 7 waves 3% slower)
__global__ void __launch_bounds__(BW_THREADS) __attribute__((amdgpu_waves_per_eu(8, 8))) k_backward(DevMesh m, DevLevel d, int64_t n_links, int run,
                                                         const int32_t* link_cell, const uint8_t* link_dir,
                                                         const int32_t* link_tri, const float* grad_q, float* grad) {
    __shared__ BwTable T;
    T.clear();
    __syncthreads();
    const double h = ldexp(1.0, -d.level);
    const int64_t i0 = (int64_t)blockIdx.x * run;
    const int64_t i1 = i0 + run < n_links ? i0 + run : n_links;
    for (int64_t base = i0; base < i1; base += BW_THREADS) {  // uniform
        const int64_t i = base + threadIdx.x;
        if (i < i1) {
            const int tri = link_tri[i];
            const float g = grad_q[i];
            const int cell = link_cell[i];
            const int64_t b = cell >> 6;
            if (tri >= 0 && tri < m.nt && g != 0.0f && b < d.nblocks) {
                const int t = cell & 63;
                const int k = link_dir[i];
                const double X[3] = {(4 * d.bcoord[3 * b] + (t & 3) + 0.5) * h,
                                     (4 * d.bcoord[3 * b + 1] + ((t >> 2) & 3) + 0.5) * h,
                                     (4 * d.bcoord[3 * b + 2] + (t >> 4) + 0.5) * h};
                const double dv[3] = {(k % 3 - 1) * h, ((k / 3) % 3 - 1) * h, (k / 9 - 1) * h};
                BwTri A;
                A.load(m, tri);
                const double(&P)[3][3] = A.P;
                const double(&n)[3] = A.n;
                const double nd = n[0] * dv[0] + n[1] * dv[1] + n[2] * dv[2];
                const double nn = n[0] * n[0] + n[1] * n[1] + n[2] * n[2];
                if (nd != 0.0 && nn != 0.0) {
                    const double q = (n[0] * (P[0][0] - X[0]) + n[1] * (P[0][1] - X[1]) + n[2] * (P[0][2] - X[2])) / nd;
                    const double H[3] = {X[0] + q * dv[0], X[1] + q * dv[1], X[2] + q * dv[2]};
                    const double r = (double)g / (nn * nd);
                    double f[3];
                    for (int j = 0; j < 3; j++) {
                        const double* u = P[(j + 1) % 3];
                        const double* w = P[(j + 2) % 3];
                        const double uu[3] = {u[0] - H[0], u[1] - H[1], u[2] - H[2]};
                        const double ww[3] = {w[0] - H[0], w[1] - H[1], w[2] - H[2]};
                        const double cr[3] = {uu[1] * ww[2] - uu[2] * ww[1], uu[2] * ww[0] - uu[0] * ww[2],
                                              uu[0] * ww[1] - uu[1] * ww[0]};
                        f[j] = (n[0] * cr[0] + n[1] * cr[1] + n[2] * cr[2]) * r;  // g lambda_j / (n.d)
                    }
                    T.add(T.slot(tri), f[0], f[1], f[2]);
                }
            }
        }
        __syncthreads();
        // the next round adds up to BW_THREADS triangles: the table is emptied
        // when they might not fit, and at the end of the run (decided on the
        // count that every thread reads before any goes on)
        const int taken = T.taken();
        __syncthreads();
        const bool last = base + BW_THREADS >= i1;
        if (taken + BW_THREADS < BW_SLOTS && !last) continue;  // uniform
        // the triangles go to registers, and the table to their vertices
        constexpr int U = BW_SLOTS / BW_THREADS;
        int tri[U];
        double f[U][3];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int s = threadIdx.x + u * BW_THREADS;
            tri[u] = T.key[s];
            for (int j = 0; j < 3; j++) f[u][j] = T.sum[j][s];
        }
        __syncthreads();
        T.clear();
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; u++) {
            if (tri[u] < 0) continue;
            BwTri A;
            A.load(m, tri[u]);
            for (int j = 0; j < 3; j++) {
                const double g = f[u][j];
                const int sl = T.near_slot(A.v[j]);
                if (sl >= 0) {
                    T.add(sl, g * A.n[0], g * A.n[1], g * A.n[2]);
                } else {  // no place: to memory at once
                    for (int a = 0; a < 3; a++) unsafeAtomicAdd(&grad[3 * (int64_t)A.v[j] + a], (float)(g * A.n[a]));
                }
            }
        }
        __syncthreads();
        for (int s = threadIdx.x; s < BW_SLOTS; s += BW_THREADS) {
            const int v = T.key[s];
            if (v < 0) continue;
            for (int a = 0; a < 3; a++) unsafeAtomicAdd(&grad[3 * (int64_t)v + a], (float)T.sum[a][s]);
        }
        __syncthreads();
        T.clear();
        __syncthreads();
    }
}

}  // namespace

int launch_backward(const DevMesh& m, const DevLevel& d, int64_t n_links, const int32_t* link_cell,
                    const uint8_t* link_dir, const int32_t* link_tri, const float* grad_q, float* grad_verts,
                    hipStream_t s) {
    if (n_links <= 0) return GEO_OK;
    // runs of BW_RUN links, shorter ones where that would leave the chip idle
    // (below 2,048 workgroups, 8 on each CU: 0.85M links on 112k triangles 36 us,
    // 50 with the 1,024 of meshes of few vertices) and on fine meshes (13.4M links on 7.2M triangles: 0.87 ms,
    // 0.90 with BW_RUN, 0.99 with 256)
    const int64_t fill = n_links < BW_DENSE * (int64_t)m.nt ? 2048 : 1024;
    int64_t run = (n_links / fill + BW_THREADS - 1) / BW_THREADS * BW_THREADS;
    const int64_t most = n_links < BW_FINE * (int64_t)m.nt ? BW_RUN_FINE : BW_RUN;
    run = run < BW_THREADS ? BW_THREADS : (run > most ? most : run);
    const int64_t g = (n_links + run - 1) / run;
    k_backward<<<(unsigned)g, BW_THREADS, 0, s>>>(m, d, n_links, (int)run, link_cell, link_dir, link_tri, grad_q, grad_verts);
    GEO_LAUNCH_CHECK();
    return GEO_OK;
}
