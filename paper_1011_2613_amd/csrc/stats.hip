// stats.hip -- suspension-wide diagnostics behind lbm_get_stats: fluid mass
// and momentum over the lattice, the fluid-phase (1 - eps)-weighted share of
// them, particle momentum and the mean hydrodynamic force.  The paper follows
// its suspensions through the area-averaged slip velocity between the phases
// and the mean drag ("Simulation results", Figs. 5 and 7); these sums give
// both.
//
// Every reduction has a fixed shape (a fixed number of workgroups, a fixed
// per-thread order, a fixed tree), so the result does not depend on the GPU
// or on timing.  Partial sums live in the context's workspace.
#include "internal.h"
#include "lb_shared.h"

namespace lbimb {

namespace {

// Stored value v of direction i in binary64 (shifted storage decoded to w_i + g_i).
template <class L, int ST>
__device__ __forceinline__ double stored_pop(int i, typename Store<ST>::T v) {
    if (ST == 0) return (double)v;
    const float wf = (float)L::w[L::wc[i]];
    const float gv = ST == 1 ? (float)v : wf * (float)v;
    return L::w[L::wc[i]] + (double)gv;
}

// Pre-collision population i of node (x, y, z) in binary64: the value the
// previous step's pull streaming leaves for it, A_i(x - c_i), or A_opp(i)(x)
// when x - c_i lies beyond a wall.
template <class L, int ST>
__device__ __forceinline__ double pre_pop(const void *A, const Geom &g, int i, int x, int y, int z) {
    using T = typename Store<ST>::T;
    int sx = x - L::cx[i], sy = y - L::cy[i], sz = z - L::cz[i];
    int j = i;
    if (g.wall_y && (sy < 0 || sy >= g.ny)) {
        sx = x; sy = y; sz = z; j = L::opp[i];
    } else {
        sx = sx < 0 ? sx + g.nx : (sx >= g.nx ? sx - g.nx : sx);
        sy = sy < 0 ? sy + g.ny : (sy >= g.ny ? sy - g.ny : sy);
        sz = sz < 0 ? sz + g.nz : (sz >= g.nz ? sz - g.nz : sz);
    }
    const uint64_t e = (((uint64_t)sz * (uint64_t)g.ny + (uint64_t)sy) * (uint64_t)L::Q + (uint64_t)j) *
                           (uint64_t)g.nx + (uint64_t)sx;
    return stored_pop<L, ST>(j, ((const T *)A)[e]);
}

// rho and j = sum_i c_i f_i of one node, directions in index order.
template <class L, int ST>
__device__ __forceinline__ void node_moments(const void *A, const Geom &g, int x, int y, int z,
                                             double &rho, double j[3]) {
    rho = 0.0;
    j[0] = j[1] = j[2] = 0.0;
#pragma unroll
    for (int i = 0; i < L::Q; i++) {
        const double f = pre_pop<L, ST>(A, g, i, x, y, z);
        rho = rho + f;
        if (L::cx[i]) j[0] = L::cx[i] > 0 ? j[0] + f : j[0] - f;
        if (L::cy[i]) j[1] = L::cy[i] > 0 ? j[1] + f : j[1] - f;
        if (L::cz[i]) j[2] = L::cz[i] > 0 ? j[2] + f : j[2] - f;
    }
}

// Fixed-order tree sum of K values per thread over a 256-thread workgroup;
// thread 0 ends up with the totals in s[0][..].
template <int K>
__device__ __forceinline__ void block_sum(double (*s)[K], const double (&v)[K]) {
    const int t = threadIdx.x;
#pragma unroll
    for (int k = 0; k < K; k++) s[t][k] = v[k];
    __syncthreads();
    for (int h = STATS_NT / 2; h >= 1; h >>= 1) {
        if (t < h)
#pragma unroll
            for (int k = 0; k < K; k++) s[t][k] = s[t][k] + s[t + h][k];
        __syncthreads();
    }
}

// Node pass, one wavefront per lattice row at a time (rows w, w + W, w + 2 W,
// ... of W wavefronts); a lane walks x = l, l + 64, ...  partial[b] = (mass,
// jx, jy, jz) of workgroup b.  The pull streaming only permutes the stored
// populations over the lattice, so their sums are taken in place, each row
// block read once as contiguous lines; a population that streams into a wall
// comes back as its opposite, so its momentum changes sign.  Bound by the
// read: 27.9 M D3Q19 nodes take 713 us in FP64 (5.9 TB/s) and 186 us in FP16
// (gathered node by node, a workgroup per row: 845 and 841 us).
template <class L, int ST>
__global__ __launch_bounds__(STATS_NT) void k_stats_nodes(const void *Av, Geom g, double *partial) {
    using T = typename Store<ST>::T;
    __shared__ double s[STATS_NT][4];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t rows = (int64_t)g.ny * g.nz;
    for (int64_t r = (int64_t)blockIdx.x * (STATS_NT / 64) + wave; r < rows; r += (int64_t)gridDim.x * (STATS_NT / 64)) {
        const int y = (int)(r % g.ny);
        const bool lo = g.wall_y && y == 0, hi = g.wall_y && y == g.ny - 1;
        const T *row = (const T *)Av + (uint64_t)r * (uint64_t)L::Q * (uint64_t)g.nx;
        for (int x = lane; x < g.nx; x += 64) {
            T v[L::Q];
#pragma unroll
            for (int i = 0; i < L::Q; i++) v[i] = row[(uint64_t)i * (uint64_t)g.nx + (uint64_t)x];
            double rho = 0.0, j[3] = {0.0, 0.0, 0.0};
#pragma unroll
            for (int i = 0; i < L::Q; i++) {
                const double f = stored_pop<L, ST>(i, v[i]);
                rho = rho + f;
                const double m = (L::cy[i] < 0 && lo) || (L::cy[i] > 0 && hi) ? -f : f;
                if (L::cx[i]) j[0] = L::cx[i] > 0 ? j[0] + m : j[0] - m;
                if (L::cy[i]) j[1] = L::cy[i] > 0 ? j[1] + m : j[1] - m;
                if (L::cz[i]) j[2] = L::cz[i] > 0 ? j[2] + m : j[2] - m;
            }
            acc[0] = acc[0] + rho;
            acc[1] = acc[1] + j[0];
            acc[2] = acc[2] + j[1];
            acc[3] = acc[3] + j[2];
        }
    }
    block_sum<4>(s, acc);
    if (threadIdx.x == 0)
        for (int k = 0; k < 4; k++) partial[(int64_t)blockIdx.x * 4 + k] = s[0][k];
}

__device__ __forceinline__ int wrap_list(const Geom &g, int axis, int c) {
    const int n = axis == 0 ? g.nx : (axis == 1 ? g.ny : g.nz);
    return c < 0 ? c + n : (c >= n ? c - n : c);
}

// Particle pass, NT threads per particle: its momentum, velocity and
// hydrodynamic force, and over the nodes of its last footprint the share
// s_pn eps_n of the node's mass and momentum (s_pn = count_pn / count_n, so
// the shares of a node's owners add up to eps_n).  The footprint's nodes are
// gathered population by population, so the pass is bound by the latency of
// these reads: the list is spread over a wavefront, or over a workgroup where
// there are too few particles to fill the GPU that way.  out holds one column
// of np values per quantity.  Measured against one thread per particle: 8 317
// spheres R = 4 343 against 4 401 us (FP64), 310 spheres R = 5.3 24 against
// 5 884 us, 21 361 discs R = 5 93 against 531 us.
template <class L, int ST, int NT>
__global__ __launch_bounds__(NT) void k_stats_particles(const void *A, Geom g, Particles P, const void *qr,
                                                        int rec32, int Smax, double *out) {
    const int p = blockIdx.x;
    const int np = P.np;
    double w5[5] = {0.0, 0.0, 0.0, 0.0, 0.0};  // rho, j and eps shares
    const int lo0 = P.bb[p], lo1 = P.bb[np + p], lo2 = P.bb[2 * np + p];
    const int seg = P.nseg > 1 ? list_seg(P, p) : 0;
    // thread t takes the list's entries t, t + NT, ... whatever the segments
    int before = 0;
    for (int sg = 0; sg < P.nseg; sg++) {
        const uint32_t *list = P.list + (int64_t)p * P.list_cap + sg * seg;
        const int len = P.list_len[(int64_t)p * P.nseg + sg];
        for (int e = ((int)threadIdx.x - before) & (NT - 1); e < len; e += NT) {
            const uint32_t v = list[e];
            const int x = wrap_list(g, 0, lo0 + (int)((v >> 10) & 127u));
            const int y = g.wall_y ? lo1 + (int)((v >> 17) & 127u) : wrap_list(g, 1, lo1 + (int)((v >> 17) & 127u));
            const int z = L::D == 3 ? wrap_list(g, 2, lo2 + (int)((v >> 24) & 127u)) : 0;
            const int64_t n = (int64_t)x + (int64_t)g.nx * ((int64_t)y + (int64_t)g.ny * z);
            double q[3];
            int tot;
            read_qrec(qr, rec32 != 0, n, q, tot);
            const int cnt = (int)(v & 1023u);
            const double eps = (double)(tot < Smax ? tot : Smax) / (double)Smax;
            const double w = ((double)cnt / (double)tot) * eps;
            double rho, j[3];
            node_moments<L, ST>(A, g, x, y, z, rho, j);
            w5[0] = w5[0] + w * rho;
            for (int d = 0; d < 3; d++) w5[1 + d] = w5[1 + d] + w * j[d];
            w5[4] = w5[4] + w;
        }
        before += len;
    }
    __shared__ double s[NT / 64][5];
#pragma unroll
    for (int k = 0; k < 5; k++) {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) w5[k] = w5[k] + __shfl_xor(w5[k], d, 64);
        if (NT > 64 && (threadIdx.x & 63) == 0) s[threadIdx.x >> 6][k] = w5[k];
    }
    if (NT > 64) {
        __syncthreads();
        if (threadIdx.x < 5)
            for (int k = 1; k < NT / 64; k++) s[0][threadIdx.x] = s[0][threadIdx.x] + s[k][threadIdx.x];
        __syncthreads();
        for (int k = 0; k < 5; k++) w5[k] = s[0][k];
    }
    if (threadIdx.x >= STATS_PK) return;
    const int k = threadIdx.x, d = k % 3;
    const double m = P.m[p];
    double r = m;
    if (k < 9) r = k < 3 ? m * P.v[d * np + p] : (k < 6 ? P.v[d * np + p] : P.Fh[d * np + p]);
#pragma unroll
    for (int q = 0; q < 5; q++)
        if (k == 9 + q) r = w5[q];
    out[(int64_t)k * np + p] = r;
}

// Final pass, one workgroup per total: the node partials of quantity 0..3, or
// the particle column of quantity 4...
constexpr int STATS_FT = 1024;

__global__ __launch_bounds__(STATS_FT) void k_stats_final(const double *node_part, int groups, const double *cols,
                                                          int np, double *tot) {
    __shared__ double s[STATS_FT / 64];
    const int k = blockIdx.x;
    double v = 0.0;
    if (k < 4) {
        for (int b = threadIdx.x; b < groups; b += STATS_FT) v = v + node_part[(int64_t)b * 4 + k];
    } else {
        for (int p = threadIdx.x; p < np; p += STATS_FT) v = v + cols[(int64_t)(k - 4) * np + p];
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v = v + __shfl_xor(v, d, 64);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < STATS_FT / 64; w++) v = v + s[w];
        tot[k] = v;
    }
}

// A wavefront per particle keeps the GPU's 1 024 SIMDs busy from about this
// many particles on; below, a workgroup per particle.
constexpr int STATS_WAVE_MIN = 1024;

template <class L, int ST>
hipError_t stats_dispatch(const StatsArgs &a, hipStream_t s) {
    hipLaunchKernelGGL((k_stats_nodes<L, ST>), dim3(STATS_NODE_GROUPS), dim3(STATS_NT), 0, s, a.A, a.g,
                       a.node_part);
    if (a.P.np >= STATS_WAVE_MIN)
        hipLaunchKernelGGL((k_stats_particles<L, ST, 64>), dim3(a.P.np), dim3(64), 0, s, a.A, a.g, a.P, a.qr,
                           a.rec32, a.Smax, a.part_cols);
    else if (a.P.np > 0)
        hipLaunchKernelGGL((k_stats_particles<L, ST, 512>), dim3(a.P.np), dim3(512), 0, s, a.A, a.g, a.P, a.qr,
                           a.rec32, a.Smax, a.part_cols);
    hipLaunchKernelGGL(k_stats_final, dim3(4 + STATS_PK), dim3(STATS_FT), 0, s, (const double *)a.node_part,
                       STATS_NODE_GROUPS, (const double *)a.part_cols, a.P.np, a.tot);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_stats(int lattice, int storage, const StatsArgs &a, hipStream_t s) {
    if (lattice == 0) {
        if (storage == 0) return stats_dispatch<D2Q9, 0>(a, s);
        if (storage == 1) return stats_dispatch<D2Q9, 1>(a, s);
        return stats_dispatch<D2Q9, 2>(a, s);
    }
    if (storage == 0) return stats_dispatch<D3Q19, 0>(a, s);
    if (storage == 1) return stats_dispatch<D3Q19, 1>(a, s);
    return stats_dispatch<D3Q19, 2>(a, s);
}

}  // namespace lbimb
