// particle_kernels.hip -- particle side of the LB-IMB-DEM step on gfx950:
// footprint / solid fraction, hydrodynamic force and torque sums (Eq. 3),
// DEM cell list, contact forces (Eqs. 4-5) and time integration.
//
// All particle arithmetic is binary64 in every storage mode.  Sums whose
// order differs from a sequential loop (the per-particle force reduction) use
// error-free TwoSum accumulation (Ogita, Rump & Oishi 2005) so the rounded
// result does not depend on the reduction tree.
#include <algorithm>

#include "internal.h"

namespace lbimb {

__device__ __forceinline__ double pdisp(double d, double L) {
    if (d > 0.5 * L) d = d - L;
    else if (d < -0.5 * L) d = d + L;
    return d;
}

__device__ __forceinline__ double ndisp(const Geom &g, int axis, int coord, double xp) {
    double d = (double)coord - xp;
    if (axis == 0) return pdisp(d, g.Lx);
    if (axis == 1) return g.wall_y ? d : pdisp(d, g.Ly);
    return pdisp(d, g.Lz);
}

// Wrap an unwrapped node coordinate; -1 beyond a wall.
__device__ __forceinline__ int wrapc(const Geom &g, int axis, int c) {
    const int n = axis == 0 ? g.nx : (axis == 1 ? g.ny : g.nz);
    if (axis == 1 && g.wall_y) return (c < 0 || c >= n) ? -1 : c;
    c %= n;
    return c < 0 ? c + n : c;
}

// Bounding box of nodes whose cell may hold samples of the particle (box_axis).
__device__ __forceinline__ void bbox(const Particles &P, int p, int D, int lo[3], int hi[3]) {
    const double r = P.R[p];
    for (int a = 0; a < 3; a++) {
        if (a >= D) { lo[a] = hi[a] = 0; continue; }
        box_axis(P.x[a * P.np + p], r, lo[a], hi[a]);
    }
}

// The lattice kernel's record of particle p, one value per thread t < 9.
__device__ __forceinline__ void write_rec(const Particles &P, int p, int t) {
    if (t >= 9) return;
    const double *src = t < 3 ? P.x : (t < 6 ? P.v : P.w);
    const double val = src[(t % 3) * P.np + p];
    PRec &r = P.rec[p];
    if (t < 3) {
        r.x[t] = val;
    } else {
        (t < 6 ? r.vf : r.wf)[t % 3] = (float)val;
        (t < 6 ? r.v : r.w)[t % 3] = val;
    }
}

// Number of sub-cell samples of a node inside a particle: offsets
// (k + 1/2)/S - 1/2 per axis from the node, inside test dx^2 + dy^2 (+ dz^2)
// <= R^2 evaluated left to right, d0/d1/d2 the node-minus-centre displacement.
// The squared offsets are separable, so a node needs S^D additions.  (Called
// only for nodes the distance bounds left undecided, so no shortcut for
// all-inside or all-outside nodes is taken here.)
template <int D, int S>
__device__ __forceinline__ int sample_count(double d0, double d1, double d2, double R2) {
    double sx[S], sz[S];
#pragma unroll
    for (int s = 0; s < S; s++) {
        const double off = ((double)s + 0.5) / (double)S - 0.5;
        const double ex = d0 + off;
        sx[s] = ex * ex;
        const double ez = d2 + off;
        sz[s] = D == 3 ? ez * ez : 0.0;
    }
    int count = 0;
    // one row of samples (fixed y offset) per iteration, kept rolled so
    // that only that row's partial sums are live
#pragma unroll 1
    for (int ky = 0; ky < S; ky++) {
        const double ey = d1 + (((double)ky + 0.5) / (double)S - 0.5);
        const double sy = ey * ey;
#pragma unroll
        for (int kx = 0; kx < S; kx++) {
            const double t = sx[kx] + sy;
            if (D == 2) {
                count += (t <= R2) ? 1 : 0;
            } else {
#pragma unroll
                for (int kz = 0; kz < S; kz++) count += (t + sz[kz] <= R2) ? 1 : 0;
            }
        }
    }
    return count;
}

// Unwrapped coordinate -> lattice coordinate.  A bounding box is narrower than
// the periodic box, so one conditional shift suffices; -1 beyond a wall.
__device__ __forceinline__ int wrap1(const Geom &g, int axis, int c) {
    const int n = axis == 0 ? g.nx : (axis == 1 ? g.ny : g.nz);
    if (axis == 1 && g.wall_y) return (c < 0 || c >= n) ? -1 : c;
    return c < 0 ? c + n : (c >= n ? c - n : c);
}

constexpr uint32_t LIST_COUNT_MASK = 1023u;

// floor(v / d) for 0 <= v < 2^24 and 1 <= d < 2^12: binary32 estimate from the
// reciprocal, then one exact integer correction step.
__device__ __forceinline__ int div_small(int v, int d, float inv_d) {
    int q = (int)((float)v * inv_d);
    const int r = v - q * d;
    if (r < 0) q -= 1;
    else if (r >= d) q += 1;
    return q;
}

__device__ __forceinline__ uint32_t list_entry(int count, int kx, int ky, int kz) {
    return (uint32_t)count | ((uint32_t)kx << 10) | ((uint32_t)ky << 17) | ((uint32_t)kz << 24);
}

// Exclusive prefix sum over the threads of a workgroup (<= 256 threads);
// `total` receives the sum.  Every thread of the workgroup must call it.
__device__ __forceinline__ int block_scan(int v, int &total) {
    __shared__ int wsum[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
    int x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    if (lane == 63 || threadIdx.x == blockDim.x - 1) wsum[wave] = x;
    __syncthreads();
    int before = 0;
    total = 0;
    for (int w = 0; w < nw; w++) {
        if (w < wave) before += wsum[w];
        total += wsum[w];
    }
    __syncthreads();
    return before + x - v;
}

// Conservative classification of a node from per-axis distance bounds: 0 when
// every sub-cell sample is certainly outside, S^D when every sample is
// certainly inside, -1 otherwise.  With h = 1/2 - 1/(2S) the largest sample
// offset, the sum of squares of every sample lies in [lo, hi] built from
// max(|d| - h, 0) and |d| + h; rounding moves the tested sums and the bounds
// by a few units in the last place, far inside the 1e-14 relative margins,
// so a decided node gets exactly the count the per-sample test gives.
template <int D, int S>
__device__ __forceinline__ int classify(double d0, double d1, double d2, double R2) {
    const double h = 0.5 - 0.5 / (double)S;
    const double a0 = fabs(d0), a1 = fabs(d1), a2 = fabs(d2);
    const double m0 = fmax(a0 - h, 0.0), m1 = fmax(a1 - h, 0.0), m2 = fmax(a2 - h, 0.0);
    const double M0 = a0 + h, M1 = a1 + h, M2 = a2 + h;
    double lo = m0 * m0 + m1 * m1, hi = M0 * M0 + M1 * M1;
    if (D == 3) {
        lo = lo + m2 * m2;
        hi = hi + M2 * M2;
    }
    if (lo * (1.0 - 1e-14) > R2) return 0;
    if (hi * (1.0 + 1e-14) <= R2) return D == 3 ? S * S * S : S * S;
    return -1;
}

// Table-lookup eps (Eq. 6): the count of a node at displacement (d0, d1, d2)
// from the centre, from rho = |r| - R and the folded direction of r (sorted
// magnitudes a >= b >= c, t1 = b/|r|, t2 = c/|r|); wholly inside for
// rho <= -H, outside for rho >= H (H = sqrt(D)/2, half a cell diagonal).
template <int D, int SMAX>
__device__ __forceinline__ int eps_lookup(const FootArgs &a, double d0, double d1, double d2, double R) {
    double r2 = d0 * d0 + d1 * d1;
    if (D == 3) r2 = r2 + d2 * d2;
    // wholly inside or outside by a relative margin of 1e-12 on |r|^2 (far
    // above the rounding of sqrt(|r|^2) - R): the same decision as below
    // without the square root
    const double ri = R - a.tabH, ro = R + a.tabH;
    if (r2 < ri * ri * (1.0 - 1e-12)) return SMAX;
    if (r2 > ro * ro * (1.0 + 1e-12)) return 0;
    const double r = sqrt(r2);
    const double rho = r - R;
    if (rho <= -a.tabH) return SMAX;
    if (rho >= a.tabH) return 0;
    int ir = (int)floor((rho + a.tabH) / a.tabW);
    ir = ir < 0 ? 0 : (ir > EPS_TAB_NRHO - 1 ? EPS_TAB_NRHO - 1 : ir);
    double x = fabs(d0), y = fabs(d1), z = D == 3 ? fabs(d2) : 0.0, t;
    if (y > x) { t = x; x = y; y = t; }
    if (z > y) { t = y; y = z; z = t; }
    if (y > x) { t = x; x = y; y = t; }
    int i1 = (int)floor(y / r * a.tabK1);
    i1 = i1 > EPS_TAB_NT - 1 ? EPS_TAB_NT - 1 : i1;
    if (D == 2) return a.tab[ir * EPS_TAB_NT + i1];
    int i2 = (int)floor(z / r * a.tabK2);
    i2 = i2 > EPS_TAB_NT - 1 ? EPS_TAB_NT - 1 : i2;
    return a.tab[(ir * EPS_TAB_NT + i1) * EPS_TAB_NT + i2];
}

// Footprint of one particle, one workgroup.  The bounding box is taken in
// chunks of nodes: (A) every node is classified by distance bounds, undecided
// nodes are queued in LDS; (B) the queued nodes get the exact per-sample count,
// the workgroup's lanes all busy with such nodes; (C1) a workgroup prefix sum
// lists the covered nodes of the chunk in node order (x fastest); (C2) the
// k-th covered node takes place k of the particle's list and an owner slot, so
// the list is the same on every run.
template <int D, int S, int NT, bool TAB>
__device__ __forceinline__ void foot_one(const FootArgs &a, int p) {
    constexpr int CHUNK = 1024;
    __shared__ uint16_t s_cnt[CHUNK];
    __shared__ uint16_t s_todo[CHUNK];
    __shared__ int s_ntodo;
    const int P = a.P.np;
    int lo[3], hi[3];
    bbox(a.P, p, D, lo, hi);
    write_rec(a.P, p, (int)threadIdx.x);
    if (threadIdx.x == 0)
        for (int d = 0; d < 3; d++) {
            a.P.bb[d * P + p] = lo[d];
            a.P.bb[(3 + d) * P + p] = hi[d];
        }
    // A centre must lie in the box on periodic axes (integration keeps it
    // there unless a particle moves a box length in one step) and be finite:
    // otherwise the bounding box cannot be wrapped and the particle gets an
    // empty footprint and an error flag.
    bool placed = true;
    for (int d = 0; d < D; d++) {
        const double c = a.P.x[d * P + p];
        const double L = d == 0 ? a.g.Lx : (d == 1 ? a.g.Ly : a.g.Lz);
        placed = placed && ((d == 1 && a.g.wall_y) ? (c > -L && c < 2.0 * L) : (c >= 0.0 && c < L));
    }
    if (!placed && threadIdx.x == 0) atomicOr(a.flags, FLAG_NONFINITE);
    const int ext0 = hi[0] - lo[0] + 1, ext1 = hi[1] - lo[1] + 1;
    const int ext2 = D == 3 ? hi[2] - lo[2] + 1 : 1;
    const int items = placed ? ext0 * ext1 * ext2 : 0;
    const double r = a.P.R[p];
    const double R2 = r * r;
    const double xp0 = a.P.x[p], xp1 = a.P.x[P + p], xp2 = D == 3 ? a.P.x[2 * P + p] : 0.0;
    const int64_t N = a.g.N;
    const int cap = a.P.list_cap;
    uint32_t *list = a.P.list + (int64_t)p * cap;
    const float inv0 = 1.0f / (float)ext0, inv1 = 1.0f / (float)ext1;
    // node of a bounding-box item: lattice coordinates (iy < 0 beyond a wall)
    auto node_of = [&](int item, int &kx, int &ky, int &kz, int &ix, int &iy, int &iz) {
        const int rest = div_small(item, ext0, inv0);
        kx = item - rest * ext0;
        kz = div_small(rest, ext1, inv1);
        ky = rest - kz * ext1;
        iy = wrap1(a.g, 1, lo[1] + ky);
        ix = wrap1(a.g, 0, lo[0] + kx);
        iz = D == 3 ? wrap1(a.g, 2, lo[2] + kz) : 0;
    };
    int base = 0;
    for (int c0 = 0; c0 < items; c0 += CHUNK) {
        const int nc = items - c0 < CHUNK ? items - c0 : CHUNK;
        if (threadIdx.x == 0) s_ntodo = 0;
        __syncthreads();
        // (A) classify
#pragma unroll 1
        for (int i = threadIdx.x; i < nc; i += NT) {
            int kx, ky, kz, ix, iy, iz;
            node_of(c0 + i, kx, ky, kz, ix, iy, iz);
            int cls = 0;
            if (iy >= 0) {
                const double d0 = ndisp(a.g, 0, ix, xp0), d1 = ndisp(a.g, 1, iy, xp1);
                const double d2 = D == 3 ? ndisp(a.g, 2, iz, xp2) : 0.0;
                if (TAB) cls = eps_lookup<D, D == 3 ? S * S * S : S * S>(a, d0, d1, d2, r);
                else cls = classify<D, S>(d0, d1, d2, R2);
            }
            if (cls < 0) s_todo[atomicAdd(&s_ntodo, 1)] = (uint16_t)i;
            else s_cnt[i] = (uint16_t)cls;
        }
        __syncthreads();
        // (B) exact per-sample counts of the undecided nodes
        const int ntodo = s_ntodo;
#pragma unroll 1
        for (int j = threadIdx.x; j < ntodo; j += NT) {
            const int i = s_todo[j];
            int kx, ky, kz, ix, iy, iz;
            node_of(c0 + i, kx, ky, kz, ix, iy, iz);
            s_cnt[i] = (uint16_t)sample_count<D, S>(ndisp(a.g, 0, ix, xp0), ndisp(a.g, 1, iy, xp1),
                                                    D == 3 ? ndisp(a.g, 2, iz, xp2) : 0.0, R2);
        }
        __syncthreads();
        // (C1) the covered nodes of the chunk in node order into s_todo (the
        // queue of (B) is spent): each thread takes ceil(nc / NT) consecutive
        // nodes of the chunk (a disc's box fills a seventh of a chunk), one
        // workgroup prefix sum places them
        {
            const int per = (nc + NT - 1) / NT;
            const int j0 = min((int)threadIdx.x * per, nc), j1 = min(j0 + per, nc);
            int m = 0;
            for (int j = j0; j < j1; j++) m += s_cnt[j] > 0 ? 1 : 0;
            int ncov;
            int at = block_scan(m, ncov);
            for (int j = j0; j < j1; j++)
                if (s_cnt[j] > 0) s_todo[at++] = (uint16_t)j;
            __syncthreads();
            // (C2) owner slots and list entries, k-th covered node in lane
            // order.  Covered nodes that fall in one aligned 8-byte word of the
            // owner counts sit in consecutive lanes; the first lane of such a
            // run claims all of them with one 64-bit atomic add and every lane
            // of the run reads its own byte of the returned word, which is what
            // one atomic add per node in lane order would have returned.
            const int lane = threadIdx.x & 63;
#pragma unroll 1
            for (int k0 = 0; k0 < ncov; k0 += NT) {
                const int k = k0 + (int)threadIdx.x;
                int count = 0, kx = 0, ky = 0, kz = 0;
                int64_t n = 0;
                long long key = -1;  // owner-count word of a covered node
                if (k < ncov) {
                    const int i = s_todo[k];
                    count = s_cnt[i];
                    int ix, iy, iz;
                    node_of(c0 + i, kx, ky, kz, ix, iy, iz);
                    n = (int64_t)ix + (int64_t)a.g.nx * ((int64_t)iy + (int64_t)a.g.ny * iz);
                    key = (long long)(n >> 3);
                }
                const int byte = (int)(n & 7);
                uint32_t mask = key >= 0 ? 1u << byte : 0u;
                int back = 0;  // lanes between this one and the first of its run
                bool run = true;
#pragma unroll
                for (int j = 1; j < 8; j++) {
                    const long long kj = __shfl_up(key, j, 64);
                    run = run && lane >= j && kj == key;
                    back += run ? 1 : 0;
                }
                run = true;
#pragma unroll
                for (int j = 1; j < 8; j++) {
                    const long long kj = __shfl_down(key, j, 64);
                    const uint32_t mj = __shfl_down(mask, j, 64);
                    run = run && lane + j < 64 && kj == key;
                    if (run) mask |= mj;
                }
                unsigned long long old = 0ull;
                if (key >= 0 && back == 0) {
                    unsigned long long inc = 0ull;
#pragma unroll
                    for (int q = 0; q < 8; q++)
                        if ((mask >> q) & 1u) inc |= 1ull << (8 * q);
                    old = atomicAdd((unsigned long long *)(a.nown + ((int64_t)key << 3)), inc);
                }
                old = __shfl(old, lane - back, 64);
                if (k < ncov) {
                    const int slot = (int)((old >> (8 * byte)) & 0xffull);
                    if (slot < MAX_OWNERS)
                        a.slots[(int64_t)slot * N + n] = ((uint32_t)p << SLOT_COUNT_BITS) | (uint32_t)count;
                    else
                        atomicOr(a.flags, FLAG_SLOT_OVERFLOW);
                    if (base + k < cap) list[base + k] = list_entry(count, kx, ky, kz);
                }
            }
            base += ncov;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (base > cap) atomicOr(a.flags, FLAG_SLOT_OVERFLOW);
        a.P.list_len[p] = base < cap ? base : cap;
    }
}

// LDS written by some lanes of a wavefront and read by others of the same
// wavefront: order the accesses within it.
__device__ __forceinline__ void lane_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------------------------- cell list
__device__ __forceinline__ int cell_coord(const Geom &g, int nc, int axis, double x) {
    const double L = axis == 0 ? g.Lx : (axis == 1 ? g.Ly : g.Lz);
    double t = x;
    if (axis == 1 && g.wall_y) t = x + 0.5;
    int c = (int)floor(t * (double)nc / L);
    return c < 0 ? 0 : (c >= nc ? nc - 1 : c);
}

__device__ __forceinline__ int cell_coord(const CellArgs &a, int axis, double x) {
    return cell_coord(a.g, axis == 0 ? a.ncx : (axis == 1 ? a.ncy : a.ncz), axis, x);
}

// Files particle p in cell c; beyond the cell's places it is only counted.
// Who reads the cell for contacts or lists reports that (cell_entries): a list
// filed ahead may never be read (the last step of a run, a step that keeps its
// neighbour lists).
__device__ __forceinline__ void file_in_cell(int *cell_count, int *cell_ids, int c, int p) {
    const int slot = atomicAdd(&cell_count[c], 1);
    if (slot < CELL_CAP) cell_ids[c * CELL_CAP + slot] = p;
}

// Particles listed in cell c.  Every particle's search includes its own cell,
// so an overfull one is always seen.
__device__ __forceinline__ int cell_entries(const CellArgs &a, int c) {
    const int n = a.cell_count[c];
    if (n > CELL_CAP) atomicOr(a.flags, FLAG_CELL_OVERFLOW);
    return min(n, CELL_CAP);
}

__global__ void k_cells(CellArgs a) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const int P = a.P.np;
    if (p >= P) return;
    const int cx = cell_coord(a, 0, a.P.x[p]);
    const int cy = cell_coord(a, 1, a.P.x[P + p]);
    const int cz = a.D == 3 ? cell_coord(a, 2, a.P.x[2 * P + p]) : 0;
    file_in_cell(a.cell_count, a.cell_ids, cx + a.ncx * (cy + a.ncy * cz), p);
}

// Neighbour cell offsets along one axis: {-1,0,1} wrapped (periodic, >= 3
// cells), {0,1} (2 cells), {0} (1 cell), or {-1,0,1} clipped at walls.
__device__ __forceinline__ int axis_cells(int c, int nc, bool periodic, int out[3]) {
    if (periodic) {
        if (nc >= 3) { out[0] = c == 0 ? nc - 1 : c - 1; out[1] = c; out[2] = c == nc - 1 ? 0 : c + 1; return 3; }
        if (nc == 2) { out[0] = 0; out[1] = 1; return 2; }
        out[0] = 0;
        return 1;
    }
    int k = 0;
    for (int d = -1; d <= 1; d++)
        if (c + d >= 0 && c + d < nc) out[k++] = c + d;
    return k;
}

// Contact test and force of Eqs. 4-5 for the pair (i, j) with the overlap
// delta = R_i + R_j - |r_i - r_j| (minimum image).  Returns false when the
// particles do not touch.
__device__ __forceinline__ bool pair_force(const CellArgs &a, int i, int j, double F[3]) {
    const int P = a.P.np, D = a.D;
    double d[3] = {0.0, 0.0, 0.0};
    for (int ax = 0; ax < D; ax++) {
        double dd = a.P.x[ax * P + i] - a.P.x[ax * P + j];
        if (!(ax == 1 && a.g.wall_y)) dd = pdisp(dd, ax == 0 ? a.g.Lx : (ax == 1 ? a.g.Ly : a.g.Lz));
        d[ax] = dd;
    }
    double d2 = d[0] * d[0] + d[1] * d[1];
    if (D == 3) d2 = d2 + d[2] * d[2];
    const double dist = sqrt(d2);
    const double delta = (a.P.R[i] + a.P.R[j]) - dist;
    if (!(delta > 0.0)) return false;
    if (F) {
        double nrm[3] = {0.0, 0.0, 0.0};
        for (int ax = 0; ax < D; ax++) nrm[ax] = d[ax] / dist;
        double vn = (a.P.v[i] - a.P.v[j]) * nrm[0] + (a.P.v[P + i] - a.P.v[P + j]) * nrm[1];
        if (D == 3) vn = vn + (a.P.v[2 * P + i] - a.P.v[2 * P + j]) * nrm[2];
        const double meff = a.P.m[i] * a.P.m[j] / (a.P.m[i] + a.P.m[j]);
        const double eta = a.ce * sqrt(meff * a.kn);
        const double fmag = a.kn * delta - eta * vn;
        for (int ax = 0; ax < D; ax++) F[ax] = F[ax] + fmag * nrm[ax];
    }
    return true;
}

// Wall contacts of particle i (Eqs. 4-5 against a wall at rest, m_eff = m_i),
// added to F after the pair forces.
__device__ __forceinline__ void wall_force(const CellArgs &a, int i, double F[3]) {
    if (!a.g.wall_y) return;
    const int P = a.P.np;
    const double eta = a.ce * sqrt(a.P.m[i] * a.kn);
    const double y = a.P.x[P + i];
    const double vy = a.P.v[P + i];
    const double dl = a.P.R[i] - (y + 0.5);
    if (dl > 0.0) {
        const double fmag = a.kn * dl - eta * vy;
        F[1] = F[1] + fmag;
    }
    const double du = a.P.R[i] - ((a.g.Ly - 0.5) - y);
    if (du > 0.0) {
        const double fmag = a.kn * du - eta * (-vy);
        F[1] = F[1] - fmag;
    }
}

// Contacts of particle i by one wavefront: each lane scans one neighbour cell,
// touching neighbours are gathered in LDS (`list`, `nl`: this wavefront's own),
// sorted by id, and the pair forces are added in ascending id (then the walls)
// by the first lane.
__device__ __forceinline__ void dem_wave(const CellArgs &a, int i, int *list, int *nl) {
    const int lane = threadIdx.x & 63;
    const int P = a.P.np;
    const int D = a.D;
    if (lane == 0) *nl = 0;
    lane_sync();
    if (i < P) {
        const int c0 = cell_coord(a, 0, a.P.x[i]);
        const int c1 = cell_coord(a, 1, a.P.x[P + i]);
        const int c2 = D == 3 ? cell_coord(a, 2, a.P.x[2 * P + i]) : 0;
        int ox[3], oy[3], oz[3];
        const int nxc = axis_cells(c0, a.ncx, true, ox);
        const int nyc = axis_cells(c1, a.ncy, !a.g.wall_y, oy);
        int nzc = 1;
        oz[0] = 0;
        if (D == 3) nzc = axis_cells(c2, a.ncz, true, oz);
        if (lane < nxc * nyc * nzc) {
            const int kx = lane % nxc, ky = (lane / nxc) % nyc, kz = lane / (nxc * nyc);
            const int c = ox[kx] + a.ncx * (oy[ky] + a.ncy * oz[kz]);
            const int cnt = cell_entries(a, c);
            for (int s = 0; s < cnt; s++) {
                const int j = a.cell_ids[c * CELL_CAP + s];
                if (j == i) continue;
                if (!pair_force(a, i, j, nullptr)) continue;
                const int slot = atomicAdd(nl, 1);
                if (slot < MAX_CONTACTS) list[slot] = j;
                else atomicOr(a.flags, FLAG_CONTACT_OVERFLOW);
            }
        }
    }
    lane_sync();
    if (i < P && lane == 0) {
        const int n = min(*nl, MAX_CONTACTS);
        for (int s = 1; s < n; s++) {
            const int v = list[s];
            int t = s - 1;
            while (t >= 0 && list[t] > v) {
                list[t + 1] = list[t];
                t--;
            }
            list[t + 1] = v;
        }
        double F[3] = {0.0, 0.0, 0.0};
        for (int s = 0; s < n; s++) pair_force(a, i, list[s], F);
        wall_force(a, i, F);
        for (int d = 0; d < 3; d++) a.P.Fc[d * P + i] = F[d];
    }
}

__global__ __launch_bounds__(256) void k_dem(CellArgs a) {
    __shared__ int list[4][MAX_CONTACTS];
    __shared__ int nlist[4];
    const int wave = threadIdx.x >> 6;
    dem_wave(a, (int)blockIdx.x * 4 + wave, list[wave], &nlist[wave]);
}

// Contacts of particle i by one thread, for many particles (dem_wave keeps a
// wavefront busy with 9 or 27 neighbour cells, most of its lanes idle in 2D): the thread
// walks the neighbour cells itself and inserts each touching neighbour into
// its own id-sorted column of LDS, then adds the pair forces in ascending id
// and the walls, the sum order of k_dem, so both kernels give the same bits.
template <int NT>
__device__ __forceinline__ void dem_thread(const CellArgs &a, int i, int (*list)[NT]) {
    const int t = threadIdx.x;
    const int P = a.P.np;
    const int D = a.D;
    if (i >= P) return;  // no barrier below
    const int c0 = cell_coord(a, 0, a.P.x[i]);
    const int c1 = cell_coord(a, 1, a.P.x[P + i]);
    const int c2 = D == 3 ? cell_coord(a, 2, a.P.x[2 * P + i]) : 0;
    int ox[3], oy[3], oz[3];
    const int nxc = axis_cells(c0, a.ncx, true, ox);
    const int nyc = axis_cells(c1, a.ncy, !a.g.wall_y, oy);
    int nzc = 1;
    oz[0] = 0;
    if (D == 3) nzc = axis_cells(c2, a.ncz, true, oz);
    int nl = 0;
    bool overflow = false;
    for (int kz = 0; kz < nzc; kz++)
        for (int ky = 0; ky < nyc; ky++)
            for (int kx = 0; kx < nxc; kx++) {
                const int c = ox[kx] + a.ncx * (oy[ky] + a.ncy * oz[kz]);
                const int cnt = cell_entries(a, c);
                for (int s = 0; s < cnt; s++) {
                    const int j = a.cell_ids[c * CELL_CAP + s];
                    if (j == i) continue;
                    if (!pair_force(a, i, j, nullptr)) continue;
                    if (nl >= MAX_CONTACTS) {
                        overflow = true;
                        continue;
                    }
                    int q = nl;
                    while (q > 0 && list[q - 1][t] > j) {
                        list[q][t] = list[q - 1][t];
                        q--;
                    }
                    list[q][t] = j;
                    nl++;
                }
            }
    if (overflow) atomicOr(a.flags, FLAG_CONTACT_OVERFLOW);
    double F[3] = {0.0, 0.0, 0.0};
    for (int s = 0; s < nl; s++) pair_force(a, i, list[s][t], F);
    wall_force(a, i, F);
    for (int d = 0; d < 3; d++) a.P.Fc[d * P + i] = F[d];
}

// True when j lies within R_i + R_j + skin of i (minimum image).
__device__ __forceinline__ bool nl_candidate(const CellArgs &a, int i, int j) {
    const int P = a.P.np;
    double d2 = 0.0;
    for (int ax = 0; ax < a.D; ax++) {
        double dd = a.P.x[ax * P + i] - a.P.x[ax * P + j];
        if (!(ax == 1 && a.g.wall_y)) dd = pdisp(dd, ax == 0 ? a.g.Lx : (ax == 1 ? a.g.Ly : a.g.Lz));
        d2 = d2 + dd * dd;
    }
    const double lim = (a.P.R[i] + a.P.R[j]) + a.skin;
    return d2 < lim * lim;
}

// Contacts of particle i from its neighbour list by one wavefront, a lane per
// listed neighbour; on a rebuild step the list is made first, from the cells
// (edge >= 2 R_max + skin), and the build positions are recorded.  The touching
// neighbours are summed in ascending id, as in dem_wave.  Cells, flag and lists
// of other particles are not written here, so every wavefront decides alone.
__device__ __forceinline__ void dem_list_wave(const CellArgs &a, int i, int *list, int *nl) {
    const int lane = threadIdx.x & 63;
    const int P = a.P.np;
    const int D = a.D;
    int n = 0, j = -1;
    if (*a.nl_flag) {
        if (lane == 0) *nl = 0;
        lane_sync();
        const int c0 = cell_coord(a, 0, a.P.x[i]);
        const int c1 = cell_coord(a, 1, a.P.x[P + i]);
        const int c2 = D == 3 ? cell_coord(a, 2, a.P.x[2 * P + i]) : 0;
        int ox[3], oy[3], oz[3];
        const int nxc = axis_cells(c0, a.ncx, true, ox);
        const int nyc = axis_cells(c1, a.ncy, !a.g.wall_y, oy);
        int nzc = 1;
        oz[0] = 0;
        if (D == 3) nzc = axis_cells(c2, a.ncz, true, oz);
        if (lane < nxc * nyc * nzc) {
            const int kx = lane % nxc, ky = (lane / nxc) % nyc, kz = lane / (nxc * nyc);
            const int c = ox[kx] + a.ncx * (oy[ky] + a.ncy * oz[kz]);
            const int cnt = cell_entries(a, c);
            for (int s = 0; s < cnt; s++) {
                const int q = a.cell_ids[c * CELL_CAP + s];
                if (q == i || !nl_candidate(a, i, q)) continue;
                const int slot = atomicAdd(nl, 1);
                if (slot < NL_CAP) list[slot] = q;
                else atomicOr(a.flags, FLAG_CONTACT_OVERFLOW);
            }
        }
        lane_sync();
        n = min(*nl, NL_CAP);
        // each lane finds the place of its entry (ids differ)
        const int mine = lane < n ? list[lane] : 0x7fffffff;
        int place = 0;
        for (int s = 0; s < n; s++) place += list[s] < mine ? 1 : 0;
        lane_sync();
        if (lane < n) list[place] = mine;
        lane_sync();
        if (lane < n) {
            j = list[lane];
            a.nl[(int64_t)i * NL_CAP + lane] = j;
        }
        if (lane == 0) a.nl_len[i] = n;
        if (lane < D) a.xb[lane * P + i] = a.P.x[lane * P + i];
    } else {
        n = a.nl_len[i];
        if (lane < n) {
            j = a.nl[(int64_t)i * NL_CAP + lane];
            list[lane] = j;
        }
        lane_sync();
    }
    static_assert(NL_CAP <= 64, "a lane per listed neighbour");
    uint64_t touching = __ballot(j >= 0 && pair_force(a, i, j, nullptr));
    if (lane == 0) {
        if (__popcll(touching) > MAX_CONTACTS) atomicOr(a.flags, FLAG_CONTACT_OVERFLOW);
        double F[3] = {0.0, 0.0, 0.0};
        for (; touching; touching &= touching - 1) pair_force(a, i, list[__builtin_ctzll(touching)], F);
        wall_force(a, i, F);
        for (int d = 0; d < 3; d++) a.P.Fc[d * P + i] = F[d];
    }
}

template <int NT>
__global__ __launch_bounds__(NT) void k_dem_thread(CellArgs a) {
    __shared__ int list[MAX_CONTACTS][NT];
    dem_thread<NT>(a, (int)blockIdx.x * NT + (int)threadIdx.x, list);
}

// Footprints on the plain step.  LPP lanes of a wavefront (one wavefront per
// workgroup) take one segment of a particle's bounding box, or with LPP < 64
// the whole box: segment s of nseg holds the items s seg .. (s + 1) seg - 1 of
// the box (x fastest, seg = ceil(items / nseg)), and its covered nodes go, in
// item order, to the particle's list from entry s seg on, their number to
// list_len[p nseg + s].  Phases per chunk of items: (A) every item is
// classified by distance bounds, the undecided ones queued; (B) the queued
// items get the exact per-sample count, all lanes busy; (C1) the covered items
// move up in place; (C2) the k-th covered node claims an owner slot and takes
// its place in the list.  Runs of consecutive nodes in one aligned 8-byte word
// of the owner counts sit in consecutive lanes: the first lane of a run claims
// them with one 64-bit atomic add, and every lane reads its own byte of the
// returned word, which is what one atomic add per node would have returned.
//
// Bound by vector-instruction issue on many particles and by the chain of
// phases on few.  So (A) steps its coordinates without divisions and
// classifies in binary32 (about 45 instructions per item; a margin far above
// the rounding sends the doubtful ones to (B)), (C1) and (C2) place nodes and
// find runs by ballots, and the claims of two rounds are in flight together.
// Measured against the classification in binary64 with divisions, a prefix sum
// over LDS and shuffled runs that this replaces, one wavefront per sphere and
// 16 lanes per disc: 8 317 spheres R = 4 58 against 78 us, 16 128 spheres R = 5
// 155 against 224 us, 21 361 discs R = 5 37 against 43 us; with segments 310
// spheres R = 5.3 11 against 44 us, 16 discs R = 6 5.4 against 22.6 us, one
// sphere R = 16 6.7 against 784 us.
template <int D, int LPP>
struct FootLds {
    static constexpr int G = 64 / LPP, CHUNK = D == 3 ? 1024 : 512;
    uint32_t ent[G][CHUNK];  // list entries; count 0: not covered
    uint16_t todo[G][CHUNK];
};

template <int D, int S, int LPP>
__device__ __forceinline__ void foot_segment(const FootArgs &a, int block, FootLds<D, LPP> &lds) {
    constexpr int G = 64 / LPP, CHUNK = FootLds<D, LPP>::CHUNK;
    uint32_t(&s_ent)[G][CHUNK] = lds.ent;
    uint16_t(&s_todo)[G][CHUNK] = lds.todo;
    const int lane = (int)threadIdx.x, grp = lane / LPP, sub = lane % LPP;
    const int P = a.P.np, nseg = LPP == 64 ? a.P.nseg : 1;
    const int unit = block * G + grp;
    const int p = LPP == 64 ? unit / nseg : unit;
    const int s = LPP == 64 ? unit - p * nseg : 0;
    const bool live = p < P;
    const int q = live ? p : 0;  // the lanes of a missing particle run every loop empty
    int lo[3], hi[3];
    bbox(a.P, q, D, lo, hi);
    if (live && s == 0) write_rec(a.P, p, sub);
    if (live && sub == 0 && s == 0)
        for (int d = 0; d < 3; d++) {
            a.P.bb[d * P + p] = lo[d];
            a.P.bb[(3 + d) * P + p] = hi[d];
        }
    const double xp[3] = {a.P.x[q], a.P.x[P + q], D == 3 ? a.P.x[2 * P + q] : 0.0};
    // A centre must lie in the box on periodic axes (integration keeps it
    // there unless a particle moves a box length in one step) and be finite:
    // otherwise the bounding box cannot be wrapped and the particle gets an
    // empty footprint and an error flag.
    bool placed = live;
    for (int d = 0; d < D; d++) {
        const double L = d == 0 ? a.g.Lx : (d == 1 ? a.g.Ly : a.g.Lz);
        placed = placed && ((d == 1 && a.g.wall_y) ? (xp[d] > -L && xp[d] < 2.0 * L) : (xp[d] >= 0.0 && xp[d] < L));
    }
    if (live && !placed && sub == 0) atomicOr(a.flags, FLAG_NONFINITE);
    const int ext0 = hi[0] - lo[0] + 1, ext1 = hi[1] - lo[1] + 1;
    const int ext2 = D == 3 ? hi[2] - lo[2] + 1 : 1;
    const int items = placed ? ext0 * ext1 * ext2 : 0;
    const int seg = (items + nseg - 1) / nseg;
    const int i0 = s * seg, i1 = min(i0 + seg, items);
    const double r = a.P.R[q], R2 = r * r;
    const int64_t N = a.g.N;
    const int room = a.P.list_cap - i0;  // places of the particle's list from the segment's start on
    uint32_t *list = a.P.list + (int64_t)q * a.P.list_cap + i0;
    // (A) in binary32: the displacement of item (kx, ky, kz) from the centre
    // is base + k to 2e-5 at most (radii up to 62), so the bounds of the
    // squared distance over the cell's samples are good to 8e-3 at R = 62 and
    // in proportion below: a margin of 2e-4 (R + 2)
    const float h = 0.5f - 0.5f / (float)S;
    const float R2f = (float)R2, margin = 2e-4f * ((float)r + 2.0f);
    float base[3];
    for (int d = 0; d < 3; d++) base[d] = d < D ? (float)((double)lo[d] - xp[d]) : 0.0f;
    constexpr int FULL = D == 3 ? S * S * S : S * S;
    // item i0 + sub, and the step of LPP items, as box coordinates
    const float inv0 = 1.0f / (float)ext0, inv1 = 1.0f / (float)ext1;
    int kx, ky, kz, sx, sy, sz;
    {
        int rest = div_small(i0 + sub, ext0, inv0);
        kx = i0 + sub - rest * ext0;
        kz = D == 3 ? div_small(rest, ext1, inv1) : 0;
        ky = rest - kz * ext1;
        rest = div_small(LPP, ext0, inv0);
        sx = LPP - rest * ext0;
        sz = D == 3 ? div_small(rest, ext1, inv1) : 0;
        sy = rest - sz * ext1;
    }
    const int ylo = a.g.wall_y ? -lo[1] : -1024, yhi = a.g.wall_y ? a.g.ny - lo[1] : 1024;
    const uint64_t below = ((uint64_t)1 << sub) - 1;
    // this group's share of a wavefront mask
    auto group = [&](uint64_t m) { return LPP == 64 ? m : (m >> (grp * LPP)) & (((uint64_t)1 << (LPP & 63)) - 1); };
    int total = 0;
    for (int c0 = i0; __any(c0 < i1); c0 += CHUNK) {
        const int nc = min(i1 - c0, CHUNK);  // may be negative in a group that is done
        int ntodo = 0;
#pragma unroll 1
        for (int i = sub; __any(i < nc); i += LPP) {
            const float d0 = fabsf(base[0] + (float)kx), d1 = fabsf(base[1] + (float)ky), d2 = fabsf(base[2] + (float)kz);
            const float m0 = fmaxf(d0 - h, 0.0f), m1 = fmaxf(d1 - h, 0.0f), M0 = d0 + h, M1 = d1 + h;
            float near = fmaf(m1, m1, m0 * m0), far = fmaf(M1, M1, M0 * M0);
            if (D == 3) {
                const float m2 = fmaxf(d2 - h, 0.0f), M2 = d2 + h;
                near = fmaf(m2, m2, near);
                far = fmaf(M2, M2, far);
            }
            const bool in = i < nc && near <= R2f + margin && ky >= ylo && ky < yhi;
            const bool todo = in && far > R2f - margin;
            if (i < nc) s_ent[grp][i] = list_entry(in ? FULL : 0, kx, ky, kz);
            const uint64_t m = group(__ballot(todo));
            if (todo) s_todo[grp][ntodo + __popcll(m & below)] = (uint16_t)i;
            ntodo += __popcll(m);
            kx += sx;
            ky += sy;
            if (kx >= ext0) { kx -= ext0; ky++; }
            if (D == 3) {
                kz += sz;
                if (ky >= ext1) { ky -= ext1; kz++; }
            }
        }
        lane_sync();
        // (B) exact per-sample counts of the undecided items
#pragma unroll 1
        for (int j = sub; j < ntodo; j += LPP) {
            const int i = s_todo[grp][j];
            const uint32_t e = s_ent[grp][i];
            const int ix = wrap1(a.g, 0, lo[0] + (int)((e >> 10) & 127u));
            const int iy = wrap1(a.g, 1, lo[1] + (int)((e >> 17) & 127u));
            const int iz = D == 3 ? wrap1(a.g, 2, lo[2] + (int)((e >> 24) & 127u)) : 0;
            const int count = sample_count<D, S>(ndisp(a.g, 0, ix, xp[0]), ndisp(a.g, 1, iy, xp[1]),
                                                 D == 3 ? ndisp(a.g, 2, iz, xp[2]) : 0.0, R2);
            s_ent[grp][i] = (e & ~LIST_COUNT_MASK) | (uint32_t)count;
        }
        lane_sync();
        // (C1) covered items move up in place (a place is never above its item)
        int ncov = 0;
#pragma unroll 1
        for (int i = sub; __any(i < nc); i += LPP) {
            const uint32_t e = i < nc ? s_ent[grp][i] : 0u;
            const bool cov = (e & LIST_COUNT_MASK) != 0u;
            const uint64_t m = group(__ballot(cov));
            if (cov) s_ent[grp][ncov + __popcll(m & below)] = e;
            ncov += __popcll(m);
        }
        lane_sync();
        // box_extent keeps a box within its list; were one longer, the run ends
        // with the flag and nothing is written beyond the list
        if (total + ncov > room) {
            if (sub == 0) atomicOr(a.flags, FLAG_SLOT_OVERFLOW);
            ncov = max(room - total, 0);
        }
        // (C2) owner slots and list entries, UN rounds of claims in flight
        constexpr int UN = 2;
#pragma unroll 1
        for (int k0 = 0; __any(k0 < ncov); k0 += UN * LPP) {
            uint32_t ent[UN];
            int64_t node[UN];
            int back[UN];
            unsigned long long old[UN];
#pragma unroll
            for (int u = 0; u < UN; u++) {
                const int k = k0 + u * LPP + sub;
                const bool act = k < ncov;
                const uint32_t e = act ? s_ent[grp][k] : 0u;
                const int ix = wrap1(a.g, 0, lo[0] + (int)((e >> 10) & 127u));
                const int iy = wrap1(a.g, 1, lo[1] + (int)((e >> 17) & 127u));
                const int iz = D == 3 ? wrap1(a.g, 2, lo[2] + (int)((e >> 24) & 127u)) : 0;
                const int64_t n = (int64_t)ix + (int64_t)a.g.nx * ((int64_t)iy + (int64_t)a.g.ny * iz);
                // a run goes on while the next lane holds the next node of the word
                const int64_t prev = __shfl_up((long long)n, 1, 64);
                const bool head = !act || sub == 0 || n != prev + 1 || (n & 7) == 0;
                const uint64_t heads = __ballot(head);
                back[u] = lane - (63 - __clzll(heads & (((uint64_t)2 << lane) - 1)));
                const uint64_t after = lane == 63 ? 0 : heads >> (lane + 1);
                const int len = after ? __ffsll((unsigned long long)after) : 64 - lane;  // at most 8 when act
                old[u] = 0ull;
                if (act && head) {
                    const unsigned long long ones = 0x0101010101010101ull >> (8 * (8 - len));
                    old[u] = atomicAdd((unsigned long long *)(a.nown + (n & ~(int64_t)7)), ones << (8 * (n & 7)));
                }
                ent[u] = e;
                node[u] = n;
            }
#pragma unroll
            for (int u = 0; u < UN; u++) {
                const unsigned long long w = __shfl(old[u], lane - back[u], 64);
                const int k = k0 + u * LPP + sub;
                if (k < ncov) {
                    const int slot = (int)((w >> (8 * (int)(node[u] & 7))) & 0xffull);
                    if (slot < MAX_OWNERS)
                        a.slots[(int64_t)slot * N + node[u]] = ((uint32_t)p << SLOT_COUNT_BITS) | (ent[u] & LIST_COUNT_MASK);
                    else
                        atomicOr(a.flags, FLAG_SLOT_OVERFLOW);
                    list[total + k] = ent[u];
                }
            }
        }
        total += ncov;
        lane_sync();
    }
    if (live && sub == 0) a.P.list_len[(int64_t)p * nseg + s] = total;
}

// Footprints and, in the workgroups before them, the contacts of the step
// (ndem workgroups; THREAD: one thread per particle, else one wavefront): both
// read the particles only, and one launch keeps the step on one stream (a fork
// to a second stream and back cost about 10 us each way in the step's chain).
// Five wavefronts per SIMD (96 registers for spheres; 118 without the bound).
// 8 317 spheres: 62 us for both, where the footprint alone took 58 beside the
// cell list and the contacts (63 us) on a second stream; 21 361 discs 38 us.
template <int D, int S, int LPP, bool THREAD>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(LPP == 64 ? 5 : 4))) void k_foot(FootArgs a, CellArgs c, int ndem) {
    constexpr size_t FB = sizeof(FootLds<D, LPP>);
    constexpr size_t DB = THREAD ? sizeof(int[MAX_CONTACTS][64]) : sizeof(int[NL_CAP + 1]);
    __shared__ __attribute__((aligned(16))) char lds[FB > DB ? FB : DB];
    const int b = (int)blockIdx.x;
    if (b < ndem) {
        int *list = (int *)lds;
        if (THREAD) dem_thread<64>(c, b * 64 + (int)threadIdx.x, (int(*)[64])list);
        else if (c.every > 0) dem_list_wave(c, b, list, list + NL_CAP);
        else dem_wave(c, b, list, list + NL_CAP);
        return;
    }
    foot_segment<D, S, LPP>(a, b - ndem, *(FootLds<D, LPP> *)lds);
}

// Footprints of every particle (one workgroup each), or of the particles of
// group G.g (workgroups walk the group's list).
template <int D, int S, int NT, bool TAB>
__global__ __launch_bounds__(NT) void k_foot_paint(FootArgs a) {
    if (a.G.g < 0) {
        foot_one<D, S, NT, TAB>(a, (int)blockIdx.x);
        return;
    }
    const int n = a.G.count[a.G.g];
    const int *lst = a.G.list + (int64_t)a.G.g * a.G.stride;
    for (int i = (int)blockIdx.x; i < n; i += (int)gridDim.x) {
        foot_one<D, S, NT, TAB>(a, lst[i]);
        __syncthreads();  // the shared buffers are reused by the next particle
    }
}

__device__ __forceinline__ double wrap_pos(double x, double L) {
    if (x < 0.0) {
        x = x + L;
        if (x >= L) x = x - L;
    } else if (x >= L) {
        x = x - L;
    }
    return x;
}

// ------------------------------------------------- hydrodynamic force, Eq. 3
struct Acc {
    double s, c;
};

__device__ __forceinline__ void acc_add(Acc &A, double p) {
    const double x = A.s + p;
    const double bb = x - A.s;
    const double e = (A.s - (x - bb)) + (p - bb);
    A.s = x;
    A.c = A.c + e;
}

__device__ __forceinline__ void acc_merge(Acc &A, const Acc &B) {
    const double x = A.s + B.s;
    const double bb = x - A.s;
    const double e = (A.s - (x - bb)) + (B.s - bb);
    A.s = x;
    A.c = (A.c + B.c) + e;
}

__device__ __forceinline__ double shfl_xor_d(double v, int m) {
    return __shfl_xor(v, m, 64);
}

// Sum of NC accumulators over LPP lanes (aligned runs of a wavefront): while
// several are left, the lanes split in halves that each keep half of them, so
// six components take 9 merges instead of 36.  Component c's sum ends up in
// lane acc_place<LPP, NC>(c) of the run (and the lanes that differ from it in
// the lower bits).
template <int LPP, int NC>
__device__ __forceinline__ void acc_reduce(Acc (&v)[NC], int sub) {
    int n = NC;
#pragma unroll
    for (int m = LPP / 2; m >= 1; m >>= 1) {
        const int h = n > 1 ? (n + 1) / 2 : 1;
        const bool up = n > 1 && (sub & m) != 0;
#pragma unroll
        for (int c = 0; c < NC; c++) {
            if (c >= h) continue;
            const Acc lo = v[c], hi = n > 1 ? (c + h < n ? v[c + h < NC ? c + h : 0] : Acc{0.0, 0.0}) : v[c];
            Acc keep = up ? hi : lo;
            const Acc give = up ? lo : hi;
            const Acc got = {shfl_xor_d(give.s, m), shfl_xor_d(give.c, m)};
            acc_merge(keep, got);
            v[c] = keep;
        }
        n = h;
    }
}

template <int LPP, int NC>
constexpr int acc_place(int c) {
    int n = NC, at = 0;
    for (int m = LPP / 2; m >= 1 && n > 1; m >>= 1) {
        const int h = (n + 1) / 2;
        if (c >= h) { at += m; c -= h; }
        n = h;
    }
    return at;
}

// NT threads per particle over its footprint list (NT <= 64: an aligned run of
// lanes of a wavefront; above: a workgroup, or with `parts` > 1 workgroups that
// take a share of the list each, this one's index being `part`): each entry gives the node and the
// particle's sample count there; q_n and the node's total count come from the
// lattice kernel.  s_pn q_n and r_pn x (s_pn q_n) go into TwoSum accumulators,
// which are merged over the lanes, then over the wavefronts in turn, then over
// the workgroups in turn by the one that finishes last (each leaves its sums
// and counts itself in; nothing waits).  F_p = -sum, T_p = -sum.  With `integrate` set, the first thread then advances
// the particle (the contact forces of the step are complete).  `sub` is the
// thread's index among the particle's; `live` is false for the runs past the
// last particle, which take part in the shuffles only.
template <int D, bool R32, int NT>
__device__ __forceinline__ void force_unit(const ForceArgs &a, int p, int sub, bool live, int part = 0) {
    static_assert(NT >= 16 && NT <= 256 && (NT & (NT - 1)) == 0, "threads per particle");
    constexpr int LPP = NT < 64 ? NT : 64, W = NT / LPP;  // lanes per wavefront, wavefronts
    constexpr int NC = D == 3 ? 6 : 3;                    // F_x, F_y, F_z, T_x, T_y, T_z or F_x, F_y, T_z
    const int lane = threadIdx.x & 63;
    const int gbase = lane - sub % LPP;
    const int P = a.P.np;
    const int q = live ? p : 0;
    const int cap = a.P.list_cap, nseg = a.P.nseg;
    const int lo0 = a.P.bb[q], lo1 = a.P.bb[P + q], lo2 = a.P.bb[2 * P + q];
    const double xp0 = a.P.x[q], xp1 = a.P.x[P + q], xp2 = D == 3 ? a.P.x[2 * P + q] : 0.0;
    // the integration inputs, one per lane (v, omega, F^c, m, I, fixed), loaded
    // beside the sums and gathered by the first thread at the end
    double pre = 0.0;
    if (live && a.integrate && sub < 12) {
        if (sub < 3) pre = a.P.v[sub * P + p];
        else if (sub < 6) pre = a.P.w[(sub - 3) * P + p];
        else if (sub < 9) pre = a.P.Fc[(sub - 6) * P + p];
        else if (sub == 9) pre = a.P.m[p];
        else if (sub == 10) pre = a.P.I[p];
        else pre = a.P.fixed[p] ? 1.0 : 0.0;
    }
    Acc A[NC];
#pragma unroll
    for (int c = 0; c < NC; c++) A[c] = Acc{0.0, 0.0};
    // lattice coordinates of an entry, formed again where needed (fewer
    // registers live across the loads)
    auto coords = [&](uint32_t e, int &ix, int &iy, int &iz) {
        ix = wrap1(a.g, 0, lo0 + (int)((e >> 10) & 127u));
        iy = wrap1(a.g, 1, lo1 + (int)((e >> 17) & 127u));
        iz = D == 3 ? wrap1(a.g, 2, lo2 + (int)((e >> 24) & 127u)) : 0;
    };
    // one segment: every thread of the particle, or with several segments one
    // wavefront each in turn
    const int seg = nseg > 1 ? list_seg(a.P, q) : 0;
    const int parts = NT > 64 ? a.parts : 1;
    const int first = nseg > 1 ? sub % LPP : part * NT + sub, width = nseg > 1 ? LPP : parts * NT;
    for (int s = nseg > 1 ? part * W + sub / LPP : 0; s < nseg; s += parts * W) {
        const uint32_t *list = a.P.list + (int64_t)q * cap + s * seg;
        const int room = cap - s * seg;  // entries of the particle's list from here on
        const int len = live ? a.P.list_len[(int64_t)q * nseg + s] : 0;
        // UN entries per thread per round: all q loads of a round are issued
        // before the first accumulation, and the list entries of the next round
        // are loaded while they are in flight (the first round's beside the list
        // length: loads below the capacity stay inside the particle's list).
        constexpr int UN = 2;
        const int stride = UN * width;
        uint32_t vn[UN];
#pragma unroll
        for (int u = 0; u < UN; u++) {
            const int e = u * width + first;
            vn[u] = e < room ? list[e] : 0u;
        }
        for (int e0 = 0; e0 < len; e0 += stride) {
            uint32_t v[UN];
#pragma unroll
            for (int u = 0; u < UN; u++) {
                const int e = e0 + u * width + first;
                v[u] = e < len ? vn[u] : 0u;
            }
            double q0[UN], q1[UN], q2[UN];
            int tot[UN];
#pragma unroll
            for (int u = 0; u < UN; u++) {
                q0[u] = q1[u] = q2[u] = 0.0;
                tot[u] = 1;
                if (v[u] != 0u) {
                    int ix, iy, iz;
                    coords(v[u], ix, iy, iz);
                    const int64_t n = (int64_t)ix + (int64_t)a.g.nx * ((int64_t)iy + (int64_t)a.g.ny * iz);
                    double qq[3];
                    read_qrec(a.qr, R32, n, qq, tot[u]);
                    q0[u] = qq[0];
                    q1[u] = qq[1];
                    q2[u] = qq[2];
                }
            }
#pragma unroll
            for (int u = 0; u < UN; u++) {
                const int e = e0 + stride + u * width + first;
                vn[u] = e < len ? list[e] : 0u;
            }
#pragma unroll
            for (int u = 0; u < UN; u++) {
                if (v[u] == 0u) continue;
                const int cnt = (int)(v[u] & LIST_COUNT_MASK);
                int ix, iy, iz;
                coords(v[u], ix, iy, iz);
                // the particle's share of the node: exactly 1 where it is the
                // only owner (cnt = tot), the division only where a wavefront
                // holds a shared node
                double sh = 1.0;
                if (__any(cnt != tot[u]) && cnt != tot[u]) sh = (double)cnt / (double)tot[u];
                const double t0 = sh * q0[u], t1 = sh * q1[u];
                const double rx = ndisp(a.g, 0, ix, xp0);
                const double ry = ndisp(a.g, 1, iy, xp1);
                acc_add(A[0], t0);
                acc_add(A[1], t1);
                if (D == 3) {
                    const double t2 = sh * q2[u];
                    const double rz = ndisp(a.g, 2, iz, xp2);
                    acc_add(A[2], t2);
                    acc_add(A[3 % NC], ry * t2 - rz * t1);
                    acc_add(A[4 % NC], rz * t0 - rx * t2);
                    acc_add(A[5 % NC], rx * t1 - ry * t0);
                } else {
                    acc_add(A[2], rx * t1 - ry * t0);
                }
            }
        }
    }
    acc_reduce<LPP, NC>(A, sub);
    double val[NC];  // the particle's sums, in every lane of its first wavefront
    if (W == 1) {
        const double mine = A[0].s + A[0].c;
#pragma unroll
        for (int c = 0; c < NC; c++) val[c] = __shfl(mine, gbase + acc_place<LPP, NC>(c), 64);
    } else {
        __shared__ Acc wsum[W][NC];
#pragma unroll
        for (int c = 0; c < NC; c++)
            if (lane == acc_place<LPP, NC>(c)) wsum[sub / LPP][c] = A[0];
        __syncthreads();
        if (sub >= 64) return;
        const int c0 = lane < NC ? lane : 0;
        Acc t = wsum[0][c0];
        for (int w = 1; w < W; w++) acc_merge(t, wsum[w][c0]);
        if (parts > 1) {
            // the other workgroups may run on another XCD: agent scope throughout
            double *const sums = a.part + (int64_t)p * parts * 2 * NC + 2 * c0;
            if (lane < NC) {
                __hip_atomic_store(sums + part * 2 * NC, t.s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(sums + part * 2 * NC + 1, t.c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            int before = 0;
            if (lane == 0)
                before = __hip_atomic_fetch_add(&a.arrived[p], 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
            if (__shfl(before, 0, 64) != parts - 1) return;
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            if (lane == 0) a.arrived[p] = 0;  // for the next step
            // lane 8 g + c adds component c of the workgroups g, g + 8, ..., then
            // the eight lanes of a component merge
            const double *const from = a.part + (int64_t)p * parts * 2 * NC + 2 * ((lane & 7) < NC ? lane & 7 : 0);
            t = Acc{0.0, 0.0};
            for (int b = lane >> 3; b < parts; b += 8)
                acc_merge(t, Acc{__hip_atomic_load(from + b * 2 * NC, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                                 __hip_atomic_load(from + b * 2 * NC + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)});
#pragma unroll
            for (int m = 8; m < 64; m <<= 1) acc_merge(t, Acc{shfl_xor_d(t.s, m), shfl_xor_d(t.c, m)});
        }
#pragma unroll
        for (int c = 0; c < NC; c++) val[c] = __shfl(t.s + t.c, c, 64);
    }
    // axis d is lane d's from here on
    const int d = sub % LPP < 3 ? sub % LPP : 2;
    const double pv = __shfl(pre, gbase + d, 64), pw = __shfl(pre, gbase + 3 + d, 64);
    const double pfc = __shfl(pre, gbase + 6 + d, 64);
    const double pm = __shfl(pre, gbase + 9, 64), pI = __shfl(pre, gbase + 10, 64);
    const double pfix = __shfl(pre, gbase + 11, 64);
    const double xo = d == 0 ? xp0 : (d == 1 ? xp1 : xp2);
    double Fv = 0.0, Tv = 0.0;
    if (D == 3) {
        Fv = -(d == 0 ? val[0] : (d == 1 ? val[1] : val[2]));
        Tv = -(d == 0 ? val[3 % NC] : (d == 1 ? val[4 % NC] : val[5 % NC]));
    } else {
        if (d < 2) Fv = -(d == 0 ? val[0] : val[1]);
        if (d == 2) Tv = -val[2];
    }
    const bool mine = live && sub < 3;
    double vn = pv, xn = xo;
    if (mine) {
        a.P.Fh[d * P + p] = Fv;
        a.P.Th[d * P + p] = Tv;
        // Symplectic Euler with dt = 1 for this particle (every reader of its
        // position in this kernel has read it): v += (F^h + F^c + m a)/m,
        // omega += T^h/I, x += v (new), periodic wrap.
        if (a.integrate && pfix == 0.0) {
            if (d < D) {
                const double ftot = Fv + pfc + pm * a.ap[d];
                vn = pv + ftot / pm;
                a.P.v[d * P + p] = vn;
                xn = xo + vn;
                if (!(d == 1 && a.g.wall_y)) xn = wrap_pos(xn, d == 0 ? a.g.Lx : (d == 1 ? a.g.Ly : a.g.Lz));
                a.P.x[d * P + p] = xn;
            }
            if (D == 3 || d == 2) a.P.w[d * P + p] = pw + Tv / pI;
            // the slab pipeline assumes at most one node of motion in y per step
            if (d == 1 && a.G.K > 1 && !(fabs(vn) <= 1.0)) atomicOr(a.flags, FLAG_FAST);
        }
    }
    if (a.integrate && a.G.K > 1 && mine && d == 1) {
        // file the particle in its group of the next step
        const int gn = slab_group(a.G, xn, a.P.R[p]);
        const int slot = atomicAdd(&a.G.ncount[gn], 1);
        a.G.nlist[(int64_t)gn * a.G.stride + slot] = p;
    }
    if (a.file) {
        // file the particle in the cell list of the next step, and clear the
        // count of the cell that held it in this one (its contacts are done)
        const int nc = d == 0 ? a.nc[0] : (d == 1 ? a.nc[1] : a.nc[2]);
        const int was = d < D ? cell_coord(a.g, nc, d, xo) : 0, is = d < D ? cell_coord(a.g, nc, d, xn) : 0;
        const int w1 = __shfl(was, gbase + 1, 64), w2 = __shfl(was, gbase + 2, 64);
        const int i1 = __shfl(is, gbase + 1, 64), i2 = __shfl(is, gbase + 2, 64);
        if (live && sub == 0) {
            a.cell_old[was + a.nc[0] * (w1 + a.nc[1] * w2)] = 0;
            file_in_cell(a.cell_new, a.cell_ids, is + a.nc[0] * (i1 + a.nc[1] * i2), p);
        }
        if (a.every > 0) {
            // the guard of the neighbour lists for the next step: how far the
            // particle has moved since the build (k_nl_check's sum), and the age
            double dd = 0.0;
            if (live && d < D) {
                dd = xn - a.xb[d * P + p];
                if (!(d == 1 && a.g.wall_y)) dd = pdisp(dd, d == 0 ? a.g.Lx : (d == 1 ? a.g.Ly : a.g.Lz));
            }
            double d2 = 0.0;
            for (int ax = 0; ax < D; ax++) {
                const double v = __shfl(dd, gbase + ax, 64);
                d2 = d2 + v * v;
            }
            const double lim = 0.49 * a.skin;
            if (live && sub == 0) {
                bool again = !(d2 < lim * lim);
                if (p == 0) {
                    const int built = *a.nl_flag;
                    const int age = built ? 1 : *a.nl_age + 1;
                    *a.nl_age = age;
                    if (built) *a.nl_builds = *a.nl_builds + 1;
                    *a.nl_flag = 0;
                    again = again || age >= a.every;
                }
                if (again) atomicOr(a.nl_next, 1);
            }
        }
    }
}

// Force, torque and integration of every particle: 64 / NT particles per
// wavefront and one wavefront per workgroup, or a.parts workgroups of NT
// threads per particle.
template <int D, bool R32, int NT>
__global__ __launch_bounds__(NT < 64 ? 64 : NT) void k_force(ForceArgs a) {
    const int t = (int)threadIdx.x;
    if (NT > 64) {
        const int p = (int)blockIdx.x / a.parts;
        force_unit<D, R32, NT>(a, p, t, true, (int)blockIdx.x - p * a.parts);
    } else {
        const int p = (int)blockIdx.x * (64 / NT) + t / NT;
        force_unit<D, R32, NT>(a, p, t % NT, p < a.P.np);
    }
}

// The same for the particles of group G.g, one wavefront each; workgroups walk
// the group's list.
template <int D, bool R32>
__global__ __launch_bounds__(64) void k_force_group(ForceArgs a) {
    const int n = a.G.count[a.G.g];
    const int *lst = a.G.list + (int64_t)a.G.g * a.G.stride;
    for (int i = (int)blockIdx.x; i < n; i += (int)gridDim.x)
        force_unit<D, R32, 64>(a, lst[i], (int)threadIdx.x, true);
}

// Files every particle in its group of the current positions.
__global__ void k_assign_groups(ForceArgs a) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const int P = a.P.np;
    if (p >= P) return;
    const int g = slab_group(a.G, a.P.x[P + p], a.P.R[p]);
    const int slot = atomicAdd(&a.G.ncount[g], 1);
    a.G.nlist[(int64_t)g * a.G.stride + slot] = p;
}

// q_n of the last step at the nodes of the current footprint lists (the nodes
// the lattice kernel covered); `out` [D][N] is zero elsewhere beforehand.
template <int D>
__global__ void k_list_q(ForceArgs a, double *out) {
    const int p = blockIdx.x;
    const int P = a.P.np;
    const int lo0 = a.P.bb[p], lo1 = a.P.bb[P + p], lo2 = a.P.bb[2 * P + p];
    const int64_t N = a.g.N;
    const int seg = a.P.nseg > 1 ? list_seg(a.P, p) : 0;  // (no boxes before the first step)
    for (int s = 0; s < a.P.nseg; s++) {
        const uint32_t *list = a.P.list + (int64_t)p * a.P.list_cap + s * seg;
        const int len = a.P.list_len[(int64_t)p * a.P.nseg + s];
        for (int e = threadIdx.x; e < len; e += blockDim.x) {
            const uint32_t v = list[e];
            const int ix = wrap1(a.g, 0, lo0 + (int)((v >> 10) & 127u));
            const int iy = wrap1(a.g, 1, lo1 + (int)((v >> 17) & 127u));
            const int iz = D == 3 ? wrap1(a.g, 2, lo2 + (int)((v >> 24) & 127u)) : 0;
            const int64_t n = (int64_t)ix + (int64_t)a.g.nx * ((int64_t)iy + (int64_t)a.g.ny * iz);
            double qq[3];
            int tot;
            read_qrec(a.qr, a.rec32 != 0, n, qq, tot);
            for (int d = 0; d < D; d++) out[d * N + n] = qq[d];
        }
    }
}

// ------------------------------------------------------ neighbour-list mode
// The lists hold, in ascending id, every j with |r_i - r_j| < R_i + R_j + skin
// (minimum image) at the last build.  A pair missing from the lists was at
// least that far apart, so it can only touch after one of the two moved at
// least skin / 2; the guard rebuilds before any particle has moved 0.49 skin
// since the build, and after `every` steps in any case.  Contacts then sum the
// touching listed neighbours in ascending id, the order of k_dem, so both
// modes give the same bits.

// Guard: raises the rebuild flag when a particle moved 0.49 skin or more since
// the last build, or the lists are `every` steps old.
__global__ void k_nl_check(CellArgs a) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const int P = a.P.np;
    if (p == 0 && *a.nl_age >= a.every) atomicOr(a.nl_flag, 1);
    if (p >= P) return;
    double d2 = 0.0;
    for (int ax = 0; ax < a.D; ax++) {
        double dd = a.P.x[ax * P + p] - a.xb[ax * P + p];
        if (!(ax == 1 && a.g.wall_y)) dd = pdisp(dd, ax == 0 ? a.g.Lx : (ax == 1 ? a.g.Ly : a.g.Lz));
        d2 = d2 + dd * dd;
    }
    const double lim = 0.49 * a.skin;
    if (!(d2 < lim * lim)) atomicOr(a.nl_flag, 1);
}

// Cell binning, on rebuild steps only (the counts are zero on entry).
__global__ void k_nl_cells(CellArgs a) {
    if (!*a.nl_flag) return;
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const int P = a.P.np;
    if (p >= P) return;
    const int cx = cell_coord(a, 0, a.P.x[p]);
    const int cy = cell_coord(a, 1, a.P.x[P + p]);
    const int cz = a.D == 3 ? cell_coord(a, 2, a.P.x[2 * P + p]) : 0;
    file_in_cell(a.cell_count, a.cell_ids, cx + a.ncx * (cy + a.ncy * cz), p);
}

// List build, on rebuild steps only: one wavefront per particle, each lane
// scans one neighbour cell (cell edge >= 2 R_max + skin), the candidates are
// gathered in LDS and sorted by id; the build positions are recorded.
__global__ __launch_bounds__(256) void k_nl_build(CellArgs a) {
    if (!*a.nl_flag) return;
    __shared__ int list[4][NL_CAP];
    __shared__ int nlist[4];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int i = blockIdx.x * 4 + wave;
    const int P = a.P.np;
    const int D = a.D;
    if (lane == 0) nlist[wave] = 0;
    __syncthreads();
    if (i < P) {
        const int c0 = cell_coord(a, 0, a.P.x[i]);
        const int c1 = cell_coord(a, 1, a.P.x[P + i]);
        const int c2 = D == 3 ? cell_coord(a, 2, a.P.x[2 * P + i]) : 0;
        int ox[3], oy[3], oz[3];
        const int nxc = axis_cells(c0, a.ncx, true, ox);
        const int nyc = axis_cells(c1, a.ncy, !a.g.wall_y, oy);
        int nzc = 1;
        oz[0] = 0;
        if (D == 3) nzc = axis_cells(c2, a.ncz, true, oz);
        if (lane < nxc * nyc * nzc) {
            const int kx = lane % nxc, ky = (lane / nxc) % nyc, kz = lane / (nxc * nyc);
            const int c = ox[kx] + a.ncx * (oy[ky] + a.ncy * oz[kz]);
            const int cnt = cell_entries(a, c);
            for (int s = 0; s < cnt; s++) {
                const int j = a.cell_ids[c * CELL_CAP + s];
                if (j == i || !nl_candidate(a, i, j)) continue;
                const int slot = atomicAdd(&nlist[wave], 1);
                if (slot < NL_CAP) list[wave][slot] = j;
                else atomicOr(a.flags, FLAG_CONTACT_OVERFLOW);
            }
        }
        if (lane < D) a.xb[lane * P + i] = a.P.x[lane * P + i];
    }
    __syncthreads();
    if (i < P && lane == 0) {
        int *l = list[wave];
        const int nl = min(nlist[wave], NL_CAP);
        for (int s = 1; s < nl; s++) {
            const int v = l[s];
            int t = s - 1;
            while (t >= 0 && l[t] > v) {
                l[t + 1] = l[t];
                t--;
            }
            l[t + 1] = v;
        }
        for (int s = 0; s < nl; s++) a.nl[(int64_t)i * NL_CAP + s] = l[s];
        a.nl_len[i] = nl;
    }
}

// Contacts from the lists (Eqs. 4-5): one thread per particle, the touching
// listed neighbours in ascending id, then the walls.
__global__ void k_dem_list(CellArgs a) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int P = a.P.np;
    if (i >= P) return;
    const int n = a.nl_len[i];
    int touching = 0;
    double F[3] = {0.0, 0.0, 0.0};
    for (int s = 0; s < n; s++) touching += pair_force(a, i, a.nl[(int64_t)i * NL_CAP + s], F) ? 1 : 0;
    if (touching > MAX_CONTACTS) atomicOr(a.flags, FLAG_CONTACT_OVERFLOW);
    wall_force(a, i, F);
    for (int d = 0; d < 3; d++) a.P.Fc[d * P + i] = F[d];
}

// After a rebuild: clear the cell counts for the next one.
__global__ void k_nl_clear(CellArgs a) {
    if (!*a.nl_flag) return;
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < a.ncell;
         c += (int64_t)gridDim.x * blockDim.x)
        a.cell_count[c] = 0;
}

// Ages the lists and lowers the rebuild flag (one thread, after every other
// kernel of the step's neighbour work has read the flag).
__global__ void k_nl_finish(CellArgs a) {
    if (*a.nl_flag) {
        *a.nl_flag = 0;
        *a.nl_age = 1;
        *a.nl_builds = *a.nl_builds + 1;
    } else {
        *a.nl_age = *a.nl_age + 1;
    }
}


// ---------------------------------------------------------------- launchers
static unsigned blocks_for(int n, int per) { return (unsigned)((n + per - 1) / per); }

// workgroups of a launch that walks one group's list
constexpr int GROUP_GRID = 4096;

// 2D runs of this many discs keep 16 lanes per disc in the footprint, four discs
// per wavefront, and a thread per disc for the contacts; with fewer, a wavefront
// or several per disc shorten the chain.  us per step with 16 lanes and a thread
// / with a wavefront for both, R = 5 on a tenth of the area, FP64: 2 048 discs
// 69.7 / 66.9, 4 096 105.6 / 105.0, 8 192 193.6 / 195.6, 12 000 283.0 / 283.3,
// 16 384 361.5 / 364.1, 21 361 464 / 472, 40 000 910 / 927: within 1 % from
// 4 096 to 16 384 discs, so the line lies where the contacts alone always gain
// (1 166 400 discs 0.54 against 4.4 ms).  8 317 spheres with a thread each for
// the contacts took 168 against 26 us.
constexpr int DISC_MANY = 16384;

template <int D, int NT, bool TAB>
static hipError_t paint_s(const FootArgs &a, hipStream_t s) {
    const dim3 g((unsigned)(a.G.g < 0 ? a.P.np : std::min(a.P.np, GROUP_GRID))), b((unsigned)NT);
    switch (a.S) {
        case 1: hipLaunchKernelGGL((k_foot_paint<D, 1, NT, TAB>), g, b, 0, s, a); break;
        case 2: hipLaunchKernelGGL((k_foot_paint<D, 2, NT, TAB>), g, b, 0, s, a); break;
        case 3: hipLaunchKernelGGL((k_foot_paint<D, 3, NT, TAB>), g, b, 0, s, a); break;
        case 4: hipLaunchKernelGGL((k_foot_paint<D, 4, NT, TAB>), g, b, 0, s, a); break;
        case 5: hipLaunchKernelGGL((k_foot_paint<D, 5, NT, TAB>), g, b, 0, s, a); break;
        case 6: hipLaunchKernelGGL((k_foot_paint<D, 6, NT, TAB>), g, b, 0, s, a); break;
        case 7: hipLaunchKernelGGL((k_foot_paint<D, 7, NT, TAB>), g, b, 0, s, a); break;
        default: hipLaunchKernelGGL((k_foot_paint<D, 8, NT, TAB>), g, b, 0, s, a); break;
    }
    return hipGetLastError();
}

// Threads per particle of the footprint kernel (compile-time knobs for
// measurement).  Measured on MI355X at 4^D samples: a disc of radius 5 runs
// fastest with one wavefront (1.3-1.4x faster than two; four are slower
// still), a sphere of radius 4 with two (one or four are slower).
#ifndef FOOT_NT2
#define FOOT_NT2 64
#endif
#ifndef FOOT_NT3
#define FOOT_NT3 128
#endif

template <int D, int LPP, bool THREAD>
static hipError_t paint_plain(const FootArgs &a, const CellArgs &c, bool dem, hipStream_t s) {
    const int ndem = !dem ? 0 : (THREAD ? (int)blocks_for(a.P.np, 64) : a.P.np);
    const dim3 g((unsigned)(ndem + (LPP == 64 ? (int64_t)a.P.np * a.P.nseg : blocks_for(a.P.np, 64 / LPP)))), b(64);
    switch (a.S) {
        case 1: hipLaunchKernelGGL((k_foot<D, 1, LPP, THREAD>), g, b, 0, s, a, c, ndem); break;
        case 2: hipLaunchKernelGGL((k_foot<D, 2, LPP, THREAD>), g, b, 0, s, a, c, ndem); break;
        case 3: hipLaunchKernelGGL((k_foot<D, 3, LPP, THREAD>), g, b, 0, s, a, c, ndem); break;
        case 4: hipLaunchKernelGGL((k_foot<D, 4, LPP, THREAD>), g, b, 0, s, a, c, ndem); break;
        case 5: hipLaunchKernelGGL((k_foot<D, 5, LPP, THREAD>), g, b, 0, s, a, c, ndem); break;
        case 6: hipLaunchKernelGGL((k_foot<D, 6, LPP, THREAD>), g, b, 0, s, a, c, ndem); break;
        case 7: hipLaunchKernelGGL((k_foot<D, 7, LPP, THREAD>), g, b, 0, s, a, c, ndem); break;
        default: hipLaunchKernelGGL((k_foot<D, 8, LPP, THREAD>), g, b, 0, s, a, c, ndem); break;
    }
    return hipGetLastError();
}

// Footprint segments per particle: with few particles a box is cut until
// about 2 048 wavefronts are busy, down to 48 items per segment.
int foot_segments(int D, int np, double rmax) {
    const double ext = (double)box_extent(rmax);
    const double items = D == 2 ? ext * ext : ext * ext * ext;
    int nseg = 1;
    while (nseg < FOOT_SEG_MAX && (int64_t)np * nseg < FOOT_SEG_UNITS / 2 && items >= 96.0 * nseg) nseg *= 2;
    return nseg;
}

bool many_discs(int D, int np) { return D == 2 && np >= DISC_MANY; }

static hipError_t paint_any(const FootArgs &a, const CellArgs &c, bool dem, int D, hipStream_t s) {
    if (D == 3) return paint_plain<3, 64, false>(a, c, dem, s);
    return many_discs(D, a.P.np) ? paint_plain<2, 16, true>(a, c, dem, s) : paint_plain<2, 64, false>(a, c, dem, s);
}

hipError_t launch_foot_paint(const FootArgs &a, int D, hipStream_t s) {
    if (a.P.np == 0) return hipSuccess;
    // the table lookup is a kernel of its own, so the sampling kernel keeps
    // its registers
    if (a.tab) return D == 2 ? paint_s<2, FOOT_NT2, true>(a, s) : paint_s<3, FOOT_NT3, true>(a, s);
    if (a.G.g < 0) return paint_any(a, CellArgs{}, false, D, s);
    return D == 2 ? paint_s<2, FOOT_NT2, false>(a, s) : paint_s<3, FOOT_NT3, false>(a, s);
}

hipError_t launch_foot_dem(const FootArgs &a, const CellArgs &c, int D, hipStream_t s) {
    return a.P.np == 0 ? hipSuccess : paint_any(a, c, true, D, s);
}

template <int D, int NT>
static void force_nt(const ForceArgs &a, dim3 g, hipStream_t s) {
    const dim3 b(NT < 64 ? 64 : NT);
    if (a.rec32) hipLaunchKernelGGL((k_force<D, true, NT>), g, b, 0, s, a);
    else hipLaunchKernelGGL((k_force<D, false, NT>), g, b, 0, s, a);
}

// Threads per particle of the force kernel on the plain step: 16 per disc and
// 64 per sphere on many particles (1 166 400 discs: 1.18 against 1.62 ms with 64
// lanes each; spheres within 3 % with 16 or 32), four times as many while that
// leaves fewer than four wavefronts per SIMD and a thread still has an entry;
// beyond 256, several workgroups per particle, an entry per thread, 256 in all
// (each one's agent-scope release and arrival cost more than the shorter walk
// saves beyond that: 16 spheres R = 10, us with 1 / 4 / 16 / 64 workgroups each:
// 49 / 21 / 17 / 33, 64 spheres with 1 / 4 / 16: 32 / 20 / 47).  With few
// particles the walk over the list bounds the step: one sphere R = 16 10.4 us
// with 64 workgroups against 46 with 1 024 threads and 240 with 64, 310 spheres R = 5.3 11 us
// with 256 against 18 with 64, 16 discs R = 6 8.1 us with 64 against 10.7 with 16.
// The slab pipeline's groups take one wavefront per particle.
static int force_threads(const ForceArgs &a) {
    int nt = a.D == 2 ? 16 : 64;
    while (nt < 256 && (int64_t)a.P.np * nt < 262144 && 4 * nt <= a.entries) nt *= 4;
    return nt;
}

hipError_t launch_force(const ForceArgs &args, hipStream_t s) {
    ForceArgs a = args;
    a.parts = 1;
    if (a.P.np == 0) return hipSuccess;
    if (a.G.g >= 0) {
        const dim3 g((unsigned)std::min(a.P.np, GROUP_GRID)), b(64);
        if (a.D == 2) {
            if (a.rec32) hipLaunchKernelGGL((k_force_group<2, true>), g, b, 0, s, a);
            else hipLaunchKernelGGL((k_force_group<2, false>), g, b, 0, s, a);
        } else {
            if (a.rec32) hipLaunchKernelGGL((k_force_group<3, true>), g, b, 0, s, a);
            else hipLaunchKernelGGL((k_force_group<3, false>), g, b, 0, s, a);
        }
        return hipGetLastError();
    }
    const int nt = force_threads(a);
    if (nt == 256) a.parts = std::max(1, std::min({a.entries / 256, FORCE_PARTS / a.P.np, 64}));
    const dim3 g(nt > 64 ? (unsigned)(a.P.np * a.parts) : blocks_for(a.P.np, 64 / nt));
    if (a.D == 2) {
        if (nt == 16) force_nt<2, 16>(a, g, s);
        else if (nt == 64) force_nt<2, 64>(a, g, s);
        else force_nt<2, 256>(a, g, s);
    } else {
        if (nt == 64) force_nt<3, 64>(a, g, s);
        else force_nt<3, 256>(a, g, s);
    }
    return hipGetLastError();
}

hipError_t launch_assign_groups(const ForceArgs &a, hipStream_t s) {
    if (a.P.np == 0) return hipSuccess;
    hipLaunchKernelGGL(k_assign_groups, dim3(blocks_for(a.P.np, 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

__global__ void k_read_flags(const uint32_t *flags, uint32_t *dst) {
    if (threadIdx.x < 4) dst[threadIdx.x] = flags[threadIdx.x];
}

hipError_t launch_read_flags(const uint32_t *flags, uint32_t *dst, hipStream_t s) {
    hipLaunchKernelGGL(k_read_flags, dim3(1), dim3(64), 0, s, flags, dst);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_read_vecs(ReadArgs a, int p0, int n) {
    const int i = (int)(blockIdx.x * 256 + threadIdx.x), v = (int)blockIdx.y;
    if (i >= 3 * n) return;
    a.dst[v][i] = a.src[v][(int64_t)(i % 3) * a.np + p0 + i / 3];
}

hipError_t launch_read_vecs(const ReadArgs &a, int nvec, int p0, int n, hipStream_t s) {
    hipLaunchKernelGGL(k_read_vecs, dim3(blocks_for(3 * (int64_t)n, 256), (unsigned)nvec), dim3(256), 0, s, a, p0, n);
    return hipGetLastError();
}

hipError_t launch_list_q(const ForceArgs &a, double *out, hipStream_t s) {
    hipError_t e = launch_fill_u64((uint64_t *)out, 0ull, (int64_t)a.D * a.g.N, s);
    if (e != hipSuccess || a.P.np == 0) return e;
    if (a.D == 2) hipLaunchKernelGGL(k_list_q<2>, dim3((unsigned)a.P.np), dim3(128), 0, s, a, out);
    else hipLaunchKernelGGL(k_list_q<3>, dim3((unsigned)a.P.np), dim3(256), 0, s, a, out);
    return hipGetLastError();
}

hipError_t launch_cells(const CellArgs &a, hipStream_t s) {
    if (a.P.np == 0) return hipSuccess;
    hipError_t e = launch_fill_u32((uint32_t *)a.cell_count, 0u, (int64_t)a.ncx * a.ncy * a.ncz, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_cells, dim3(blocks_for(a.P.np, 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_dem(const CellArgs &a, hipStream_t s) {
    if (a.P.np == 0) return hipSuccess;
    if (many_discs(a.D, a.P.np))
        hipLaunchKernelGGL(k_dem_thread<128>, dim3(blocks_for(a.P.np, 128)), dim3(128), 0, s, a);
    else
        hipLaunchKernelGGL(k_dem, dim3(blocks_for(a.P.np, 4)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_nl_check(const CellArgs &a, hipStream_t s) {
    hipLaunchKernelGGL(k_nl_check, dim3(blocks_for(a.P.np, 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_nl_rebuild(const CellArgs &a, hipStream_t s) {
    if (a.P.np == 0) return hipSuccess;
    hipLaunchKernelGGL(k_nl_check, dim3(blocks_for(a.P.np, 256)), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_nl_cells, dim3(blocks_for(a.P.np, 256)), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_nl_build, dim3(blocks_for(a.P.np, 4)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_nl_contacts(const CellArgs &a, hipStream_t s) {
    if (a.P.np == 0) return hipSuccess;
    hipLaunchKernelGGL(k_dem_list, dim3(blocks_for(a.P.np, 256)), dim3(256), 0, s, a);
    const unsigned cb = (unsigned)std::min<int64_t>((a.ncell + 255) / 256, 4096);
    hipLaunchKernelGGL(k_nl_clear, dim3(cb), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_nl_finish, dim3(1), dim3(1), 0, s, a);
    return hipGetLastError();
}


}  // namespace lbimb
