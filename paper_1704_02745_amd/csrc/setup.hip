// System setup on the GPU (section 2.7 of the paper; Eq. 3 right-hand side).
//
// This file is compiled with -ffp-contract=off: the node classification,
// the edge means and the charge weights must round exactly as the plain
// (unfused) arithmetic they are defined by.
#include "solver.hpp"

#include <cmath>
#include <vector>

namespace pb {

namespace {

constexpr double kFourPi = 12.566370614359172;   // 4*pi rounded to double
constexpr double kCoulombKcal = 332.0637133;     // e^2/(4 pi eps0), kcal A/mol
constexpr int kMaxAtoms = (1 << 21) - 1;          // pair id = 8*atom + corner < 2^24
constexpr double kPeriodicMaxIndex = 268435456.0;  // 2^28: bound on |(c - o)/h| with the periodic boundary

__global__ void k_fill_u8(uint8_t* p, int64_t n, uint8_t v) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

__global__ void k_fill_i32(int* p, int64_t n, int v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_fill_u64(uint64_t* p, int64_t n, uint64_t v) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

// What the setup accumulates into, cleared in one launch: the flags word's 256
// bytes, the padded mask and the charge grid.
__global__ void k_setup_clear(int* __restrict__ flags, uint8_t* __restrict__ mask, int64_t nmask,
                              double* __restrict__ q, int64_t nn) {
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    if (t0 < 64) flags[t0] = 0;
    const int64_t words = ((uintptr_t)mask & 7) == 0 ? nmask / 8 : 0;   // a caller's mask may lie anywhere
    for (int64_t t = t0; t < words; t += step) reinterpret_cast<uint64_t*>(mask)[t] = 0;
    for (int64_t t = 8 * words + t0; t < nmask; t += step) mask[t] = 0;
    for (int64_t t = t0; t < nn; t += step) q[t] = 0.0;
}

// Node classification: one workgroup per atom walks the atom's bounding
// window of padded nodes and marks the ones strictly inside the sphere.
// Concurrent writers only ever store 1, so the result is order independent.
__device__ __forceinline__ void classify_atom(int64_t a, const double* __restrict__ xyz,
                                              const double* __restrict__ radius, int nx, int ny, int nz, double h,
                                              double ox, double oy, double oz, int per, uint8_t* __restrict__ mask) {
    const double cx = xyz[3 * a], cy = xyz[3 * a + 1], cz = xyz[3 * a + 2];
    const double r = radius[a];
    const double rr = r * r;
    const double o[3] = {ox, oy, oz};
    const double c[3] = {cx, cy, cz};
    const int n3[3] = {nx, ny, nz};
    int lo[3], hi[3];
    for (int d = 0; d < 3; ++d) {
        double l = floor((c[d] - r - o[d]) / h) - 1.0;
        double u = ceil((c[d] + r - o[d]) / h) + 1.0;
        if (per) {
            // periodic: the unwrapped window around the sphere (the nodes it
            // covers are marked at their wrapped index)
            if (!(fabs(l) < kPeriodicMaxIndex && fabs(u) < kPeriodicMaxIndex)) return;
        } else {
            l = fmin(fmax(l, -1.0), (double)n3[d]);
            u = fmin(fmax(u, -1.0), (double)n3[d]);
        }
        lo[d] = (int)l;
        hi[d] = (int)u;   // inclusive
    }
    const int wx = hi[0] - lo[0] + 1, wy = hi[1] - lo[1] + 1, wz = hi[2] - lo[2] + 1;
    if (wx <= 0 || wy <= 0 || wz <= 0) return;
    const int64_t total = (int64_t)wx * wy * wz;
    const int64_t px = nx + 2, py = ny + 2;
    for (int64_t t = threadIdx.x; t < total; t += blockDim.x) {
        const int i = lo[0] + (int)(t % wx);
        const int j = lo[1] + (int)((t / wx) % wy);
        const int k = lo[2] + (int)(t / ((int64_t)wx * wy));
        const double x = ox + h * (double)i;
        const double y = oy + h * (double)j;
        const double z = oz + h * (double)k;
        const double dx = x - cx, dy = y - cy, dz = z - cz;
        const double d2 = dx * dx + dy * dy + dz * dz;
        if (d2 < rr) {
            if (per) {
                const int iw = ((i % nx) + nx) % nx, jw = ((j % ny) + ny) % ny, kw = ((k % nz) + nz) % nz;
                mask[(iw + 1) + px * ((jw + 1) + py * (int64_t)(kw + 1))] = 1;
            } else {
                mask[(i + 1) + px * ((j + 1) + py * (int64_t)(k + 1))] = 1;
            }
        }
    }
}

__global__ void k_classify(const double* __restrict__ xyz, const double* __restrict__ radius, int64_t natoms, int nx,
                           int ny, int nz, double h, double ox, double oy, double oz, int per,
                           uint8_t* __restrict__ mask) {
    if (blockIdx.x < natoms) classify_atom(blockIdx.x, xyz, radius, nx, ny, nz, h, ox, oy, oz, per, mask);
}

// Periodic: fill the ghost layer of the padded mask with the wrapped nodes,
// one axis at a time (x, then y over whole padded rows, then z over whole
// padded planes) so edges and corners wrap too.
__global__ void k_wrap_ghosts(uint8_t* __restrict__ m, int nx, int ny, int nz, int axis) {
    const int64_t px = nx + 2, py = ny + 2, pz = nz + 2;
    const int64_t n = axis == 0 ? (int64_t)ny * nz : axis == 1 ? px * nz : px * py;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n;
         t += (int64_t)gridDim.x * blockDim.x) {
        if (axis == 0) {
            const int64_t j = 1 + t % ny, k = 1 + t / ny;
            uint8_t* row = m + px * (j + py * k);
            row[0] = row[nx];
            row[nx + 1] = row[1];
        } else if (axis == 1) {
            const int64_t i = t % px, k = 1 + t / px;
            uint8_t* col = m + i + px * py * k;
            col[0] = col[px * ny];
            col[px * (ny + 1)] = col[px];
        } else {
            const int64_t i = t % px, j = t / px;
            uint8_t* line = m + i + px * j;
            line[0] = line[px * py * nz];
            line[px * py * (pz - 1)] = line[px * py];
        }
    }
}

__device__ __forceinline__ double node_eps(uint8_t m, double ein, double eout) {
    return m ? ein : eout;
}

__device__ __forceinline__ double harmonic(double a, double b) {
    return 2.0 * a * b / (a + b);
}

// Staggered edge dielectrics, the salt term and (b given) the right-hand side
// 4*pi*q/h^3 plus, for nodes on the box faces, the ghost potential times the
// ghost-side edge dielectric over h^2 (x-, x+, y-, y+, z-, z+ in that order; none
// in a periodic box, which repeats). One thread per node and its three lower
// edges, and one past the last node of each axis for the upper ones. Bound by the
// writes: 257^3 in 0.25 ms, where a thread per element with 64-bit divisions and
// a pass of its own for the right-hand side took 0.32. An edge takes one of three
// values, so their divisions are done once per thread. I: an integer type that
// holds the thread count.
template <typename I>
__global__ void k_fields(const uint8_t* __restrict__ mask, int nx, int ny, int nz, double ein, double eout,
                         double kbar2, const double* __restrict__ q, const double* __restrict__ ghost, double h3,
                         double ih2, int per, double* __restrict__ ex, double* __restrict__ ey,
                         double* __restrict__ ez, double* __restrict__ k2, double* __restrict__ b) {
    const double hoo = harmonic(eout, eout), hio = harmonic(ein, eout), hii = harmonic(ein, ein);
    auto edge = [&](uint8_t m, uint8_t n) { return m && n ? hii : (m || n ? hio : hoo); };
    const int64_t px = nx + 2, pxy = px * (ny + 2);
    const I mx = (I)(nx + 1), my = (I)(ny + 1), total = mx * my * (I)(nz + 1);
    for (int64_t tt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; tt < (int64_t)total;
         tt += (int64_t)gridDim.x * blockDim.x) {
        const I t = (I)tt, row = t / mx, pk = row / my;
        const int i = (int)(t - row * mx), j = (int)(row - pk * my), k = (int)pk;
        const uint8_t* at = mask + (i + 1) + px * (j + 1) + pxy * (k + 1);
        const uint8_t m = at[0];
        const double exm = edge(at[-1], m), eym = edge(at[-px], m), ezm = edge(at[-pxy], m);
        const bool ix = i < nx, jy = j < ny, kz = k < nz;
        const int64_t yz = j + (int64_t)ny * k;
        if (jy && kz) ex[i + (nx + 1) * yz] = exm;
        if (ix && kz) ey[i + (int64_t)nx * (j + (int64_t)(ny + 1) * k)] = eym;
        if (ix && jy) ez[i + (int64_t)nx * yz] = ezm;
        if (!(ix && jy && kz)) continue;
        const int64_t n = i + (int64_t)nx * yz;
        k2[n] = m ? 0.0 : kbar2;
        if (!b) continue;
        const double charge = kFourPi * q[n] / h3;
        if (per) {
            b[n] = charge;
            continue;
        }
        const int64_t fx = (int64_t)ny * nz, fy = (int64_t)nx * nz, fz = (int64_t)nx * ny;
        const double* gy = ghost + 2 * fx;
        const double* gz = gy + 2 * fy;
        double fold = 0.0;
        if (i == 0) fold = fold + exm * ih2 * ghost[yz];
        if (i == nx - 1) fold = fold + edge(m, at[1]) * ih2 * ghost[fx + yz];
        if (j == 0) fold = fold + eym * ih2 * gy[i + (int64_t)nx * k];
        if (j == ny - 1) fold = fold + edge(m, at[px]) * ih2 * gy[fy + i + (int64_t)nx * k];
        if (k == 0) fold = fold + ezm * ih2 * gz[i + (int64_t)nx * j];
        if (k == nz - 1) fold = fold + edge(m, at[pxy]) * ih2 * gz[fz + i + (int64_t)nx * j];
        b[n] = charge + fold;
    }
}

// ---------------------------------------------------------------- fractional edges
//
// Weighted harmonic edge dielectric 1/(f/eps_in + (1-f)/eps_out), f the
// fraction of the edge segment inside the union of the spheres. Atoms are
// binned into cells of m*h (m = ceil(R_max/h)) over the padded node range;
// each edge visits the cells within R_max of its segment, clips each
// sphere's chord to [0,1] and keeps the union as a sorted list of disjoint
// segments (intervals that overlap or touch merge), whose lengths are summed
// in increasing order.
constexpr int kMaxSegments = 16;
// The device path of the fractional model is switched off: its first device
// run ended in a memory fault whose cause is not yet found (the same kernel
// text compiled for the host stays in bounds and matches the FP64 model bit
// for bit). pb_setup_ex refuses PB_EDGE_FRACTION while this is false.
constexpr bool kFractionEdgesEnabled = false;

__global__ __launch_bounds__(1024) void k_max_radius(const double* __restrict__ r, int64_t n, double* __restrict__ out) {
    __shared__ double s[1024];
    double m = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 1024) m = fmax(m, r[i]);
    s[threadIdx.x] = m;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s[threadIdx.x] = fmax(s[threadIdx.x], s[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = s[0];
}

__device__ __forceinline__ int padded_cell(double c, double o, double h, int n, int m) {
    double g = floor((c - o) / h) + 1.0;
    g = fmin(fmax(g, 0.0), (double)(n + 1));
    return (int)g / m;
}

// key = cell << 24 | atom (cells in x-fastest order over the padded nodes)
__global__ void k_cell_keys(const double* __restrict__ xyz, int64_t natoms, int nx, int ny, int nz, double h,
                            double ox, double oy, double oz, int m, int ncx, int ncy, uint64_t* __restrict__ keys) {
    const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= natoms) return;
    const int cx = padded_cell(xyz[3 * a], ox, h, nx, m);
    const int cy = padded_cell(xyz[3 * a + 1], oy, h, ny, m);
    const int cz = padded_cell(xyz[3 * a + 2], oz, h, nz, m);
    const uint64_t cell = (uint64_t)cx + (uint64_t)ncx * ((uint64_t)cy + (uint64_t)ncy * (uint64_t)cz);
    keys[a] = (cell << 24) | (uint64_t)a;
}

// first/last+1 sorted position of each cell's atoms (cells start empty)
__global__ void k_cell_bounds(const uint64_t* __restrict__ keys, int64_t natoms, int* __restrict__ start,
                              int* __restrict__ end) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= natoms) return;
    const uint64_t c = keys[p] >> 24;
    if (p == 0 || (keys[p - 1] >> 24) != c) start[c] = (int)p;
    if (p == natoms - 1 || (keys[p + 1] >> 24) != c) end[c] = (int)(p + 1);
}

__global__ void k_edges_fraction(const double* __restrict__ xyz, const double* __restrict__ radius,
                                 const uint64_t* __restrict__ keys, const int* __restrict__ cstart,
                                 const int* __restrict__ cend, int nx, int ny, int nz, double h, double ox, double oy,
                                 double oz, double rmax, int m, int ncx, int ncy, int ncz, double ein, double eout,
                                 double* __restrict__ ex, double* __restrict__ ey, double* __restrict__ ez,
                                 int* __restrict__ flags) {
    const int64_t nex = (int64_t)(nx + 1) * ny * nz;
    const int64_t ney = (int64_t)nx * (ny + 1) * nz;
    const int64_t nez = (int64_t)nx * ny * (nz + 1);
    const int64_t total = nex + ney + nez;
    const double o[3] = {ox, oy, oz};
    const int n3[3] = {nx, ny, nz};
    const int nc[3] = {ncx, ncy, ncz};
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
         t += (int64_t)gridDim.x * blockDim.x) {
        int axis, idx[3];
        double* outp;
        if (t < nex) {
            axis = 0;
            idx[0] = (int)(t % (nx + 1)) - 1; idx[1] = (int)((t / (nx + 1)) % ny); idx[2] = (int)(t / ((int64_t)(nx + 1) * ny));
            outp = ex + t;
        } else if (t < nex + ney) {
            const int64_t u = t - nex;
            axis = 1;
            idx[0] = (int)(u % nx); idx[1] = (int)((u / nx) % (ny + 1)) - 1; idx[2] = (int)(u / ((int64_t)nx * (ny + 1)));
            outp = ey + u;
        } else {
            const int64_t u = t - nex - ney;
            axis = 2;
            idx[0] = (int)(u % nx); idx[1] = (int)((u / nx) % ny); idx[2] = (int)(u / ((int64_t)nx * ny)) - 1;
            outp = ez + u;
        }
        double p[3];
        for (int d = 0; d < 3; ++d) p[d] = o[d] + h * (double)idx[d];   // the edge's first node
        int clo[3], chi[3];
        for (int d = 0; d < 3; ++d) {
            const double lo = p[d] - rmax, hi = p[d] + (d == axis ? h : 0.0) + rmax;
            clo[d] = padded_cell(lo, o[d], h, n3[d], m);
            chi[d] = min(padded_cell(hi, o[d], h, n3[d], m), nc[d] - 1);
        }
        double s0[kMaxSegments], s1[kMaxSegments];
        int ns = 0;
        bool overflow = false;
        for (int cz = clo[2]; cz <= chi[2]; ++cz)
            for (int cy = clo[1]; cy <= chi[1]; ++cy)
                for (int cx = clo[0]; cx <= chi[0]; ++cx) {
                    const int64_t cell = (int64_t)cx + (int64_t)ncx * ((int64_t)cy + (int64_t)ncy * cz);
                    for (int q = cstart[cell]; q < cend[cell]; ++q) {
                        const int64_t a = (int64_t)(keys[q] & 0xFFFFFFull);
                        const double c[3] = {xyz[3 * a], xyz[3 * a + 1], xyz[3 * a + 2]};
                        const double R = radius[a];
                        const double RR = R * R;
                        double d2 = 0.0;
                        for (int d = 0; d < 3; ++d) {
                            if (d == axis) continue;
                            const double dd = p[d] - c[d];
                            d2 = d2 + dd * dd;
                        }
                        if (!(d2 < RR)) continue;
                        const double w = sqrt(RR - d2);
                        double t0 = ((c[axis] - w) - p[axis]) / h;
                        double t1 = ((c[axis] + w) - p[axis]) / h;
                        t0 = fmax(t0, 0.0);
                        t1 = fmin(t1, 1.0);
                        if (!(t1 > t0)) continue;
                        // insert into the sorted disjoint union (merge what overlaps or touches)
                        int i = 0;
                        while (i < ns && s1[i] < t0) ++i;          // segments entirely before
                        int j = i;
                        double a0 = t0, a1 = t1;
                        while (j < ns && s0[j] <= a1) {            // segments touching [a0, a1]
                            a0 = fmin(a0, s0[j]);
                            a1 = fmax(a1, s1[j]);
                            ++j;
                        }
                        const int removed = j - i;
                        if (removed == 0) {
                            if (ns == kMaxSegments) { overflow = true; continue; }
                            for (int k = ns; k > i; --k) { s0[k] = s0[k - 1]; s1[k] = s1[k - 1]; }
                            ++ns;
                        } else if (removed > 1) {
                            for (int k = i + 1; k + removed - 1 < ns; ++k) {
                                s0[k] = s0[k + removed - 1];
                                s1[k] = s1[k + removed - 1];
                            }
                            ns -= removed - 1;
                        }
                        s0[i] = a0;
                        s1[i] = a1;
                    }
                }
        if (overflow) atomicOr(flags, 4);
        double f = 0.0;
        for (int i = 0; i < ns; ++i) f = f + (s1[i] - s0[i]);
        *outp = (f == 0.0) ? eout : (f == 1.0) ? ein : 1.0 / (f / ein + (1.0 - f) / eout);
    }
}

// Trilinear cell of one atom along one axis: i0 = clamp(floor(g), 0, n-2),
// f = g - i0. Periodic: i0 = floor(g) mod n, f = g - floor(g) (the second
// node of the cell is (i0 + 1) mod n).
__device__ __forceinline__ bool cell_axis(double c, double o, double h, int n, int per, int& i0, double& f) {
    const double g = (c - o) / h;
    if (per) {
        if (!(fabs(g) < kPeriodicMaxIndex)) return false;
        const double fl = floor(g);
        f = g - fl;
        const long long w = (long long)fl % n;
        i0 = (int)(w < 0 ? w + n : w);
        return true;
    }
    if (!(g >= 0.0) || !(g <= (double)(n - 1))) return false;
    double fl = floor(g);
    fl = fmin(fmax(fl, 0.0), (double)(n - 2));
    i0 = (int)fl;
    f = g - fl;
    return true;
}

// Node index of corner c (bit 0: +x, bit 1: +y, bit 2: +z) of a cell.
__device__ __forceinline__ int64_t corner_node(int i0, int j0, int k0, int c, int nx, int ny, int nz) {
    int i = i0 + (c & 1), j = j0 + ((c >> 1) & 1), k = k0 + ((c >> 2) & 1);
    if (i == nx) i = 0;   // only reached with the periodic cell
    if (j == ny) j = 0;
    if (k == nz) k = 0;
    return (int64_t)i + (int64_t)nx * ((int64_t)j + (int64_t)ny * k);
}

// Charge spreading, step 1: one sort key per (atom, corner) pair,
// key = node_index << 24 | (8*atom + corner). Sorting the keys groups the
// contributions of each node in increasing atom order. Past the pairs, and for
// an atom outside the box: all ones.
__device__ __forceinline__ uint64_t spread_key(int64_t p, const double* __restrict__ xyz, int64_t natoms, int nx,
                                               int ny, int nz, double h, double ox, double oy, double oz, int per,
                                               int* __restrict__ flags) {
    if (p >= 8 * natoms) return ~0ull;
    const int64_t a = p >> 3;
    const int c = (int)(p & 7);
    int i0, j0, k0;
    double fx, fy, fz;
    bool ok = cell_axis(xyz[3 * a], ox, h, nx, per, i0, fx);
    ok = cell_axis(xyz[3 * a + 1], oy, h, ny, per, j0, fy) && ok;
    ok = cell_axis(xyz[3 * a + 2], oz, h, nz, per, k0, fz) && ok;
    if (!ok) {
        atomicOr(flags, 1);
        return ~0ull;
    }
    return ((uint64_t)corner_node(i0, j0, k0, c, nx, ny, nz) << 24) | (uint64_t)p;
}
__global__ void k_spread_keys(const double* __restrict__ xyz, int64_t natoms, int nx, int ny, int nz,
                              double h, double ox, double oy, double oz, int per,
                              uint64_t* __restrict__ keys, int64_t n, int* __restrict__ flags) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) keys[p] = spread_key(p, xyz, natoms, nx, ny, nz, h, ox, oy, oz, per, flags);
}

// One compare-exchange step of a bitonic sorting network (ascending).
__global__ void k_bitonic_step(uint64_t* __restrict__ a, int64_t n, int64_t j, int64_t k) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t l = i ^ j;
    if (l > i) {
        const uint64_t x = a[i], y = a[l];
        const bool up = (i & k) == 0;
        if ((x > y) == up) {
            a[i] = y;
            a[l] = x;
        }
    }
}

// The steps of the same network whose pairs lie within one aligned chunk of
// kSortChunk keys (j < kSortChunk), in LDS: block b sorts chunk b through
// stages k_first..k_last (powers of two), starting stage k_first at j_first.
// The keys are distinct, so any correct sort leaves the same order.
constexpr int kSortChunk = 2048;
__global__ __launch_bounds__(1024) void k_bitonic_local(uint64_t* __restrict__ a, int64_t n, int64_t k_first,
                                                        int64_t k_last, int64_t j_first) {
    __shared__ uint64_t s[kSortChunk];
    const int chunk = (int)min<int64_t>(n, kSortChunk);
    const int64_t base = (int64_t)blockIdx.x * chunk;
    for (int e = threadIdx.x; e < chunk; e += blockDim.x) s[e] = a[base + e];
    __syncthreads();
    for (int64_t k = k_first; k <= k_last; k <<= 1) {
        for (int64_t j = (k == k_first) ? j_first : (k >> 1); j > 0; j >>= 1) {
            for (int e = threadIdx.x; e < chunk; e += blockDim.x) {
                const int le = e ^ (int)j;
                if (le > e) {
                    const uint64_t x = s[e], y = s[le];
                    const bool up = ((base + e) & k) == 0;
                    if ((x > y) == up) {
                        s[e] = y;
                        s[le] = x;
                    }
                }
            }
            __syncthreads();
        }
    }
    for (int e = threadIdx.x; e < chunk; e += blockDim.x) a[base + e] = s[e];
}

// Charge spreading, step 2: the first key of each node's run sums the run in
// key order (increasing atom index), starting from zero, and stores q_node.
__device__ __forceinline__ void spread_run(const uint64_t* keys, int64_t i, int64_t npairs,
                                           const double* __restrict__ xyz, const double* __restrict__ charge, int nx,
                                           int ny, int nz, double h, double ox, double oy, double oz, int per,
                                           double* __restrict__ q) {
    const uint64_t key = keys[i];
    if (key == ~0ull) return;
    const uint64_t node = key >> 24;
    if (i > 0 && (keys[i - 1] >> 24) == node) return;
    double s = 0.0;
    for (int64_t t = i; t < npairs; ++t) {
        const uint64_t kt = keys[t];
        if (kt == ~0ull || (kt >> 24) != node) break;
        const int64_t p = (int64_t)(kt & 0xFFFFFFull);
        const int64_t a = p >> 3;
        const int c = (int)(p & 7);
        int i0, j0, k0;
        double fx, fy, fz;
        cell_axis(xyz[3 * a], ox, h, nx, per, i0, fx);
        cell_axis(xyz[3 * a + 1], oy, h, ny, per, j0, fy);
        cell_axis(xyz[3 * a + 2], oz, h, nz, per, k0, fz);
        const double wx = (c & 1) ? fx : 1.0 - fx;
        const double wy = (c & 2) ? fy : 1.0 - fy;
        const double wz = (c & 4) ? fz : 1.0 - fz;
        s = s + charge[a] * wx * wy * wz;
    }
    q[node] = s;
}
__global__ void k_spread_sum(const uint64_t* __restrict__ keys, int64_t npairs,
                             const double* __restrict__ xyz, const double* __restrict__ charge,
                             int nx, int ny, int nz, double h, double ox, double oy, double oz, int per,
                             double* __restrict__ q) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < npairs) spread_run(keys, i, npairs, xyz, charge, nx, ny, nz, h, ox, oy, oz, per, q);
}
// Both steps for up to kSortChunk keys by one workgroup, the keys in LDS: n keys
// (a power of two >= 2), the same network with one pair per thread and turn.
__device__ __forceinline__ void spread_small(uint64_t* s, int n, const double* __restrict__ xyz,
                                             const double* __restrict__ charge, int64_t natoms, int nx, int ny, int nz,
                                             double h, double ox, double oy, double oz, int per,
                                             double* __restrict__ q, int* __restrict__ flags) {
    for (int p = threadIdx.x; p < n; p += blockDim.x)
        s[p] = spread_key(p, xyz, natoms, nx, ny, nz, h, ox, oy, oz, per, flags);
    for (int k = 2; k <= n; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            __syncthreads();
            for (int t = threadIdx.x; t < n / 2; t += blockDim.x) {
                const int e = ((t & ~(j - 1)) << 1) | (t & (j - 1));
                const uint64_t x = s[e], y = s[e + j];
                if ((x > y) == ((e & k) == 0)) {
                    s[e] = y;
                    s[e + j] = x;
                }
            }
        }
    __syncthreads();
    for (int i = threadIdx.x; i < 8 * (int)natoms; i += blockDim.x)
        spread_run(s, i, 8 * natoms, xyz, charge, nx, ny, nz, h, ox, oy, oz, per, q);
}

// Ghost point `t` of the six faces (x-, x+, y-, y+, z-, z+), in that order;
// within a face the faster index comes first (y then z, x then z, x then y).
__device__ __forceinline__ void ghost_point(int64_t t, int nx, int ny, int nz, double h,
                                            double ox, double oy, double oz,
                                            double& px, double& py, double& pz) {
    const int64_t fx = (int64_t)ny * nz, fy = (int64_t)nx * nz;
    if (t < 2 * fx) {
        const int side = t >= fx;
        const int64_t u = t - side * fx;
        px = ox + h * (side ? (double)nx : -1.0);
        py = oy + h * (double)(u % ny);
        pz = oz + h * (double)(u / ny);
    } else if (t < 2 * fx + 2 * fy) {
        const int64_t v = t - 2 * fx;
        const int side = v >= fy;
        const int64_t u = v - side * fy;
        px = ox + h * (double)(u % nx);
        py = oy + h * (side ? (double)ny : -1.0);
        pz = oz + h * (double)(u / nx);
    } else {
        const int64_t fz = (int64_t)nx * ny;
        const int64_t v = t - 2 * fx - 2 * fy;
        const int side = v >= fz;
        const int64_t u = v - side * fz;
        px = ox + h * (double)(u % nx);
        py = oy + h * (double)(u / nx);
        pz = oz + h * (side ? (double)nz : -1.0);
    }
}

// Debye-Hueckel potential on the face ghosts: each thread owns one ghost
// point and sums over all atoms in index order; atoms are staged in LDS.
// This is the arithmetic-bound part of setup (6 n^2 points x natoms terms).
constexpr int kDhBlock = 256;
// 1/sqrt(r2) for r2 > 0: the hardware estimate and two Newton steps,
// y <- y (1 + (1 - r2 y^2)/2), each roughly doubling the correct bits.
__device__ __forceinline__ double rsqrt_nr(double r2) {
    // the hardware estimate, then two Newton steps y += y (1/2 - (r2/2) y^2)
    const double h = 0.5 * r2;
    double y = __builtin_amdgcn_rsq(r2);
    y = fma(y, fma(-(h * y), y, 0.5), y);
    y = fma(y, fma(-(h * y), y, 0.5), y);
    return y;
}

// 2^(j/64), j = 0..63, each the double nearest to the exact value.
constexpr int kExpTab = 64;
__constant__ double kExp2Frac[kExpTab] = {
    0x1.0000000000000p+0, 0x1.02c9a3e778061p+0, 0x1.059b0d3158574p+0, 0x1.0874518759bc8p+0,
    0x1.0b5586cf9890fp+0, 0x1.0e3ec32d3d1a2p+0, 0x1.11301d0125b51p+0, 0x1.1429aaea92de0p+0,
    0x1.172b83c7d517bp+0, 0x1.1a35beb6fcb75p+0, 0x1.1d4873168b9aap+0, 0x1.2063b88628cd6p+0,
    0x1.2387a6e756238p+0, 0x1.26b4565e27cddp+0, 0x1.29e9df51fdee1p+0, 0x1.2d285a6e4030bp+0,
    0x1.306fe0a31b715p+0, 0x1.33c08b26416ffp+0, 0x1.371a7373aa9cbp+0, 0x1.3a7db34e59ff7p+0,
    0x1.3dea64c123422p+0, 0x1.4160a21f72e2ap+0, 0x1.44e086061892dp+0, 0x1.486a2b5c13cd0p+0,
    0x1.4bfdad5362a27p+0, 0x1.4f9b2769d2ca7p+0, 0x1.5342b569d4f82p+0, 0x1.56f4736b527dap+0,
    0x1.5ab07dd485429p+0, 0x1.5e76f15ad2148p+0, 0x1.6247eb03a5585p+0, 0x1.6623882552225p+0,
    0x1.6a09e667f3bcdp+0, 0x1.6dfb23c651a2fp+0, 0x1.71f75e8ec5f74p+0, 0x1.75feb564267c9p+0,
    0x1.7a11473eb0187p+0, 0x1.7e2f336cf4e62p+0, 0x1.82589994cce13p+0, 0x1.868d99b4492edp+0,
    0x1.8ace5422aa0dbp+0, 0x1.8f1ae99157736p+0, 0x1.93737b0cdc5e5p+0, 0x1.97d829fde4e50p+0,
    0x1.9c49182a3f090p+0, 0x1.a0c667b5de565p+0, 0x1.a5503b23e255dp+0, 0x1.a9e6b5579fdbfp+0,
    0x1.ae89f995ad3adp+0, 0x1.b33a2b84f15fbp+0, 0x1.b7f76f2fb5e47p+0, 0x1.bcc1e904bc1d2p+0,
    0x1.c199bdd85529cp+0, 0x1.c67f12e57d14bp+0, 0x1.cb720dcef9069p+0, 0x1.d072d4a07897cp+0,
    0x1.d5818dcfba487p+0, 0x1.da9e603db3285p+0, 0x1.dfc97337b9b5fp+0, 0x1.e502ee78b3ff6p+0,
    0x1.ea4afa2a490dap+0, 0x1.efa1bee615a27p+0, 0x1.f50765b6e4540p+0, 0x1.fa7c1819e90d8p+0,
};

// e^x for x <= 0 (the screening factor e^(-kappa d)), without the range
// checks of a general exponential, with `tab` the table above (an LDS copy
// on the device). Tang's table-driven reduction: x = (64 n + j) ln2/64 + r,
// |r| <= ln2/128, so e^x = 2^n 2^(j/64) e^r. ln2/64 is taken in two parts, a
// head with 32 significant bits (n * head is exact for any n this range
// gives) and the rounded remainder. e^r - 1 is the Taylor series to degree
// 5, whose truncation is below 4e-17 relative on that interval; the result
// is 2^(j/64) + 2^(j/64) (e^r - 1) in one rounding, and ldexp applies 2^n
// (rounding results below the normal range as they underflow).
__device__ __forceinline__ double exp_nonpos(double x, const double* tab) {
    constexpr double k64InvLn2 = 92.332482616893658;
    constexpr double kHead = 0x1.62e42fee00000p-7;
    constexpr double kTail = 0x1.a39ef35793c76p-39;
    const double fk = rint(x * k64InvLn2);
    const int k = (int)fk;
    const double r = fma(-fk, kTail, fma(-fk, kHead, x));
    const double r2 = r * r;
    double p = fma(r, 1.0 / 120.0, 1.0 / 24.0);
    p = fma(p, r, 1.0 / 6.0);
    p = fma(p, r, 0.5);
    const double em1 = fma(p, r2, r);
    const double t = tab[k & (kExpTab - 1)];
    return ldexp(fma(t, em1, t), k >> 6);
}

// Screened Coulomb sum of every atom at each ghost-face point, atoms in
// index order through LDS records (x, y, z, q): phi = (1/eps_out) sum q e^(-kd)/d.
// Ghost points lie one node outside the box and atoms inside it, so d >= h > 0.
__device__ __forceinline__ void dh_direct_block(
        int64_t block, const double* __restrict__ xyz, const double* __restrict__ charge, int64_t natoms,
        int nx, int ny, int nz, double h, double ox, double oy, double oz,
        double kd, double eout, double* __restrict__ ghost, int64_t nghost) {
    __shared__ double4 sa[kDhBlock];
    __shared__ double s_tab[kExpTab];
    if (threadIdx.x < kExpTab) s_tab[threadIdx.x] = kExp2Frac[threadIdx.x];
    const int64_t t = block * kDhBlock + threadIdx.x;
    double px = 0, py = 0, pz = 0;
    if (t < nghost) ghost_point(t, nx, ny, nz, h, ox, oy, oz, px, py, pz);
    double s = 0.0;
    for (int64_t a0 = 0; a0 < natoms; a0 += kDhBlock) {
        __syncthreads();
        const int64_t a = a0 + threadIdx.x;
        if (a < natoms) sa[threadIdx.x] = make_double4(xyz[3 * a], xyz[3 * a + 1], xyz[3 * a + 2], charge[a]);
        __syncthreads();
        const int m = (int)min<int64_t>(kDhBlock, natoms - a0);
        if (kd == 0.0) {
#pragma unroll 4
            for (int b = 0; b < m; ++b) {
                const double4 c = sa[b];
                const double dx = px - c.x, dy = py - c.y, dz = pz - c.z;
                const double y = rsqrt_nr(dx * dx + dy * dy + dz * dz);
                s = fma(c.w, y, s);
            }
        } else {
#pragma unroll 4
            for (int b = 0; b < m; ++b) {
                const double4 c = sa[b];
                const double dx = px - c.x, dy = py - c.y, dz = pz - c.z;
                const double r2 = dx * dx + dy * dy + dz * dz;
                const double y = rsqrt_nr(r2);
                s = fma(c.w * exp_nonpos(-kd * (r2 * y), s_tab), y, s);
            }
        }
    }
    if (t < nghost) ghost[t] = s / eout;
}

__global__ __launch_bounds__(kDhBlock) void k_dh_faces(
        const double* __restrict__ xyz, const double* __restrict__ charge, int64_t natoms,
        int nx, int ny, int nz, double h, double ox, double oy, double oz,
        double kd, double eout, double* __restrict__ ghost, int64_t nghost) {
    dh_direct_block(blockIdx.x, xyz, charge, natoms, nx, ny, nz, h, ox, oy, oz, kd, eout, ghost, nghost);
}

// The parts of a small molecule's setup that need nothing of one another, in
// one launch: workgroup 0 spreads the charges (up to kSortChunk keys), one per
// atom classifies nodes, the rest take the boundary sum. Each is a chain of
// latencies that leaves the device idle: 33^3 with 50 atoms, 11 launches and
// 118 us in all before, 61 with this (3 launches).
__global__ __launch_bounds__(kDhBlock) void k_setup_small(
        const double* __restrict__ xyz, const double* __restrict__ radius, const double* __restrict__ charge,
        int natoms, int nkeys, int nx, int ny, int nz, double h, double ox, double oy, double oz, int per, double kd,
        double eout, uint8_t* __restrict__ mask, double* __restrict__ q, int* __restrict__ flags,
        double* __restrict__ ghost, int64_t nghost) {
    __shared__ uint64_t s_keys[kSortChunk];
    const int block = (int)blockIdx.x;
    if (block == 0) spread_small(s_keys, nkeys, xyz, charge, natoms, nx, ny, nz, h, ox, oy, oz, per, q, flags);
    else if (block <= natoms) classify_atom(block - 1, xyz, radius, nx, ny, nz, h, ox, oy, oz, per, mask);
    else dh_direct_block(block - 1 - natoms, xyz, charge, natoms, nx, ny, nz, h, ox, oy, oz, kd, eout, ghost, nghost);
}
// Whether it is the faster form, a direct boundary sum provided: the keys fit the
// LDS, and its one workgroup, whose threads sum the charges of up to eight nodes one
// after another, is done with them soon. Where many share a node it is not (256 atoms
// on 7^3 nodes: 237 us against 191; 200 on 7^3, 128 on 5^3: equal), and in a
// periodic box, which has no boundary sum beside it, not with many keys on few
// nodes (256 atoms, 12^3: 173 us against 152, 25^3: 156 against 152, 33^3: 148 against
// 164; 128 atoms, 9^3: 132 against 126, 12^3: equal, 20^3: 116 against 126).
bool setup_in_one(int64_t nkeys, int64_t natoms, int64_t nn, bool per) {
    const int64_t per_atom = !per || nkeys <= 512 ? 2 : (nkeys <= 1024 ? 16 : 128);   // nodes, at least
    return nkeys <= kSortChunk && per_atom * natoms <= nn;
}

// ---- the same sum with interpolated far fields
//
// The direct sum is bound by FP64 issue (about 36 slots a term, 7.9e9 terms at
// 257^3 with 20,000 atoms: 11.0 ms), so the number of terms has to fall. Seen
// from an atom at some distance the field is smooth over a tile of a face:
// it is summed at 32 x 32 Chebyshev points of the tile instead of every node,
// and carried to the nodes by the Lagrange polynomials. Two levels: tiles of up
// to 130 nodes a side, and their quarters. An atom goes to the largest tile
// over a node that it is far enough from, and to the node itself where it is
// far enough from neither; which one is a test of the atom against the tile, so
// every atom counts once at every node, in one fixed order.
//
// Far enough: along a line of the tile of half-length w the field of an atom
// is analytic inside the ellipse with foci at the line's ends on which the atom's
// image lies, and 32 points leave an error of rho^-32, rho the ellipse's
// parameter. With m the least distance from the atom to the midpoints of the
// tile's lines (both directions), m >= 1.5 w makes that 2e-15 of the field's
// maximum over the tile; the screening factor grows off the real line, which
// 0.1 kappa w more makes up for (measured against direct evaluation, atoms at
// exactly that distance: 1.9e-15 at kappa w = 0, 2.1e-15 at 2, 3.1e-15 at 4.5). A
// level whose tiles are wider than kappa w = 4.5, or hold fewer than 1.5 times as
// many nodes as points, is not used.
//
// The points bound it (1.3 ms of 1.63 at 257^3): the same FP64 issue, a sixth of
// the terms. Measured: the whole preparation of 257^3 with 20,000 atoms 11.7 -> 2.4 ms,
// 193 x 177 x 161 with 8,000 2.26 -> 0.87 ms; against the exact sum the faces are
// nearer than the direct sum's (largest error 1.8e-15 of the largest value, 1.2e-14
// before).
constexpr int kDhP = 32;                   // Chebyshev points per tile and direction
constexpr int kDhPoints = kDhP * kDhP;
constexpr int kDhTile = 130;               // largest tile of the first level, nodes per side
constexpr double kDhFar = 1.5, kDhFarKappa = 0.1, kDhMaxKappaW = 4.5;
constexpr int kDhRows = 16;                // node rows per block of the interpolation

struct DhFace {
    int axis, side;        // normal axis; 0: low, 1: high face
    int nu, nv;            // nodes along the fast and the slow direction
    int ku, kv;            // first-level tiles; 2 ku x 2 kv of the second
    int on1, on2;          // levels in use
    int tile0;             // first tile of the face in the array of points (first level, then second)
    int64_t ghost0;        // first ghost point
};
struct DhPlan {
    DhFace f[6];
    int tiles;             // tiles of the used levels
    int tiles2;            // second-level tiles of all faces, used or not
    int chunks;            // atom ranges summed by blocks of their own
    int nx, ny, nz;
    double h, ox, oy, oz, kd;
};

// Tile (i, j) of a face's level: node ranges, and centre and half-width in node
// indices along each direction.
struct DhTile {
    int u0, u1, v0, v1;
    double cu, cv, wu, wv;
};
__host__ __device__ __forceinline__ DhTile dh_tile(const DhFace& f, int level, int i, int j) {
    const int ku = f.ku * level, kv = f.kv * level;   // level 1 or 2
    DhTile t;
    t.u0 = (int)((int64_t)i * f.nu / ku);
    t.u1 = (int)((int64_t)(i + 1) * f.nu / ku);
    t.v0 = (int)((int64_t)j * f.nv / kv);
    t.v1 = (int)((int64_t)(j + 1) * f.nv / kv);
    t.cu = 0.5 * (t.u0 + t.u1 - 1);
    t.cv = 0.5 * (t.v0 + t.v1 - 1);
    t.wu = 0.5 * (t.u1 - 1 - t.u0);
    t.wv = 0.5 * (t.v1 - 1 - t.v0);
    return t;
}
__device__ __forceinline__ void dh_face_axes(const DhPlan& P, const DhFace& f, double& ou, double& ov, double& on) {
    ou = f.axis == 0 ? P.oy : P.ox;
    ov = f.axis == 2 ? P.oy : P.oz;
    const double o = f.axis == 0 ? P.ox : (f.axis == 1 ? P.oy : P.oz);
    const int n = f.axis == 0 ? P.nx : (f.axis == 1 ? P.ny : P.nz);
    on = o + P.h * (f.side ? (double)n : -1.0);
}
// Whether an atom at (u, v, n) from the tile's centre is far enough (see above).
__device__ __forceinline__ bool dh_far(double u, double v, double n, double wu, double wv, double kd) {
    const double eu = fmax(fabs(u) - wu, 0.0), ev = fmax(fabs(v) - wv, 0.0), n2 = n * n;
    const double fu = (kDhFar + kDhFarKappa * kd * wu) * wu, fv = (kDhFar + kDhFarKappa * kd * wv) * wv;
    return n2 + u * u + ev * ev >= fu * fu && n2 + v * v + eu * eu >= fv * fv;
}

// The terms of the atoms [a0, a1) that belong to this block's points: level 1
// and 2 the tile's Chebyshev points, 0 its nodes. Atoms are taken 256 at a time,
// tested one per thread and packed into LDS in index order; they are summed when
// another 256 might not fit.
constexpr int kDhBatch = 512;   // atoms packed before they are summed
struct DhSum {
    double4 atom[kDhBatch];
    double tab[kExpTab];
    int count[kDhBlock / 64];
};
__device__ __forceinline__ double dh_block_sum(const DhPlan& P, const DhFace& f, const DhTile& t1, const DhTile& t2,
                                               int level, double px, double py, double pz,
                                               const double* __restrict__ xyz, const double* __restrict__ charge,
                                               int64_t a0, int64_t a1, DhSum& s) {
    if (threadIdx.x < kExpTab) s.tab[threadIdx.x] = kExp2Frac[threadIdx.x];
    double ou, ov, on;
    dh_face_axes(P, f, ou, ov, on);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double sum = 0.0;
    int m = 0;   // packed so far
    for (int64_t base = a0; base < a1; base += kDhBlock) {
        const int64_t a = base + threadIdx.x;
        bool take = false;
        double4 c = make_double4(0.0, 0.0, 0.0, 0.0);
        if (a < a1) {
            c = make_double4(xyz[3 * a], xyz[3 * a + 1], xyz[3 * a + 2], charge[a]);
            const double u = f.axis == 0 ? c.y : c.x, v = f.axis == 2 ? c.y : c.z;
            const double n = (f.axis == 0 ? c.x : (f.axis == 1 ? c.y : c.z)) - on;
            const bool far1 = f.on1 && dh_far(u - (ou + P.h * t1.cu), v - (ov + P.h * t1.cv), n, P.h * t1.wu,
                                              P.h * t1.wv, P.kd);
            const bool far2 = f.on2 && !far1 && level != 1 &&
                              dh_far(u - (ou + P.h * t2.cu), v - (ov + P.h * t2.cv), n, P.h * t2.wu, P.h * t2.wv, P.kd);
            take = level == 1 ? far1 : (level == 2 ? far2 : !far1 && !far2);
        }
        const unsigned long long mask = __ballot(take);
        __syncthreads();   // the counts and records before are no longer read
        if (lane == 0) s.count[wave] = __popcll(mask);
        __syncthreads();
        int at = m + __popcll(mask & ((1ull << lane) - 1));
#pragma unroll
        for (int w = 0; w < kDhBlock / 64; ++w) {
            if (w < wave) at += s.count[w];
            m += s.count[w];
        }
        if (take) s.atom[at] = c;
        if (m <= kDhBatch - kDhBlock && base + kDhBlock < a1) continue;   // room for another 256
        __syncthreads();
        if (P.kd == 0.0) {
#pragma unroll 4
            for (int b = 0; b < m; ++b) {
                const double4 q = s.atom[b];
                const double dx = px - q.x, dy = py - q.y, dz = pz - q.z;
                sum = fma(q.w, rsqrt_nr(dx * dx + dy * dy + dz * dz), sum);
            }
        } else {
#pragma unroll 4
            for (int b = 0; b < m; ++b) {
                const double4 q = s.atom[b];
                const double dx = px - q.x, dy = py - q.y, dz = pz - q.z;
                const double r2 = dx * dx + dy * dy + dz * dz;
                const double y = rsqrt_nr(r2);
                sum = fma(q.w * exp_nonpos(-P.kd * (r2 * y), s.tab), y, sum);
            }
        }
        m = 0;
    }
    return sum;
}

__device__ __forceinline__ void dh_position(const DhPlan& P, const DhFace& f, double iu, double iv, double& px,
                                            double& py, double& pz) {
    double ou, ov, on;
    dh_face_axes(P, f, ou, ov, on);
    const double u = ou + P.h * iu, v = ov + P.h * iv;
    px = f.axis == 0 ? on : u;
    py = f.axis == 1 ? on : (f.axis == 0 ? u : v);
    pz = f.axis == 2 ? on : v;
}

// Sums at the Chebyshev points: blocks of 256 points, four per tile, by atom
// ranges (blockIdx.y) so that a few tiles fill the device.
__global__ __launch_bounds__(kDhBlock) void k_dh_points(DhPlan P, const double* __restrict__ xyz,
                                                        const double* __restrict__ charge, int64_t natoms,
                                                        double* __restrict__ partial) {
    __shared__ DhSum s;
    const int tile = blockIdx.x / (kDhPoints / kDhBlock);
    const int pt = (blockIdx.x % (kDhPoints / kDhBlock)) * kDhBlock + threadIdx.x;
    int fi = 0;
    for (int k = 1; k < 6; ++k)
        if ((P.f[k].on1 || P.f[k].on2) && tile >= P.f[k].tile0) fi = k;
    const DhFace f = P.f[fi];
    int t = tile - f.tile0;
    const int n1 = f.on1 ? f.ku * f.kv : 0;
    const int level = t < n1 ? 1 : 2;
    DhTile t1, t2{};
    if (level == 1) {
        t1 = dh_tile(f, 1, t % f.ku, t / f.ku);
    } else {
        t -= n1;
        const int i = t % (2 * f.ku), j = t / (2 * f.ku);
        t1 = dh_tile(f, 1, i / 2, j / 2);
        t2 = dh_tile(f, 2, i, j);
    }
    const DhTile& T = level == 1 ? t1 : t2;
    const int ca = pt % kDhP, cb = pt / kDhP;
    double px, py, pz;
    dh_position(P, f, T.cu + T.wu * cospi((2 * ca + 1) / (2.0 * kDhP)), T.cv + T.wv * cospi((2 * cb + 1) / (2.0 * kDhP)),
                px, py, pz);
    const int64_t per = (natoms + gridDim.y - 1) / gridDim.y;
    const int64_t a0 = min((int64_t)blockIdx.y * per, natoms), a1 = min(a0 + per, natoms);
    partial[((int64_t)blockIdx.y * P.tiles + tile) * kDhPoints + pt] =
        dh_block_sum(P, f, t1, t2, level, px, py, pz, xyz, charge, a0, a1, s);
}

// The ranges' sums in order.
__global__ void k_dh_collect(const double* __restrict__ partial, int chunks, int64_t n, double* __restrict__ c) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    double v = partial[t];
    for (int k = 1; k < chunks; ++k) v += partial[k * n + t];
    c[t] = v;
}

__device__ __forceinline__ const DhFace& dh_face_of_tile2(const DhPlan& P, int tile2, int& i, int& j) {
    int k = 0;
    for (; k < 5; ++k) {
        const int n = 4 * P.f[k].ku * P.f[k].kv;
        if (tile2 < n) break;
        tile2 -= n;
    }
    i = tile2 % (2 * P.f[k].ku);
    j = tile2 / (2 * P.f[k].ku);
    return P.f[k];
}

// Near atoms, node by node: block (tile of the second level, 256 of its nodes).
__global__ __launch_bounds__(kDhBlock) void k_dh_near(DhPlan P, const double* __restrict__ xyz,
                                                      const double* __restrict__ charge, int64_t natoms,
                                                      double* __restrict__ ghost) {
    __shared__ DhSum s;
    int i, j;
    const DhFace f = dh_face_of_tile2(P, blockIdx.y, i, j);
    const DhTile t1 = dh_tile(f, 1, i / 2, j / 2), t2 = dh_tile(f, 2, i, j);
    const int nu = t2.u1 - t2.u0, n = nu * (t2.v1 - t2.v0);
    if ((int)blockIdx.x * kDhBlock >= n) return;
    const int at = min((int)(blockIdx.x * kDhBlock + threadIdx.x), n - 1);
    const int u = t2.u0 + at % nu, v = t2.v0 + at / nu;
    double px, py, pz;
    dh_position(P, f, (double)u, (double)v, px, py, pz);
    const double sum = dh_block_sum(P, f, t1, t2, 0, px, py, pz, xyz, charge, 0, natoms, s);
    if ((int)(blockIdx.x * kDhBlock + threadIdx.x) < n) ghost[f.ghost0 + (int64_t)v * f.nu + u] = sum;
}

// The Lagrange polynomials of the Chebyshev points at x in [-1, 1]
// (barycentric form), into w[0..kDhP) at stride `stride`.
__device__ __forceinline__ void dh_weights(double x, const double* node, const double* bary, double* w, int stride) {
    double sum = 0.0;
    int hit = -1;
    for (int k = 0; k < kDhP; ++k) {
        const double d = x - node[k];
        if (d == 0.0) hit = k;
        const double l = bary[k] / (d == 0.0 ? 1.0 : d);
        w[k * stride] = l;
        sum += l;
    }
    for (int k = 0; k < kDhP; ++k) w[k * stride] = hit < 0 ? w[k * stride] / sum : (k == hit ? 1.0 : 0.0);
}

// Far fields to the nodes of a second-level tile, kDhRows node rows per block:
// first along v to the rows, then along u to the nodes, of both levels; the
// near sum is added and the whole divided by the dielectric.
constexpr int kDhCols = (kDhTile + 1) / 2 + 1;   // most nodes across a second-level tile
__global__ __launch_bounds__(kDhBlock) void k_dh_nodes(DhPlan P, const double* __restrict__ c, double eout,
                                                       double* __restrict__ ghost) {
    __shared__ double C[kDhPoints], lu[kDhP][kDhCols], lv[kDhP][kDhRows], rows[kDhP][kDhRows];
    __shared__ double node[kDhP], bary[kDhP];   // Chebyshev points and their barycentric weights
    if (threadIdx.x < kDhP) {
        const double t = (2 * (int)threadIdx.x + 1) / (2.0 * kDhP);
        node[threadIdx.x] = cospi(t);
        bary[threadIdx.x] = (threadIdx.x & 1 ? -1.0 : 1.0) * sinpi(t);
    }
    int i, j;
    const DhFace f = dh_face_of_tile2(P, blockIdx.y, i, j);
    const DhTile t2 = dh_tile(f, 2, i, j);
    const int r0 = t2.v0 + blockIdx.x * kDhRows, nr = min(kDhRows, t2.v1 - r0), nc = t2.u1 - t2.u0;
    if (nr <= 0) return;
    constexpr int M = (kDhRows * kDhCols + kDhBlock - 1) / kDhBlock;
    double out[M];
#pragma unroll
    for (int m = 0; m < M; ++m) out[m] = 0.0;
    for (int level = 1; level <= 2; ++level) {
        if (!(level == 1 ? f.on1 : f.on2)) continue;
        const DhTile T = level == 1 ? dh_tile(f, 1, i / 2, j / 2) : t2;
        const int tile = f.tile0 + (level == 1 ? (j / 2) * f.ku + i / 2
                                               : (f.on1 ? f.ku * f.kv : 0) + j * 2 * f.ku + i);
        __syncthreads();
        for (int k = threadIdx.x; k < kDhPoints; k += kDhBlock) C[k] = c[(int64_t)tile * kDhPoints + k];
        const int w = threadIdx.x;
        if (w < nc) dh_weights((t2.u0 + w - T.cu) / T.wu, node, bary, &lu[0][w], kDhCols);
        else if (w >= 128 && w < 128 + nr) dh_weights((r0 + w - 128 - T.cv) / T.wv, node, bary, &lv[0][w - 128], kDhRows);
        __syncthreads();
        for (int k = threadIdx.x; k < kDhP * kDhRows; k += kDhBlock) {
            const int a = k % kDhP, r = k / kDhP;
            double v = 0.0;
            if (r < nr)
                for (int b = 0; b < kDhP; ++b) v = fma(lv[b][r], C[b * kDhP + a], v);
            rows[a][r] = v;
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const int k = threadIdx.x + m * kDhBlock;
            if (k < nr * nc) {
                const int r = k / nc, u = k - r * nc;
                double v = out[m];
                for (int a = 0; a < kDhP; ++a) v = fma(rows[a][r], lu[a][u], v);
                out[m] = v;
            }
        }
    }
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const int k = threadIdx.x + m * kDhBlock;
        if (k < nr * nc) {
            const int r = k / nc, u = k - r * nc;
            const int64_t t = f.ghost0 + (int64_t)(r0 + r) * f.nu + t2.u0 + u;
            ghost[t] = (ghost[t] + out[m]) / eout;
        }
    }
}

// The tiles of a grid's faces. kd and h decide with the sizes which levels are
// in use; without them (h = 0) the levels that the sizes allow.
DhPlan dh_plan(int nx, int ny, int nz, int64_t natoms, double h, double ox, double oy, double oz, double kd) {
    DhPlan P{};
    P.nx = nx; P.ny = ny; P.nz = nz;
    P.h = h; P.ox = ox; P.oy = oy; P.oz = oz; P.kd = kd;
    int64_t ghost = 0, by_size = 0;
    for (int k = 0; k < 6; ++k) {
        DhFace& f = P.f[k];
        f.axis = k / 2;
        f.side = k % 2;
        f.nu = f.axis == 0 ? ny : nx;
        f.nv = f.axis == 2 ? ny : nz;
        f.ku = (f.nu + kDhTile - 1) / kDhTile;
        f.kv = (f.nv + kDhTile - 1) / kDhTile;
        f.ghost0 = ghost;
        ghost += (int64_t)f.nu * f.nv;
        const double points = (double)f.nu * f.nv;
        for (int level = 1; level <= 2; ++level) {
            const int tiles = level * level * f.ku * f.kv;
            const double w = 0.5 * h * std::max((f.nu + level * f.ku - 1) / (level * f.ku), (f.nv + level * f.kv - 1) / (level * f.kv));
            const bool fits = points >= 1.5 * kDhPoints * tiles && f.nu >= 2 * level * f.ku && f.nv >= 2 * level * f.kv;
            (level == 1 ? f.on1 : f.on2) = fits && kd * w <= kDhMaxKappaW ? 1 : 0;
            by_size += fits ? tiles : 0;
        }
        f.tile0 = P.tiles;
        P.tiles += (f.on1 ? f.ku * f.kv : 0) + (f.on2 ? 4 * f.ku * f.kv : 0);
        P.tiles2 += 4 * f.ku * f.kv;
    }
    // atom ranges of about 512, more where the tiles are too few to fill the
    // device (down to 64 atoms a range)
    const int64_t fill = by_size > 0 ? 2048 / (by_size * (kDhPoints / kDhBlock)) : 1;
    P.chunks = (int)std::max<int64_t>(1, std::min<int64_t>(16, std::max(natoms / 512, std::min(natoms / 64, fill))));
    return P;
}
// The direct sum: more tiles than a grid takes, or so few
// terms that they cost less than the four launches (97 x 105 x 89 with 900 atoms:
// 120 us against 157; 129^3 with 2,000: 395 against 216). In a flat box fewer atoms
// are far from its large faces (129 x 60 x 300 with 2,000 atoms, the whole
// preparation: 639 us against 693). And where all tiles are as large as their faces,
// or halves of them: most atoms are then near, and the few blocks of k_dh_near take as
// long as the direct sum (with salt and the atoms in an ellipsoid of three quarters of
// the box: 65^3 with 4,142 704 us direct, 759 interpolated, 78^3 with 2,876 538 and 586,
// 60 x 131 x 78 with 5,036 830 and 914; without salt 431 and 441, 348 and 362, 500 and 525;
// with quarters of a face: 79^3 with 2,804 534 and 394, 131^3 with 1,019 390 and 290,
// 131 x 131 x 60 with 3,486 822 and 671).
bool dh_direct(const DhPlan& P, int64_t natoms) {
    const double flat = (double)std::max(P.nx, std::max(P.ny, P.nz)) / (double)std::min(P.nx, std::min(P.ny, P.nz));
    const double nghost = 2.0 * ((double)P.nx * P.ny + (double)P.nx * P.nz + (double)P.ny * P.nz);
    bool quarters = false;
    for (const DhFace& f : P.f) quarters = quarters || f.on2 || (f.on1 && f.ku > 1 && f.kv > 1);
    return !quarters || P.tiles2 > 65535 || nghost * (double)natoms < 1e8 * flat;
}
size_t dh_scratch_bytes(int nx, int ny, int nz, int64_t natoms) {
    const DhPlan P = dh_plan(nx, ny, nz, natoms, 0.0, 0.0, 0.0, 0.0, 0.0);
    return dh_direct(P, natoms) ? 0 : sizeof(double) * (size_t)P.tiles * kDhPoints * (size_t)(P.chunks + 1);
}
pb_status dh_faces(const double* xyz, const double* charge, int64_t natoms, int nx, int ny, int nz, double h, double ox,
                   double oy, double oz, double kd, double eout, double* ghost, int64_t nghost, double* scratch,
                   hipStream_t st) {
    const DhPlan P = dh_plan(nx, ny, nz, natoms, h, ox, oy, oz, kd);
    if (dh_direct(P, natoms)) {
        hipLaunchKernelGGL(k_dh_faces, dim3((unsigned)((nghost + kDhBlock - 1) / kDhBlock)), dim3(kDhBlock), 0, st, xyz,
                           charge, natoms, nx, ny, nz, h, ox, oy, oz, kd, eout, ghost, nghost);
        return PB_OK;
    }
    const int64_t n = (int64_t)P.tiles * kDhPoints;
    double* c = scratch + n * P.chunks;
    hipLaunchKernelGGL(k_dh_points, dim3(P.tiles * (kDhPoints / kDhBlock), P.chunks), dim3(kDhBlock), 0, st, P, xyz,
                       charge, natoms, scratch);
    hipLaunchKernelGGL(k_dh_collect, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (const double*)scratch,
                       P.chunks, n, c);
    int most = 0, rows = 0;
    for (const DhFace& f : P.f) {
        const int u = (f.nu + 2 * f.ku - 1) / (2 * f.ku), v = (f.nv + 2 * f.kv - 1) / (2 * f.kv);
        most = std::max(most, u * v);
        rows = std::max(rows, v);
    }
    hipLaunchKernelGGL(k_dh_near, dim3((most + kDhBlock - 1) / kDhBlock, P.tiles2), dim3(kDhBlock), 0, st, P, xyz,
                       charge, natoms, ghost);
    hipLaunchKernelGGL(k_dh_nodes, dim3((rows + kDhRows - 1) / kDhRows, P.tiles2), dim3(kDhBlock), 0, st, P,
                       (const double*)c, eout, ghost);
    return PB_OK;
}

// The right-hand side of k_fields from edge arrays (fractional edges).
__global__ void k_rhs(const double* __restrict__ q, const double* __restrict__ ex,
                      const double* __restrict__ ey, const double* __restrict__ ez,
                      const double* __restrict__ ghost, int nx, int ny, int nz,
                      double h3, double ih2, double* __restrict__ b) {
    const int64_t nn = (int64_t)nx * ny * nz;
    const int64_t fx = (int64_t)ny * nz, fy = (int64_t)nx * nz, fz = (int64_t)nx * ny;
    const double* gxm = ghost;
    const double* gxp = ghost + fx;
    const double* gym = ghost + 2 * fx;
    const double* gyp = gym + fy;
    const double* gzm = gym + 2 * fy;
    const double* gzp = gzm + fz;
    for (int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; n < nn;
         n += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = n % nx, j = (n / nx) % ny, k = n / fz;
        double fold = 0.0;
        if (i == 0) fold = fold + ex[(nx + 1) * (j + ny * k)] * ih2 * gxm[j + ny * k];
        if (i == nx - 1) fold = fold + ex[nx + (nx + 1) * (j + ny * k)] * ih2 * gxp[j + ny * k];
        if (j == 0) fold = fold + ey[i + (int64_t)nx * ((ny + 1) * k)] * ih2 * gym[i + nx * k];
        if (j == ny - 1) fold = fold + ey[i + (int64_t)nx * (ny + (ny + 1) * k)] * ih2 * gyp[i + nx * k];
        if (k == 0) fold = fold + ez[i + nx * j] * ih2 * gzm[i + nx * j];
        if (k == nz - 1) fold = fold + ez[i + nx * j + fz * nz] * ih2 * gzp[i + nx * j];
        b[n] = kFourPi * q[n] / h3 + fold;
    }
}

// Potential at each atom centre by the spreading weights; product q_a*phi_a.
__global__ void k_energy_atoms(const double* __restrict__ xyz, const double* __restrict__ charge,
                               int64_t natoms, int nx, int ny, int nz, double h,
                               double ox, double oy, double oz, int per, const double* __restrict__ x,
                               double* __restrict__ atom_phi, double* __restrict__ qphi,
                               int* __restrict__ flags) {
    const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= natoms) return;
    int i0, j0, k0;
    double fx, fy, fz;
    bool ok = cell_axis(xyz[3 * a], ox, h, nx, per, i0, fx);
    ok = cell_axis(xyz[3 * a + 1], oy, h, ny, per, j0, fy) && ok;
    ok = cell_axis(xyz[3 * a + 2], oz, h, nz, per, k0, fz) && ok;
    if (!ok) {
        atomicOr(flags, 1);
        qphi[a] = 0.0;
        if (atom_phi) atom_phi[a] = 0.0;
        return;
    }
    double t[8];
    for (int c = 0; c < 8; ++c) {
        const double wx = (c & 1) ? fx : 1.0 - fx;
        const double wy = (c & 2) ? fy : 1.0 - fy;
        const double wz = (c & 4) ? fz : 1.0 - fz;
        t[c] = wx * wy * wz * x[corner_node(i0, j0, k0, c, nx, ny, nz)];
    }
    const double phi = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
    if (atom_phi) atom_phi[a] = phi;
    qphi[a] = charge[a] * phi;
}

// Fixed-order sum of n doubles by one workgroup of 1024 threads. Each load's latency
// bounds it where the adds wait for their own load: 16 are on their way at a time
// (201^3, whose arrays have left the last-level cache once all fields are written: 2.7
// ms with one at a time, 1.1 now).
__global__ __launch_bounds__(1024) void k_sum_fixed(const double* __restrict__ v, int64_t n,
                                                    double* __restrict__ out) {
    __shared__ double s[1024];
    double acc = 0.0;
    int64_t i = threadIdx.x;
    for (; i + 15 * 1024 < n; i += 16 * 1024) {
        double x[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) x[k] = v[i + k * 1024];
#pragma unroll
        for (int k = 0; k < 16; ++k) acc += x[k];
    }
    for (; i < n; i += 1024) acc += v[i];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = s[0];
}

// b -= sums[0] / n when sums[1] == 0 (periodic boundary without salt: the
// operator annihilates constants, b gets a uniform neutralising background).
__global__ void k_neutralise(double* __restrict__ b, int64_t n, const double* __restrict__ sums) {
    if (sums[1] != 0.0) return;
    const double m = sums[0] / (double)n;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n;
         t += (int64_t)gridDim.x * blockDim.x)
        b[t] = b[t] - m;
}

inline int64_t next_pow2(int64_t v) {
    int64_t p = 1;
    while (p < v) p <<= 1;
    return p;
}

inline unsigned blocks_for(int64_t n, int bs, int64_t cap = 65536) {
    int64_t b = (n + bs - 1) / bs;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (unsigned)b;
}

// Ascending sort of n keys (n a power of two >= 2): the stages up to the
// chunk size in one LDS launch; each later stage k takes its steps with
// j >= kSortChunk one launch each, then the rest in one LDS launch.
pb_status bitonic_sort(uint64_t* keys, int64_t n, hipStream_t st) {
    const int64_t chunk = std::min<int64_t>(n, kSortChunk);
    const unsigned nb = (unsigned)(n / chunk);
    hipLaunchKernelGGL(k_bitonic_local, dim3(nb), dim3(1024), 0, st, keys, n, (int64_t)2, chunk, (int64_t)1);
    for (int64_t k = 2 * chunk; k <= n; k <<= 1) {
        for (int64_t j = k >> 1; j >= chunk; j >>= 1)
            hipLaunchKernelGGL(k_bitonic_step, dim3(blocks_for(n, 256, 1 << 30)), dim3(256), 0, st, keys, n, j, k);
        hipLaunchKernelGGL(k_bitonic_local, dim3(nb), dim3(1024), 0, st, keys, n, k, k, chunk >> 1);
    }
    PB_HIP(hipGetLastError());
    return PB_OK;
}


}  // namespace

SetupWs carve_setup(void* base, int nx, int ny, int nz, int64_t natoms, bool frac) {
    SetupWs w{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = align_up(off + bytes, 256);
        return o;
    };
    const int64_t npairs = next_pow2(std::max<int64_t>(2, 8 * natoms));
    const int64_t nn = (int64_t)nx * ny * nz;
    const int64_t nmask = (int64_t)(nx + 2) * (ny + 2) * (nz + 2);
    const int64_t ngh = 2 * ((int64_t)ny * nz + (int64_t)nx * nz + (int64_t)nx * ny);
    size_t o_flags = take(256);
    size_t o_keys = take(sizeof(uint64_t) * npairs);
    size_t o_q = take(sizeof(double) * nn);
    size_t o_mask = take((size_t)nmask);
    size_t o_gh = take(sizeof(double) * ngh);
    size_t o_dh = take(dh_scratch_bytes(nx, ny, nz, natoms));
    size_t o_cs = 0, o_ce = 0;
    if (frac) {
        o_cs = take(sizeof(int) * (size_t)nmask);
        o_ce = take(sizeof(int) * (size_t)nmask);
    }
    w.bytes = off;
    if (base) {
        char* b = (char*)base;
        w.flags = (int*)(b + o_flags);
        w.keys = (uint64_t*)(b + o_keys);
        w.qgrid = (double*)(b + o_q);
        w.mask = (uint8_t*)(b + o_mask);
        w.ghost = (double*)(b + o_gh);
        w.dh = (double*)(b + o_dh);
        w.cell_start = frac ? (int*)(b + o_cs) : nullptr;
        w.cell_end = frac ? (int*)(b + o_ce) : nullptr;
    }
    return w;
}

namespace {

bool setup_opts_ok(const pb_setup_opts* o) {
    return o && (o->edge_model == PB_EDGE_NODE || o->edge_model == PB_EDGE_FRACTION);
}

bool grid_ok(const pb_grid* g) {
    const int m = (g && g->boundary == PB_BOUNDARY_PERIODIC) ? 3 : 2;
    return g && (g->boundary == PB_BOUNDARY_FREE || g->boundary == PB_BOUNDARY_PERIODIC) && g->nx >= m &&
           g->ny >= m && g->nz >= m && std::isfinite(g->h) && g->h > 0.0 &&
           std::isfinite(g->origin[0]) && std::isfinite(g->origin[1]) && std::isfinite(g->origin[2]) &&
           (int64_t)(g->nx + 2) * (g->ny + 2) * (int64_t)(g->nz + 2) < (int64_t(1) << 40);
}

}  // namespace

// Every launch of the setup on `st` (the outputs and the flags in w.flags
// are final once the stream reaches this point). The fractional-edge model
// reads the largest radius back to size its cell list, so it synchronises
// once; the two-point model never does.
pb_status setup_enqueue(const pb_grid* g, int64_t natoms, const double* xyz, const double* radius,
                        const double* charge, double eps_in, double eps_out, double kappa_d2, bool frac,
                        double* eps_x, double* eps_y, double* eps_z, double* kappa2, double* rhs, double* qgrid,
                        uint8_t* mask, const SetupWs& w, hipStream_t st) {
    const int nx = g->nx, ny = g->ny, nz = g->nz;
    const double h = g->h, ox = g->origin[0], oy = g->origin[1], oz = g->origin[2];
    const int64_t nn = (int64_t)nx * ny * nz;
    const int64_t nmask = (int64_t)(nx + 2) * (ny + 2) * (nz + 2);
    const int64_t ngh = 2 * ((int64_t)ny * nz + (int64_t)nx * nz + (int64_t)nx * ny);
    uint8_t* m = mask ? mask : w.mask;
    double* q = qgrid ? qgrid : w.qgrid;
    const int per = g->boundary == PB_BOUNDARY_PERIODIC ? 1 : 0;

    const int64_t P = next_pow2(std::max<int64_t>(2, 8 * natoms));
    const double kd = std::sqrt(kappa_d2);
    const bool small = setup_in_one(P, natoms, nn, per) &&
                       (per || dh_direct(dh_plan(nx, ny, nz, natoms, h, ox, oy, oz, kd), natoms));
    hipLaunchKernelGGL(k_setup_clear, dim3(blocks_for(std::max(nmask / 8, nn), 256)), dim3(256), 0, st, w.flags, m,
                       nmask, q, nn);
    if (small)
        hipLaunchKernelGGL(k_setup_small,
                           dim3((unsigned)(1 + natoms + (per ? 0 : (ngh + kDhBlock - 1) / kDhBlock))), dim3(kDhBlock),
                           0, st, xyz, radius, charge, (int)natoms, (int)P, nx, ny, nz, h, ox, oy, oz, per, kd, eps_out,
                           m, q, w.flags, w.ghost, ngh);
    else if (natoms > 0)
        hipLaunchKernelGGL(k_classify, dim3((unsigned)natoms), dim3(256), 0, st, xyz, radius, natoms,
                           nx, ny, nz, h, ox, oy, oz, per, m);
    if (per) {
        hipLaunchKernelGGL(k_wrap_ghosts, dim3(blocks_for((int64_t)ny * nz, 256)), dim3(256), 0, st, m, nx, ny,
                           nz, 0);
        hipLaunchKernelGGL(k_wrap_ghosts, dim3(blocks_for((int64_t)(nx + 2) * nz, 256)), dim3(256), 0, st, m,
                           nx, ny, nz, 1);
        hipLaunchKernelGGL(k_wrap_ghosts, dim3(blocks_for((int64_t)(nx + 2) * (ny + 2), 256)), dim3(256), 0, st,
                           m, nx, ny, nz, 2);
    }
    if (!small) {
        // charges: keys, sort, per-node run sums
        if (natoms > 0) {
            hipLaunchKernelGGL(k_spread_keys, dim3(blocks_for(P, 256, 1 << 30)), dim3(256), 0, st, xyz, natoms, nx, ny,
                               nz, h, ox, oy, oz, per, w.keys, P, w.flags);
            const pb_status es = bitonic_sort(w.keys, P, st);
            if (es != PB_OK) return es;
            hipLaunchKernelGGL(k_spread_sum, dim3(blocks_for(8 * natoms, 256, 1 << 30)), dim3(256), 0, st, w.keys,
                               8 * natoms, xyz, charge, nx, ny, nz, h, ox, oy, oz, per, q);
        }
        // boundary potential on the face ghosts (free space only)
        if (!per) {
            const pb_status es = dh_faces(xyz, charge, natoms, nx, ny, nz, h, ox, oy, oz, kd, eps_out, w.ghost, ngh,
                                          w.dh, st);
            if (es != PB_OK) return es;
        }
    }
    const int64_t fields = (int64_t)(nx + 1) * (ny + 1) * (nz + 1);
    const double h3 = std::pow(h, 3.0), ih2 = 1.0 / (h * h);
    const bool two_point = !(frac && natoms > 0);   // the fractional edges come before the right-hand side
    auto launch_fields = [&](auto index) {
        hipLaunchKernelGGL(k_fields<decltype(index)>, dim3(blocks_for(fields, 256)), dim3(256), 0, st, m, nx, ny, nz,
                           eps_in, eps_out, eps_out * kappa_d2, (const double*)q, (const double*)w.ghost, h3, ih2, per,
                           eps_x, eps_y, eps_z, kappa2, two_point ? rhs : nullptr);
    };
    if (fields < (int64_t(1) << 31)) launch_fields((unsigned)0);
    else launch_fields((int64_t)0);
    if (frac && natoms > 0) {
        // cell list of the atoms, then the fractional edges over the two-point ones
        double* rmax_d = (double*)w.keys;   // the keys are done with
        hipLaunchKernelGGL(k_max_radius, dim3(1), dim3(1024), 0, st, radius, natoms, rmax_d);
        double rmax = 0.0;
        PB_HIP(hipMemcpyAsync(&rmax, rmax_d, sizeof(double), hipMemcpyDeviceToHost, st));
        PB_HIP(hipStreamSynchronize(st));
        PB_ARG(std::isfinite(rmax) && rmax >= 0.0, "pb_setup: non-finite atom radius");
        const int mcell = std::max(1, (int)std::ceil(rmax / h));
        const int ncx = (nx + 2 + mcell - 1) / mcell, ncy = (ny + 2 + mcell - 1) / mcell, ncz = (nz + 2 + mcell - 1) / mcell;
        const int64_t ncells = (int64_t)ncx * ncy * ncz;
        const int64_t Pc = next_pow2(std::max<int64_t>(2, natoms));
        hipLaunchKernelGGL(k_fill_u64, dim3(blocks_for(Pc, 256)), dim3(256), 0, st, w.keys, Pc, ~0ull);
        hipLaunchKernelGGL(k_cell_keys, dim3(blocks_for(natoms, 256, 1 << 30)), dim3(256), 0, st, xyz, natoms, nx, ny,
                           nz, h, ox, oy, oz, mcell, ncx, ncy, w.keys);
        for (int64_t k = 2; k <= Pc; k <<= 1)
            for (int64_t j = k >> 1; j > 0; j >>= 1)
                hipLaunchKernelGGL(k_bitonic_step, dim3(blocks_for(Pc, 256, 1 << 30)), dim3(256), 0, st, w.keys, Pc,
                                   j, k);
        hipLaunchKernelGGL(k_fill_i32, dim3(blocks_for(ncells, 256)), dim3(256), 0, st, w.cell_start, ncells, 0);
        hipLaunchKernelGGL(k_fill_i32, dim3(blocks_for(ncells, 256)), dim3(256), 0, st, w.cell_end, ncells, 0);
        hipLaunchKernelGGL(k_cell_bounds, dim3(blocks_for(natoms, 256, 1 << 30)), dim3(256), 0, st,
                           (const uint64_t*)w.keys, natoms, w.cell_start, w.cell_end);
        const int64_t nedge3 = (int64_t)(nx + 1) * ny * nz + (int64_t)nx * (ny + 1) * nz + (int64_t)nx * ny * (nz + 1);
        hipLaunchKernelGGL(k_edges_fraction, dim3(blocks_for(nedge3, 256)), dim3(256), 0, st, xyz, radius,
                           (const uint64_t*)w.keys, (const int*)w.cell_start, (const int*)w.cell_end, nx, ny, nz, h,
                           ox, oy, oz, rmax, mcell, ncx, ncy, ncz, eps_in, eps_out, eps_x, eps_y, eps_z, w.flags);
        hipLaunchKernelGGL(k_rhs, dim3(blocks_for(nn, 256)), dim3(256), 0, st, q, eps_x, eps_y, eps_z, w.ghost, nx, ny,
                           nz, h3, ih2, rhs);
    }
    if (per) {   // sums of b and kbar^2 (fixed order) into the unused ghost buffer, then the background
        hipLaunchKernelGGL(k_sum_fixed, dim3(1), dim3(1024), 0, st, (const double*)rhs, nn, w.ghost);
        hipLaunchKernelGGL(k_sum_fixed, dim3(1), dim3(1024), 0, st, (const double*)kappa2, nn, w.ghost + 1);
        hipLaunchKernelGGL(k_neutralise, dim3(blocks_for(nn, 256)), dim3(256), 0, st, rhs, nn,
                           (const double*)w.ghost);
    }
    PB_HIP(hipGetLastError());
    return PB_OK;
}

size_t energy_scratch_bytes(int64_t natoms) { return sizeof(double) * (size_t)std::max<int64_t>(natoms, 1); }

pb_status energy_enqueue(const pb_grid* g, int64_t natoms, const double* xyz, const double* charge, const double* x,
                         double* qphi, int* flags, double* sum, hipStream_t st) {
    if (natoms > 0)
        hipLaunchKernelGGL(k_energy_atoms, dim3(blocks_for(natoms, 256, 1 << 30)), dim3(256), 0, st, xyz, charge,
                           natoms, g->nx, g->ny, g->nz, g->h, g->origin[0], g->origin[1], g->origin[2],
                           g->boundary == PB_BOUNDARY_PERIODIC ? 1 : 0, x, (double*)nullptr, qphi, flags);
    hipLaunchKernelGGL(k_sum_fixed, dim3(1), dim3(1024), 0, st, (const double*)qphi, natoms, sum);
    PB_HIP(hipGetLastError());
    return PB_OK;
}

double energy_kcal(double sum_q_phi) { return 0.5 * sum_q_phi * kCoulombKcal; }

namespace {

}  // namespace

}  // namespace pb

using namespace pb;

extern "C" size_t pb_setup_workspace_bytes(const pb_grid* g, int64_t natoms) {
    if (!grid_ok(g) || natoms < 0 || natoms > kMaxAtoms) return 0;
    return carve_setup(nullptr, g->nx, g->ny, g->nz, natoms).bytes;
}

extern "C" size_t pb_setup_ex_workspace_bytes(const pb_grid* g, int64_t natoms, const pb_setup_opts* opts) {
    if (!grid_ok(g) || natoms < 0 || natoms > kMaxAtoms || !setup_opts_ok(opts)) return 0;
    return carve_setup(nullptr, g->nx, g->ny, g->nz, natoms, opts->edge_model == PB_EDGE_FRACTION).bytes;
}

extern "C" pb_status pb_setup(const pb_grid* g, int64_t natoms, const double* xyz,
                              const double* radius, const double* charge, double eps_in,
                              double eps_out, double kappa_d2, double* eps_x, double* eps_y,
                              double* eps_z, double* kappa2, double* rhs, double* qgrid,
                              uint8_t* mask, void* workspace, size_t workspace_bytes,
                              void* stream_) {
    pb_setup_opts o{};
    o.edge_model = PB_EDGE_NODE;
    return pb_setup_ex(g, natoms, xyz, radius, charge, eps_in, eps_out, kappa_d2, &o, eps_x, eps_y, eps_z, kappa2,
                       rhs, qgrid, mask, workspace, workspace_bytes, stream_);
}

extern "C" pb_status pb_setup_ex(const pb_grid* g, int64_t natoms, const double* xyz,
                                 const double* radius, const double* charge, double eps_in,
                                 double eps_out, double kappa_d2, const pb_setup_opts* opts, double* eps_x,
                                 double* eps_y, double* eps_z, double* kappa2, double* rhs, double* qgrid,
                                 uint8_t* mask, void* workspace, size_t workspace_bytes, void* stream_) {
    PB_ARG(setup_opts_ok(opts), "pb_setup: invalid options (edge_model)");
    const bool frac = opts->edge_model == PB_EDGE_FRACTION;
    PB_ARG(!frac || (g && g->boundary == PB_BOUNDARY_FREE),
           "pb_setup: the fractional-edge dielectric is available with the free-space boundary only");
    PB_ARG(!frac || kFractionEdgesEnabled,
           "pb_setup: the fractional-edge dielectric (PB_EDGE_FRACTION) is switched off in this library");
    PB_ARG(grid_ok(g), "pb_setup: grid needs a valid boundary, nx,ny,nz >= 2 (>= 3 periodic), finite h > 0 "
                       "and a finite origin");
    PB_ARG(natoms >= 0 && natoms <= kMaxAtoms, "pb_setup: natoms must be in [0, 2^21-1]");
    PB_ARG(natoms == 0 || (xyz && radius && charge), "pb_setup: null atom array");
    PB_ARG(eps_x && eps_y && eps_z && kappa2 && rhs, "pb_setup: null output array");
    PB_ARG(std::isfinite(eps_in) && std::isfinite(eps_out) && eps_in > 0 && eps_out > 0,
           "pb_setup: dielectric constants must be finite and > 0");
    PB_ARG(std::isfinite(kappa_d2) && kappa_d2 >= 0, "pb_setup: kappa_d2 must be finite and >= 0");
    PB_ARG(workspace != nullptr, "pb_setup: null workspace");
    const int nx = g->nx, ny = g->ny, nz = g->nz;
    SetupWs w = carve_setup(workspace, nx, ny, nz, natoms, frac);
    if (workspace_bytes < w.bytes) {
        set_error("pb_setup: workspace of %zu bytes, %zu needed", workspace_bytes, w.bytes);
        return PB_ERR_NOMEM;
    }
    hipStream_t st = (hipStream_t)stream_;
    const pb_status e = setup_enqueue(g, natoms, xyz, radius, charge, eps_in, eps_out, kappa_d2, frac, eps_x, eps_y,
                                      eps_z, kappa2, rhs, qgrid, mask, w, st);
    if (e != PB_OK) return e;
    const int per = g->boundary == PB_BOUNDARY_PERIODIC ? 1 : 0;
    PB_HIP(hipGetLastError());
    int flags = 0;
    PB_HIP(hipMemcpyAsync(&flags, w.flags, sizeof(int), hipMemcpyDeviceToHost, st));
    PB_HIP(hipStreamSynchronize(st));
    if (flags & 4) {
        set_error("pb_setup: more than 16 separate inside pieces on one edge (fractional edges)");
        return PB_ERR_ARG;
    }
    if (flags) {
        set_error(per ? "pb_setup: an atom centre lies beyond 2^28 nodes from the origin"
                      : "pb_setup: an atom centre lies outside the node box");
        return PB_ERR_ARG;
    }
    return PB_OK;
}

extern "C" size_t pb_energy_workspace_bytes(int64_t natoms) {
    if (natoms < 0 || natoms > kMaxAtoms) return 0;
    return 512 + align_up(sizeof(double) * (size_t)std::max<int64_t>(natoms, 1), 256);
}

extern "C" pb_status pb_energy(const pb_grid* g, int64_t natoms, const double* xyz,
                               const double* charge, const double* x, double* atom_phi,
                               double* energy, void* workspace, size_t workspace_bytes,
                               void* stream_) {
    PB_ARG(grid_ok(g), "pb_energy: grid needs a valid boundary, nx,ny,nz >= 2 (>= 3 periodic), finite h > 0 "
                       "and a finite origin");
    PB_ARG(natoms >= 0 && natoms <= kMaxAtoms, "pb_energy: natoms must be in [0, 2^21-1]");
    PB_ARG(natoms == 0 || (xyz && charge), "pb_energy: null atom array");
    PB_ARG(x && energy && workspace, "pb_energy: null x, energy or workspace");
    const size_t need = pb_energy_workspace_bytes(natoms);
    if (workspace_bytes < need) {
        set_error("pb_energy: workspace of %zu bytes, %zu needed", workspace_bytes, need);
        return PB_ERR_NOMEM;
    }
    hipStream_t st = (hipStream_t)stream_;
    char* b = (char*)workspace;
    int* flags = (int*)b;
    double* out = (double*)(b + 256);
    double* qphi = (double*)(b + 512);
    hipLaunchKernelGGL(k_fill_u8, dim3(1), dim3(64), 0, st, (uint8_t*)flags, (int64_t)256, (uint8_t)0);
    if (natoms > 0)
        hipLaunchKernelGGL(k_energy_atoms, dim3(blocks_for(natoms, 256, 1 << 30)), dim3(256), 0, st, xyz,
                           charge, natoms, g->nx, g->ny, g->nz, g->h, g->origin[0], g->origin[1],
                           g->origin[2], g->boundary == PB_BOUNDARY_PERIODIC ? 1 : 0, x, atom_phi, qphi, flags);
    hipLaunchKernelGGL(k_sum_fixed, dim3(1), dim3(1024), 0, st, qphi, natoms, out);
    PB_HIP(hipGetLastError());
    double host[2];
    int hflags = 0;
    PB_HIP(hipMemcpyAsync(host, out, sizeof(double), hipMemcpyDeviceToHost, st));
    PB_HIP(hipMemcpyAsync(&hflags, flags, sizeof(int), hipMemcpyDeviceToHost, st));
    PB_HIP(hipStreamSynchronize(st));
    if (hflags) {
        set_error("pb_energy: an atom centre lies outside the node box");
        return PB_ERR_ARG;
    }
    *energy = 0.5 * host[0] * kCoulombKcal;
    return PB_OK;
}
