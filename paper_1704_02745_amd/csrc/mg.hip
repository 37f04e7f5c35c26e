// Geometric-multigrid-preconditioned CG on the stencil of Eq. 3.
//
// The paper points to geometric multigrid as the next step for these systems
// (sections 3.2 and 4) without fixing a scheme. This one:
//   levels    vertex coarsening by two per axis: coarse node I sits at fine
//             node 2I+1 (floor(n/2) nodes, spacing 2h); coarsening stops when
//             an axis would drop below 3 nodes or a level has <= 512 nodes;
//   operator  every level is Eq. 3 at its spacing, with edge dielectrics from
//             the finer level: the series (harmonic) combination of the two
//             fine edges an edge spans, averaged over the nine fine lines
//             around it with weights (1,2,1)x(1,2,1)/16, and kbar^2 averaged
//             with full weighting; so each level is a 7-point stencil and
//             the fine-level kernels apply to all of them;
//   transfer  trilinear prolongation P (coarse ghosts zero), R = P^T/8;
//   cycle     the preconditioner z = M r is one V-cycle from z = 0 with two
//             damped-Jacobi sweeps (omega 0.8) before and after the coarse
//             correction and 40 sweeps on the coarsest level: a fixed
//             symmetric positive definite operator, as CG requires;
//   outer     the section 2.2 listing with that M, host-driven like the DIA
//             form (device-side scalars, the host polls the stopping flag).
#include "jpcg_device.hpp"
#include "pcg_common.hpp"
#include "solver.hpp"

#include <type_traits>
#include <vector>

namespace pb {
namespace {

constexpr int kMgNu = 2;            // Jacobi sweeps before and after the coarse correction
constexpr int kMgCoarseSweeps = 40;  // sweeps on the coarsest level
constexpr int64_t kMgMinNodes = 512;
constexpr int kMgCus = 256;
constexpr double kMgOmega = 0.8;

__device__ __forceinline__ double w3(int a) { return a == 0 ? 0.5 : 0.25; }   // a in -1..1
// a / d in the smoothers: exact division in FP64; in FP32 a times the
// hardware reciprocal of d (within 1 ulp), which keeps the sweeps, whose
// neighbour terms each need one, from being bound by division.
__device__ __forceinline__ double mg_div(double a, double d) { return a / d; }
__device__ __forceinline__ float mg_div(float a, float d) { return a * __builtin_amdgcn_rcpf(d); }
// a * b + c with one rounding
__device__ __forceinline__ double mg_fma(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float mg_fma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double series2(double a, double b) { return 2.0 * a * b / (a + b); }

// One coarser level from a finer one (FP64 staggered edge arrays and kbar^2
// in the caller's layouts); one thread per output element.
__global__ void k_mg_coarsen(const double* __restrict__ ex, const double* __restrict__ ey,
                             const double* __restrict__ ez, const double* __restrict__ k2, int nx, int ny, int nz,
                             double* __restrict__ cex, double* __restrict__ cey, double* __restrict__ cez,
                             double* __restrict__ ck2, int ncx, int ncy, int ncz) {
    const int64_t nex = (int64_t)(ncx + 1) * ncy * ncz, ney = (int64_t)ncx * (ncy + 1) * ncz;
    const int64_t nez = (int64_t)ncx * ncy * (ncz + 1), nk = (int64_t)ncx * ncy * ncz;
    const int64_t total = nex + ney + nez + nk;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total;
         t += (int64_t)gridDim.x * blockDim.x) {
        if (t < nex) {   // x-edges [K][J][E]: lines over (j, k) around (2J+1, 2K+1)
            const int E = (int)(t % (ncx + 1)), J = (int)((t / (ncx + 1)) % ncy), K = (int)(t / ((int64_t)(ncx + 1) * ncy));
            double acc = 0.0, ws = 0.0;
            for (int a = -1; a <= 1; ++a) {
                const int j = 2 * J + 1 + a;
                if (j < 0 || j >= ny) continue;
                for (int b = -1; b <= 1; ++b) {
                    const int k = 2 * K + 1 + b;
                    if (k < 0 || k >= nz) continue;
                    const double* line = ex + (int64_t)(nx + 1) * (j + (int64_t)ny * k);
                    const double e1 = line[2 * E];
                    const double e2 = (2 * E + 1 <= nx) ? line[2 * E + 1] : e1;
                    const double w = w3(a) * w3(b);
                    acc = acc + w * series2(e1, e2);
                    ws = ws + w;
                }
            }
            cex[t] = acc / ws;
        } else if (t < nex + ney) {   // y-edges [K][E][I]: lines over (i, k)
            const int64_t u = t - nex;
            const int I = (int)(u % ncx), E = (int)((u / ncx) % (ncy + 1)), K = (int)(u / ((int64_t)ncx * (ncy + 1)));
            double acc = 0.0, ws = 0.0;
            for (int a = -1; a <= 1; ++a) {
                const int i = 2 * I + 1 + a;
                if (i < 0 || i >= nx) continue;
                for (int b = -1; b <= 1; ++b) {
                    const int k = 2 * K + 1 + b;
                    if (k < 0 || k >= nz) continue;
                    const double e1 = ey[i + (int64_t)nx * (2 * E + (int64_t)(ny + 1) * k)];
                    const double e2 = (2 * E + 1 <= ny) ? ey[i + (int64_t)nx * (2 * E + 1 + (int64_t)(ny + 1) * k)] : e1;
                    const double w = w3(a) * w3(b);
                    acc = acc + w * series2(e1, e2);
                    ws = ws + w;
                }
            }
            cey[u] = acc / ws;
        } else if (t < nex + ney + nez) {   // z-edges [E][J][I]: lines over (i, j)
            const int64_t u = t - nex - ney;
            const int I = (int)(u % ncx), J = (int)((u / ncx) % ncy), E = (int)(u / ((int64_t)ncx * ncy));
            double acc = 0.0, ws = 0.0;
            for (int a = -1; a <= 1; ++a) {
                const int i = 2 * I + 1 + a;
                if (i < 0 || i >= nx) continue;
                for (int b = -1; b <= 1; ++b) {
                    const int j = 2 * J + 1 + b;
                    if (j < 0 || j >= ny) continue;
                    const int64_t plane = (int64_t)nx * ny;
                    const double e1 = ez[i + (int64_t)nx * j + plane * (2 * E)];
                    const double e2 = (2 * E + 1 <= nz) ? ez[i + (int64_t)nx * j + plane * (2 * E + 1)] : e1;
                    const double w = w3(a) * w3(b);
                    acc = acc + w * series2(e1, e2);
                    ws = ws + w;
                }
            }
            cez[u] = acc / ws;
        } else {   // kbar^2 [K][J][I]: full weighting
            const int64_t u = t - nex - ney - nez;
            const int I = (int)(u % ncx), J = (int)((u / ncx) % ncy), K = (int)(u / ((int64_t)ncx * ncy));
            double acc = 0.0, ws = 0.0;
            for (int c = -1; c <= 1; ++c) {
                const int k = 2 * K + 1 + c;
                if (k < 0 || k >= nz) continue;
                for (int b = -1; b <= 1; ++b) {
                    const int j = 2 * J + 1 + b;
                    if (j < 0 || j >= ny) continue;
                    for (int a = -1; a <= 1; ++a) {
                        const int i = 2 * I + 1 + a;
                        if (i < 0 || i >= nx) continue;
                        const double w = w3(a) * w3(b) * w3(c);
                        acc = acc + w * k2[i + (int64_t)nx * (j + (int64_t)ny * k)];
                        ws = ws + w;
                    }
                }
            }
            ck2[u] = acc / ws;
        }
    }
}

// A level's operator in the padded layout (couplings zero across the box
// faces, the diagonal with every edge), rounded to T.
template <typename T>
__global__ void k_mg_op(const double* __restrict__ ex, const double* __restrict__ ey, const double* __restrict__ ez,
                        const double* __restrict__ k2, int nx, int ny, int nz, int64_t sp, double hh, Op<T> op) {
    const int64_t plane = (int64_t)nx * ny, npad = sp * nz;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < npad;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t k = t / sp, pp = t - k * sp;
        T* cx = (T*)op.cx;
        T* cy = (T*)op.cy;
        T* cz = (T*)op.cz;
        T* d = (T*)op.d;
        if (pp >= plane) {
            cx[t] = T(0); cy[t] = T(0); cz[t] = T(0); d[t] = T(1);
            continue;
        }
        const int64_t j = pp / nx, i = pp - j * nx, n = pp + plane * k;
        const double exm = ex[i + (int64_t)(nx + 1) * (j + (int64_t)ny * k)];
        const double exp_ = ex[i + 1 + (int64_t)(nx + 1) * (j + (int64_t)ny * k)];
        const double eym = ey[i + (int64_t)nx * (j + (int64_t)(ny + 1) * k)];
        const double eyp = ey[i + (int64_t)nx * (j + 1 + (int64_t)(ny + 1) * k)];
        const double ezm = ez[i + (int64_t)nx * (j + (int64_t)ny * k)];
        const double ezp = ez[i + (int64_t)nx * (j + (int64_t)ny * (k + 1))];
        cx[t] = (T)((i < nx - 1) ? exp_ / hh : 0.0);
        cy[t] = (T)((j < ny - 1) ? eyp / hh : 0.0);
        cz[t] = (T)((k < nz - 1) ? ezp / hh : 0.0);
        d[t] = (T)((((((exm + exp_) + eym) + eyp) + ezm) + ezp) / hh + k2[n]);
    }
}

// (A v) at padded position t (free-space stencil; zero couplings cut the
// faces and the pad slots).
template <typename T>
__device__ __forceinline__ T mg_apply(const Op<T>& op, const T* __restrict__ v, int64_t t, int nx, int64_t sp,
                                      int64_t npad) {
    T nb = op.cx[t] * (t + 1 < npad ? v[t + 1] : T(0));
    nb += (t >= 1 ? op.cx[t - 1] * v[t - 1] : T(0));
    nb += op.cy[t] * (t + nx < npad ? v[t + nx] : T(0));
    nb += (t >= nx ? op.cy[t - nx] * v[t - nx] : T(0));
    nb += op.cz[t] * (t + sp < npad ? v[t + sp] : T(0));
    nb += (t >= sp ? op.cz[t - sp] * v[t - sp] : T(0));
    return op.d[t] * v[t] - nb;
}

// One damped-Jacobi sweep out = in + omega (b - A in)/d.
template <typename T>
__global__ void k_mg_jacobi(Op<T> op, const T* __restrict__ b, const T* __restrict__ in, T* __restrict__ out,
                            int nx, int64_t sp, int64_t npad, T omega, const SyncState* S) {
    if (S && stop(S)) return;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < npad;
         t += (int64_t)gridDim.x * blockDim.x) {
        const T r = b[t] - mg_apply(op, in, t, nx, sp, npad);
        out[t] = in[t] + mg_div(omega * r, op.d[t]);
    }
}

// The first two damped-Jacobi sweeps from zero in one pass. The first
// sweep's output x1 = omega b / d is formed where the second needs it (the
// node and its six neighbours) with one arithmetic everywhere, so the result
// equals two separate sweeps bit for bit.
template <typename T>
__device__ __forceinline__ T mg_x1(const Op<T>& op, const T* __restrict__ b, int64_t t, T omega) {
    return mg_div(omega * b[t], op.d[t]);
}

template <typename T>
__device__ __forceinline__ T mg_jacobi2z_at(const Op<T>& op, const T* __restrict__ b, int64_t t, int nx, int64_t sp,
                                            int64_t npad, T omega) {
    T nb = op.cx[t] * (t + 1 < npad ? mg_x1(op, b, t + 1, omega) : T(0));
    nb += (t >= 1 ? op.cx[t - 1] * mg_x1(op, b, t - 1, omega) : T(0));
    nb += op.cy[t] * (t + nx < npad ? mg_x1(op, b, t + nx, omega) : T(0));
    nb += (t >= nx ? op.cy[t - nx] * mg_x1(op, b, t - nx, omega) : T(0));
    nb += op.cz[t] * (t + sp < npad ? mg_x1(op, b, t + sp, omega) : T(0));
    nb += (t >= sp ? op.cz[t - sp] * mg_x1(op, b, t - sp, omega) : T(0));
    const T x1 = mg_x1(op, b, t, omega);
    const T r = b[t] - (op.d[t] * x1 - nb);
    return x1 + mg_div(omega * r, op.d[t]);
}
template <typename T>
__global__ void k_mg_jacobi2z(Op<T> op, const T* __restrict__ b, T* __restrict__ out, int nx, int64_t sp,
                              int64_t npad, T omega, const SyncState* S) {
    if (S && stop(S)) return;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < npad;
         t += (int64_t)gridDim.x * blockDim.x)
        out[t] = mg_jacobi2z_at(op, b, t, nx, sp, npad, omega);
}

// The finest level's last post-smoothing sweep fused with the outer
// iteration's r.z and r.r (the level's right-hand side is the outer residual
// r): block b sweeps positions [b*per, (b+1)*per), threads striding by the
// block size, and stores the block sums in the fixed order of block_sum_store.
template <typename T>
__global__ __launch_bounds__(kBS) void k_mg_jacobi_dot2(Op<T> op, const T* __restrict__ b, const T* __restrict__ in,
                                                        T* __restrict__ out, int nx, int64_t sp, int64_t npad,
                                                        T omega, int64_t per, double* __restrict__ partials,
                                                        const SyncState* S) {
    if (stop(S)) return;
    double acc[2] = {0.0, 0.0};
    const int64_t lo = (int64_t)blockIdx.x * per, hi = min(lo + per, npad);
    for (int64_t t = lo + threadIdx.x; t < hi; t += kBS) {
        const T res = b[t] - mg_apply(op, in, t, nx, sp, npad);
        const T z = in[t] + mg_div(omega * res, op.d[t]);
        out[t] = z;
        acc[0] += (double)b[t] * (double)z;
        acc[1] += (double)b[t] * (double)b[t];
    }
    block_sum_store<2>(acc, partials + (size_t)blockIdx.x * kMaxPartials);
}

template <typename T>
__global__ void k_mg_residual(Op<T> op, const T* __restrict__ b, const T* __restrict__ x, T* __restrict__ r, int nx,
                              int64_t sp, int64_t npad, const SyncState* S) {
    if (S && stop(S)) return;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < npad;
         t += (int64_t)gridDim.x * blockDim.x)
        r[t] = b[t] - mg_apply(op, x, t, nx, sp, npad);
}

// q = A v (the outer iteration's product).
template <typename T>
__global__ void k_mg_apply(Op<T> op, const T* __restrict__ v, T* __restrict__ q, int nx, int64_t sp, int64_t npad,
                           const SyncState* S) {
    if (S && stop(S)) return;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < npad;
         t += (int64_t)gridDim.x * blockDim.x)
        q[t] = mg_apply(op, v, t, nx, sp, npad);
}

// bc = R r (full weighting; fine nodes outside the grid contribute zero).
// Grid: blockIdx.y is the coarse plane K; the x-dimension strides over the
// coarse plane's positions (pad slots get zero).
template <typename T>
__device__ __forceinline__ T mg_restrict_at(const T* __restrict__ r, int nx, int ny, int nz, int64_t sp, int I, int J,
                                            int K) {
    T acc = T(0);
    for (int c = -1; c <= 1; ++c) {
        const int k = 2 * K + 1 + c;
        if (k < 0 || k >= nz) continue;
        for (int b = -1; b <= 1; ++b) {
            const int j = 2 * J + 1 + b;
            if (j < 0 || j >= ny) continue;
            const T* row = r + (int64_t)k * sp + (int64_t)j * nx;
            for (int a = -1; a <= 1; ++a) {
                const int i = 2 * I + 1 + a;
                if (i < 0 || i >= nx) continue;
                acc += (T)(w3(a) * w3(b) * w3(c)) * row[i];
            }
        }
    }
    return acc;
}
template <typename T>
__global__ void k_mg_restrict(const T* __restrict__ r, int nx, int ny, int nz, int64_t sp, T* __restrict__ bc,
                              int ncx, int ncy, int ncz, int64_t spc, const SyncState* S) {
    if (S && stop(S)) return;
    const int K = blockIdx.y;
    const int pc = ncx * ncy;
    for (int pp = blockIdx.x * blockDim.x + threadIdx.x; pp < (int)spc; pp += gridDim.x * blockDim.x) {
        const int64_t t = (int64_t)K * spc + pp;
        if (pp >= pc) {
            bc[t] = T(0);
            continue;
        }
        const int J = pp / ncx, I = pp - J * ncx;
        bc[t] = mg_restrict_at(r, nx, ny, nz, sp, I, J, K);
    }
}

// x += P xc (trilinear: fine f odd takes coarse (f-1)/2, fine f even the mean
// of coarse f/2-1 and f/2; coarse ghosts are zero). One thread per cell of
// the coarse grid shifted by one fine node: cell (I, J, K), I in -1..ncx-1,
// holds the fine nodes 2I+1 (odd) and 2I+2 (even) of each axis, all of which
// interpolate from the same eight coarse nodes I..I+1 x J..J+1 x K..K+1, read
// once. Each fine node sums its terms in z, y, x order, zero weights skipped.
// Grid: blockIdx.y is K+1; the x-dimension strides over (I, J).
template <typename T>
__device__ __forceinline__ void mg_prolong_cell(const T* __restrict__ xc, int ncx, int ncy, int ncz, int64_t spc,
                                                T* __restrict__ x, int nx, int ny, int nz, int64_t sp, int I, int J,
                                                int K) {
    T v[2][2][2];   // coarse (K+kk, J+jj, I+ii), zero outside the coarse grid
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
            for (int ii = 0; ii < 2; ++ii) {
                const int ck = K + kk, cj = J + jj, ci = I + ii;
                const bool in = ck >= 0 && ck < ncz && cj >= 0 && cj < ncy && ci >= 0 && ci < ncx;
                v[kk][jj][ii] = in ? xc[(int64_t)ck * spc + (int64_t)cj * ncx + ci] : T(0);
            }
    // per axis, fine node 2C+1+e (e = 0 odd, 1 even): its terms (coarse
    // offset, weight) in order; n = number of terms
#pragma unroll
    for (int ez = 0; ez < 2; ++ez) {
        const int k = 2 * K + 1 + ez;
        if (k < 0 || k >= nz) continue;
#pragma unroll
        for (int ey = 0; ey < 2; ++ey) {
            const int j = 2 * J + 1 + ey;
            if (j < 0 || j >= ny) continue;
#pragma unroll
            for (int ex = 0; ex < 2; ++ex) {
                const int i = 2 * I + 1 + ex;
                if (i < 0 || i >= nx) continue;
                T add = T(0);
                for (int tz = 0; tz <= ez; ++tz) {
                    const int ck = K + tz;
                    if (ck < 0 || ck >= ncz) continue;
                    const T wz = ez ? T(0.5) : T(1);
                    for (int ty = 0; ty <= ey; ++ty) {
                        const int cj = J + ty;
                        if (cj < 0 || cj >= ncy) continue;
                        const T wy = ey ? T(0.5) : T(1);
                        for (int tx = 0; tx <= ex; ++tx) {
                            const int ci = I + tx;
                            if (ci < 0 || ci >= ncx) continue;
                            const T wx = ex ? T(0.5) : T(1);
                            add += wx * wy * wz * v[tz][ty][tx];
                        }
                    }
                }
                x[(int64_t)k * sp + (int64_t)j * nx + i] += add;
            }
        }
    }
}
template <typename T>
__global__ void k_mg_prolong_add(const T* __restrict__ xc, int ncx, int ncy, int ncz, int64_t spc,
                                 T* __restrict__ x, int nx, int ny, int nz, int64_t sp, const SyncState* S) {
    if (S && stop(S)) return;
    const int K = (int)blockIdx.y - 1;
    const int cw = ncx + 1, cells = cw * (ncy + 1);
    for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < cells; c += gridDim.x * blockDim.x) {
        const int J = c / cw - 1, I = c - (J + 1) * cw - 1;
        mg_prolong_cell(xc, ncx, ncy, ncz, spc, x, nx, ny, nz, sp, I, J, K);
    }
}

// Launch shape of the plane-indexed kernels: blockIdx.y = plane.
dim3 plane_grid(int64_t positions, int planes) {
    return dim3((unsigned)std::min<int64_t>(std::max<int64_t>(1, (positions + kBS - 1) / kBS), 1024), (unsigned)planes);
}

// The outer iteration's direction and product in one pass over a block's
// range of rows: p = z + beta p_old (formed wherever the product needs it,
// with one rounding, so neighbours see the value the node's owner stores),
// q = A p, and the block's p.q.
template <typename T>
__global__ __launch_bounds__(kBS) void k_mg_direction_apply(Op<T> op, const T* __restrict__ z,
                                                            const T* __restrict__ pold, T* __restrict__ pnew,
                                                            T* __restrict__ q, int nx, int64_t sp, int64_t npad,
                                                            int64_t per, double* __restrict__ partials,
                                                            const SyncState* S) {
    if (stop(S)) return;
    const T beta = (T)S->beta;
    auto P = [&](int64_t u) { return mg_fma(beta, pold[u], z[u]); };
    double acc[1] = {0.0};
    const int64_t lo = (int64_t)blockIdx.x * per, hi = min(lo + per, npad);
    for (int64_t t = lo + threadIdx.x; t < hi; t += kBS) {
        T nb = op.cx[t] * (t + 1 < npad ? P(t + 1) : T(0));
        nb += (t >= 1 ? op.cx[t - 1] * P(t - 1) : T(0));
        nb += op.cy[t] * (t + nx < npad ? P(t + nx) : T(0));
        nb += (t >= nx ? op.cy[t - nx] * P(t - nx) : T(0));
        nb += op.cz[t] * (t + sp < npad ? P(t + sp) : T(0));
        nb += (t >= sp ? op.cz[t - sp] * P(t - sp) : T(0));
        const T pt = P(t);
        const T qt = op.d[t] * pt - nb;
        pnew[t] = pt;
        q[t] = qt;
        acc[0] += (double)pt * (double)qt;
    }
    block_sum_store<1>(acc, partials + (size_t)blockIdx.x * kMaxPartials);
}

// The outer update x += alpha p, rnew = r_old - alpha q.
template <typename T>
__global__ void k_mg_update(T* __restrict__ x, const T* __restrict__ p, const T* __restrict__ rold,
                            const T* __restrict__ q, T* __restrict__ rnew, int64_t npad, const SyncState* S) {
    if (stop(S)) return;
    const T alpha = (T)S->alpha;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < npad;
         t += (int64_t)gridDim.x * blockDim.x) {
        x[t] = mg_fma(alpha, p[t], x[t]);
        rnew[t] = mg_fma(-alpha, q[t], rold[t]);
    }
}

// The coarsest level: `sweeps` damped-Jacobi sweeps from zero by one
// workgroup (the level is small); buf[(sweeps-1) & 1] holds the result.
// With `lds` set the sweeps run on LDS copies of the operator, right-hand
// side and iterates (the launch brings 7 npad values of dynamic LDS), with
// the same arithmetic, and the result is copied out at the end.
template <typename T>
__device__ __forceinline__ void mg_coarse_sweeps(const Op<T>& o, const T* __restrict__ b, T* __restrict__ u0,
                                                 T* __restrict__ u1, int nx, int64_t sp, int64_t npad, T omega,
                                                 int sweeps) {
    for (int it = 0; it < sweeps; ++it) {
        const T* in = (it & 1) ? u0 : u1;
        T* out = (it & 1) ? u1 : u0;
        for (int64_t t = threadIdx.x; t < npad; t += blockDim.x) {
            if (it == 0) {
                out[t] = mg_div(omega * b[t], o.d[t]);
            } else {
                const T r = b[t] - mg_apply(o, in, t, nx, sp, npad);
                out[t] = in[t] + mg_div(omega * r, o.d[t]);
            }
        }
        __syncthreads();
    }
}
template <typename T>
__global__ __launch_bounds__(1024) void k_mg_coarse(Op<T> op, const T* __restrict__ b, T* __restrict__ buf0,
                                                    T* __restrict__ buf1, int nx, int64_t sp, int64_t npad, T omega,
                                                    int sweeps, int lds, const SyncState* S) {
    if (S && stop(S)) return;
    if (!lds) {
        mg_coarse_sweeps(op, b, buf0, buf1, nx, sp, npad, omega, sweeps);
        return;
    }
    extern __shared__ __align__(16) unsigned char coarse_lds[];
    T* cx = reinterpret_cast<T*>(coarse_lds);
    T* cy = cx + npad;
    T* cz = cy + npad;
    T* d = cz + npad;
    T* bl = d + npad;
    T* u0 = bl + npad;
    T* u1 = u0 + npad;
    for (int64_t t = threadIdx.x; t < npad; t += blockDim.x) {
        cx[t] = op.cx[t];
        cy[t] = op.cy[t];
        cz[t] = op.cz[t];
        d[t] = op.d[t];
        bl[t] = b[t];
    }
    __syncthreads();
    mg_coarse_sweeps(Op<T>{cx, cy, cz, d}, (const T*)bl, u0, u1, nx, sp, npad, omega, sweeps);
    const T* res = ((sweeps - 1) & 1) ? u1 : u0;
    T* dst = ((sweeps - 1) & 1) ? buf1 : buf0;
    for (int64_t t = threadIdx.x; t < npad; t += blockDim.x) dst[t] = res[t];
}

// Outer-iteration pieces: p = z with the sums r.z, r.r, b.b; and r.z, r.r.
template <typename T>
__global__ __launch_bounds__(kBS) void k_mg_init_dots(const T* __restrict__ r, const T* __restrict__ z,
                                                      const T* __restrict__ b, T* __restrict__ p, int64_t npad,
                                                      int64_t per, double* __restrict__ partials) {
    double acc[3] = {0.0, 0.0, 0.0};
    const int64_t lo = (int64_t)blockIdx.x * per, hi = min(lo + per, npad);
    for (int64_t t = lo + threadIdx.x; t < hi; t += kBS) {
        p[t] = z[t];
        acc[0] += (double)r[t] * (double)z[t];
        acc[1] += (double)r[t] * (double)r[t];
        acc[2] += (double)b[t] * (double)b[t];
    }
    block_sum_store<3>(acc, partials + (size_t)blockIdx.x * kMaxPartials);
}

// r.z and r.r block sums (the outer iteration's, when the hierarchy has a
// single level and the V-cycle has no post-smoothing sweep to fuse them into).
template <typename T>
__global__ __launch_bounds__(kBS) void k_mg_dot2(const T* __restrict__ r, const T* __restrict__ z, int64_t npad,
                                                 int64_t per, double* __restrict__ partials, const SyncState* S) {
    if (stop(S)) return;
    double acc[2] = {0.0, 0.0};
    const int64_t lo = (int64_t)blockIdx.x * per, hi = min(lo + per, npad);
    for (int64_t t = lo + threadIdx.x; t < hi; t += kBS) {
        acc[0] += (double)r[t] * (double)z[t];
        acc[1] += (double)r[t] * (double)r[t];
    }
    block_sum_store<2>(acc, partials + (size_t)blockIdx.x * kMaxPartials);
}

template <typename T>
__global__ void k_mg_sub(const T* __restrict__ b, const T* __restrict__ q, T* __restrict__ r, int64_t npad) {
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < npad;
         t += (int64_t)gridDim.x * blockDim.x)
        r[t] = b[t] - q[t];
}

struct LevelShape {
    Layout L;
    double h;
};

std::vector<LevelShape> level_shapes(const Layout& L0, double h) {
    std::vector<LevelShape> v{{L0, h}};
    for (;;) {
        const Layout& L = v.back().L;
        if (std::min(L.nx, std::min(L.ny, L.nz)) / 2 < 3 || L.n <= kMgMinNodes) break;
        v.push_back({make_layout(L.nx / 2, L.ny / 2, L.nz / 2), 2.0 * v.back().h});
    }
    return v;
}

template <typename T>
struct MgLevel {
    Layout L;
    double h;
    Op<T> op;
    T *b, *xa, *xb, *r;                 // right-hand side, two iterate buffers, residual (flat sweeps)
    double *ex, *ey, *ez, *k2;          // this level's edges and kbar^2 (coarse levels)
    uint32_t* codes;                    // level 0, FP32: code words of the operator
    void* code_scratch;
};

// Whether k_mg_march takes a grid: the planes of its shortest chunk, halo
// included, within the 2^31 bytes of its offsets.
bool march_fits(const Layout& L) { return 9 * 4 * L.sp <= (int64_t)0x7fffffff; }

// Workspace carving (nullptr base: sizes only). Level 0 borrows the solve's
// operator, residual and z buffers.
template <typename T>
size_t mg_carve(void* base, const Layout& L0, double h, std::vector<MgLevel<T>>* out) {
    size_t off = 0;
    auto take = [&](size_t bytes) -> void* {
        const size_t o = off;
        off = align_up(off + bytes, 256);
        return base ? (void*)((char*)base + o) : nullptr;
    };
    const auto shapes = level_shapes(L0, h);
    for (size_t l = 0; l < shapes.size(); ++l) {
        MgLevel<T> m{};
        m.L = shapes[l].L;
        m.h = shapes[l].h;
        const size_t nT = sizeof(T) * (size_t)m.L.npad;
        if (l > 0) {
            const Layout& L = m.L;
            m.ex = (double*)take(sizeof(double) * (size_t)(L.nx + 1) * L.ny * L.nz);
            m.ey = (double*)take(sizeof(double) * (size_t)L.nx * (L.ny + 1) * L.nz);
            m.ez = (double*)take(sizeof(double) * (size_t)L.nx * L.ny * (L.nz + 1));
            m.k2 = (double*)take(sizeof(double) * (size_t)L.n);
            m.op.cx = (T*)take(nT);
            m.op.cy = (T*)take(nT);
            m.op.cz = (T*)take(nT);
            m.op.d = (T*)take(nT);
            m.b = (T*)take(nT);
            m.xa = (T*)take(nT);
        }
        m.xb = (T*)take(nT);
        if (sizeof(T) == 8 || !march_fits(L0)) m.r = (T*)take(nT);
        if (l == 0 && sizeof(T) == 4) {   // level 0's code words and the dictionary build's scratch
            m.codes = (uint32_t*)take(4 * (size_t)m.L.npad);
            m.code_scratch = take(coded_scratch_bytes());
        }
        if (out) out->push_back(m);
    }
    return off;
}

unsigned mg_grid(int64_t n) { return stream_grid(n); }

// The outer iteration's r.z and r.r taken in the finest level's last sweep
// (nblk, per: the ranges of FP64); sums: how many block sums there are.
struct DotFuse {
    double* partials;
    int nblk;
    int64_t per;
    int sums;
};

template <typename T>
__global__ void k_mg_zero_pads(T* __restrict__ a, int64_t plane, int64_t sp, int64_t n) {
    const int64_t gap = sp - plane;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x)
        a[t / gap * sp + plane + t % gap] = T(0);
}

// ---- FP32: one pass per leg of the V-cycle
//
// A sweep by itself reads and writes whole arrays for some 50 instructions a
// node, and on the coarse levels lasts less than its launch. Here a workgroup
// marches a tile of columns through the planes of a chunk and carries several
// operations along, each one plane behind the one before it:
//   down       x1 = omega b / d (plane k), x2 = the second sweep (k-1), r = b - A x2
//              (k-2), its restriction (k-3): b and the operator in, x2 and the
//              coarse right-hand side out;
//   up         x = x2 + P xc (k), the two post-smoothing sweeps (k-1, k-2), and
//              on level 0 the sums r.z and r.r;
//   direction  p = z + beta p_old (k), q = A p (k-1) and p.q.
// The tile with its halo is one column per thread; a plane's values and x- and
// y-couplings lie in LDS for the neighbours, the column's own planes above and
// below in registers; one barrier per plane. The halo (2 to 3 columns a side
// and 2 planes a chunk's end) is computed again by each tile that needs it:
// 1.3 to 1.4 of the nodes, cheaper than the passes over memory it replaces.
// Nodes outside the grid are zero. Each value is made by the same operations for
// the code words as for the arrays.
//
// Bound by instruction issue (about 50 vector, 16 LDS and 30 scalar ones a plane
// and wave): four planes are unrolled so that the last planes' registers and LDS
// buffers need no moves or index sums, and the arrays share one scalar offset
// (80 scalar instructions without that: 103 us up, 91 now at 257^3). 64 VGPRs and
// under 80 KB of LDS keep two workgroups of 1024 on a compute unit.
// Level 0 of 257^3 in FP32, code words: the way down 90 + 85 + 82 + 44 -> 76 us (as
// update's share, sweep, residual, restriction before), up 47 + 85 + 84 -> 93, the
// direction 133 -> 89; 128^3, arrays: 40 -> 27 down and 32 -> 25 up; 32^3: 15 -> 7 and
// 14 -> 7, where the chain of planes in a chunk bounds it. A whole iteration,
// coarser levels included, 1000 -> 530 us at 257^3 and 230 -> 140 us at 129^3.
struct MgGeo {
    int nx, ny, nz, ncx, ncy, ncz;   // this level and the next coarser one
    int64_t sp, spc;
    int tx, ty, chunk, jobs;         // tiles, planes per chunk (even), tiles x chunks
};
enum { kMgDown, kMgUp, kMgDir };
// Owned columns of a tile of NT threads; with its halo 33 x 31, 32 x 32 and 32 x 32
// columns, or 17 x 15, 16 x 16 and 16 x 16. Whole coarse cells, so even.
template <int MODE, int NT> struct MgTile {
    static constexpr int lo = MODE == kMgDir ? 1 : 2;                        // halo before, after
    static constexpr int hi = MODE == kMgDown ? 3 : (MODE == kMgUp ? 2 : 1);
    static constexpr int side = NT == 1024 ? 32 : 16;
    static constexpr int fx = MODE == kMgDir ? side - 2 : side - 4, fy = MODE == kMgDown ? fx - 2 : fx;
    static constexpr int rx = fx + lo + hi, ry = fy + lo + hi;
    static constexpr int pad = side + 2, plane = NT + 2 * pad;   // neighbours of the tile's corners
    static_assert(rx * ry <= NT && rx < pad, "one column per thread");
};

// Arrays through raw buffer resources that start at the first plane a job reads:
// a plane's offset is one scalar for all of them, and lanes without a node carry
// an offset past every resource, read zero and store nothing.
using MgRsrc = __amdgpu_buffer_rsrc_t;
constexpr uint32_t kMgNoNode = 0x80000000u;
__device__ __forceinline__ MgRsrc mg_rsrc(const void* base, int64_t first) {
    return __builtin_amdgcn_make_buffer_rsrc((char*)const_cast<void*>(base) + 4 * first, 0, 0x7fffffff, 0x00020000);
}
__device__ __forceinline__ uint32_t mg_ldw(MgRsrc r, uint32_t at, int plane) {
    return __builtin_amdgcn_raw_buffer_load_b32(r, (int)at, plane, 0);
}
__device__ __forceinline__ float mg_ld(MgRsrc r, uint32_t at, int plane) {
    return __builtin_bit_cast(float, mg_ldw(r, at, plane));
}
__device__ __forceinline__ void mg_st(float v, MgRsrc r, uint32_t at, int plane) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, (int)at, plane, 0);
}

// Readers: what a column fetches of its operator row, and the values in it.
struct MgRow4 {
    float cx, cy, cz, d;
};
struct ArrCol {
    const float *pcx, *pcy, *pcz, *pd;
    static constexpr int depth = 1;   // planes fetched ahead
    using Raw = MgRow4;
    struct Rsrc { MgRsrc cx, cy, cz, d; };
    __device__ __forceinline__ void bind() {}
    __device__ __forceinline__ Rsrc open(int64_t first) const {
        return {mg_rsrc(pcx, first), mg_rsrc(pcy, first), mg_rsrc(pcz, first), mg_rsrc(pd, first)};
    }
    __device__ __forceinline__ Raw fetch(const Rsrc& r, uint32_t at, int plane) const {
        return {mg_ld(r.cx, at, plane), mg_ld(r.cy, at, plane), mg_ld(r.cz, at, plane), mg_ld(r.d, at, plane)};
    }
    __device__ __forceinline__ MgRow4 decode(const Raw& w) const { return w; }
};
struct CodeCol {
    const uint32_t* pw;
    const float* dict;
    const float* tab;    // the dictionary's LDS copy, set by bind()
    static constexpr int depth = 2;
    using Raw = uint32_t;
    using Rsrc = MgRsrc;
    __device__ __forceinline__ void bind() {
        __shared__ float s_tab[kCodedTableSize];
        for (int i = threadIdx.x; i < kCodedTableSize; i += blockDim.x) s_tab[i] = dict[i];
        __syncthreads();
        tab = s_tab;
    }
    __device__ __forceinline__ Rsrc open(int64_t first) const { return mg_rsrc(pw, first); }
    __device__ __forceinline__ Raw fetch(Rsrc r, uint32_t at, int plane) const { return mg_ldw(r, at, plane); }
    __device__ __forceinline__ MgRow4 decode(Raw w) const {
        return {tab[w & 255u], tab[(w >> 8) & 255u], tab[(w >> 16) & 255u], tab[w >> 24]};
    }
};

// Sum over the workgroup, in a fixed order; valid in thread 0.
template <int NT>
__device__ __forceinline__ double mg_block_sum(double v, double* s) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < NT / 64; ++w) r += s[w];
    return r;
}

// in: x2 (up), z (direction); in2: the next coarser level's correction (up),
// p_old (direction). out: x2 (down), z (up), p (direction); out2: the next
// coarser right-hand side (down), q (direction). Results go to other buffers
// than the inputs (tiles read each other's nodes). Workgroups take jobs
// blockIdx, blockIdx + gridDim, ...; partials: with sums, one entry per workgroup.
template <int MODE, int NT, typename RD>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(8))) void k_mg_march(RD op, const float* __restrict__ b,
                                                         const float* __restrict__ in, const float* __restrict__ in2,
                                                         float* __restrict__ out, float* __restrict__ out2, MgGeo G,
                                                         float omega, double* __restrict__ partials,
                                                         const SyncState* S) {
    using Tile = MgTile<MODE, NT>;
    if (S && stop(S)) return;
    __shared__ float s_v0[4][Tile::plane], s_cx[4][Tile::plane], s_cy[4][Tile::plane];
    __shared__ float s_v1[2][MODE == kMgDir ? 1 : Tile::plane];
    __shared__ float s_r[2][MODE == kMgDown ? Tile::plane : 1];
    __shared__ double s_sum[NT / 64];
    op.bind();
    const int ly = threadIdx.x / Tile::rx, lx = threadIdx.x - ly * Tile::rx, c = Tile::pad + threadIdx.x;
    const bool owned_xy = lx >= Tile::lo && lx < Tile::lo + Tile::fx && ly >= Tile::lo && ly < Tile::lo + Tile::fy;
    float beta = 0.0f;
    if constexpr (MODE == kMgDir) beta = (float)S->beta;
    double acc0 = 0.0, acc1 = 0.0;
    // the eight XCDs take runs of neighbouring tiles each
    const int per8 = (G.jobs + 7) / 8;
    for (int id = blockIdx.x; id < per8 * 8; id += gridDim.x) {
        const int job = (id & 7) * per8 + (id >> 3);
        if (job >= G.jobs) continue;
        const int tile = job % (G.tx * G.ty), x0 = tile % G.tx * Tile::fx, y0 = tile / G.tx * Tile::fy;
        const int z0 = job / (G.tx * G.ty) * G.chunk, z1 = min(z0 + G.chunk, (G.nz + 1) & ~1);
        const int i = x0 + lx - Tile::lo, j = y0 + ly - Tile::lo;
        const bool col = i >= 0 && i < G.nx && j >= 0 && j < G.ny && ly < Tile::ry;
        const bool own = owned_xy && col;
        const uint32_t at = col ? 4u * (uint32_t)(j * G.nx + i) : kMgNoNode, to = own ? at : kMgNoNode;
        // up: byte offsets of the four coarse nodes around the column, whose mean is
        // the value on a coarse plane: an odd coordinate's node counts twice, one
        // outside the grid lies past the plane and reads as zero
        uint32_t o[4];
        if constexpr (MODE == kMgUp) {
            const int I = (i - 1) >> 1, J = (j - 1) >> 1;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int ci = I + ((u & 1) & ~i), cj = J + ((u >> 1) & ~j);
                o[u] = col && ci >= 0 && ci < G.ncx && cj >= 0 && cj < G.ncy ? 4u * (uint32_t)(cj * G.ncx + ci)
                                                                           : kMgNoNode;
            }
        }
        auto coarse = [&](int K) {   // mean of the four on the coarse plane K
            if (K < 0 || K >= G.ncz) return 0.0f;
            const MgRsrc r = mg_rsrc(in2, K * G.spc);
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = mg_ld(r, o[u], 0);
            return 0.25f * ((v[0] + v[1]) + (v[2] + v[3]));
        };
        // down: the thread's coarse node, its corner in a plane of LDS and its place
        int cq = 0;
        uint32_t toc = kMgNoNode;
        if constexpr (MODE == kMgDown) {
            const int J = threadIdx.x / (Tile::fx / 2), I = threadIdx.x - J * (Tile::fx / 2);
            const int ci = x0 / 2 + I, cj = y0 / 2 + J;
            cq = Tile::pad + (2 * J + Tile::lo) * Tile::rx + 2 * I + Tile::lo;
            if (J < Tile::fy / 2 && ci < G.ncx && cj < G.ncy) toc = 4u * (uint32_t)(cj * G.ncx + ci);
        }
        const int k0 = z0 - Tile::lo;
        const int end = MODE == kMgDown ? z1 + 3 : (MODE == kMgUp ? z1 + 1 : z1);   // last step
        // planes read, from `first` on, and planes owned, from z0 on
        const int first = max(k0, 0), nread = min(z1 + Tile::hi, G.nz) - first, nown = min(z1, G.nz) - z0;
        const int sp = 4 * (int)G.sp;
        const int64_t base = first * G.sp;
        const typename RD::Rsrc rw = op.open(base);
        const MgRsrc rb = mg_rsrc(b, base), ri = mg_rsrc(in, base), ri2 = mg_rsrc(in2, base), ro = mg_rsrc(out, base),
                     ro2 = mg_rsrc(out2, base);
        constexpr int D = RD::depth;
        constexpr bool keep = D > 1 || MODE != kMgUp;   // registers for all own values, else LDS for some
        typename RD::Raw w[D] = {};
        float fb[D] = {}, f0[D] = {}, f1[D] = {}, fc = 0.0f;   // b; in, in2; the coarse plane of an even k
        auto fetch = [&](int k, int plane, int u, bool even) {
            if ((unsigned)(k - first) >= (unsigned)nread) return;
            w[u] = op.fetch(rw, at, plane);
            if constexpr (MODE != kMgDir) fb[u] = mg_ld(rb, at, plane);
            if constexpr (MODE != kMgDown) f0[u] = mg_ld(ri, at, plane);
            if constexpr (MODE == kMgDir) f1[u] = mg_ld(ri2, at, plane);
            if constexpr (MODE == kMgUp)
                if (even) fc = coarse(k >> 1);
        };
        int plane = (k0 - first) * sp;   // offset of plane k
#pragma unroll
        for (int u = 0; u < D; ++u) fetch(k0 + u, plane + u * sp, u, u == 0);
        float cnow = MODE == kMgUp ? coarse((k0 >> 1) - 1) : 0.0f;
        // the column's last planes, by plane - k0 modulo 4; nodes outside the grid have
        // the value zero (their couplings then do not matter)
        float cx[4] = {}, cy[4] = {}, cz[4] = {}, d[4] = {}, bv[4] = {}, v0[4] = {}, v1[4] = {};
        bool node[4] = {};
        float rsum = 0;      // down: a coarse node's restriction so far
        __syncthreads();     // the job before has left the LDS
        auto step = [&](int k, auto slot) {
            constexpr int e0 = decltype(slot)::value, e1 = (e0 + 3) & 3, e2 = (e0 + 2) & 3, e3 = (e0 + 1) & 3;
            constexpr int u = e0 & (D - 1), q0 = e0 & 1, q1 = q0 ^ 1;
            constexpr bool even = q0 == 0;   // k - k0, and with it k (up, down)
            const MgRow4 a = op.decode(w[u]);
            cx[e0] = a.cx; cy[e0] = a.cy; cz[e0] = a.cz; d[e0] = a.d;
            node[e0] = col && (unsigned)(k - first) < (unsigned)nread;
            if constexpr (MODE != kMgDir) bv[e0] = fb[u];
            float v;
            if constexpr (MODE == kMgDown) v = mg_div(omega * bv[e0], d[e0]);
            if constexpr (MODE == kMgDir) v = mg_fma(beta, f1[u], f0[u]);
            if constexpr (MODE == kMgUp) {
                v = f0[u] + (even ? 0.5f * (cnow + fc) : cnow);
                if (even) cnow = fc;
            }
            v0[e0] = node[e0] ? v : 0.0f;
            fetch(k + D, plane + D * sp, u, (e0 + D) % 2 == 0);
            s_v0[e0][c] = v0[e0];
            s_cx[e0][c] = cx[e0];
            s_cy[e0][c] = cy[e0];
            if constexpr (MODE == kMgDir)
                if ((unsigned)(k - z0) < (unsigned)nown) mg_st(v0[e0], ro, to, plane);
            lds_barrier();
            // plane k-1: the operator on v0
            float nb = (keep ? cx[e1] : s_cx[e1][c]) * s_v0[e1][c + 1];
            nb = mg_fma(s_cx[e1][c - 1], s_v0[e1][c - 1], nb);
            nb = mg_fma(keep ? cy[e1] : s_cy[e1][c], s_v0[e1][c + Tile::rx], nb);
            nb = mg_fma(s_cy[e1][c - Tile::rx], s_v0[e1][c - Tile::rx], nb);
            nb = mg_fma(cz[e1], v0[e0], nb);
            nb = mg_fma(cz[e2], keep ? v0[e2] : s_v0[e2][c], nb);
            const float av = mg_fma(d[e1], v0[e1], -nb);
            const bool in1 = (unsigned)(k - 1 - z0) < (unsigned)nown;
            if constexpr (MODE == kMgDir) {
                if (in1) {
                    mg_st(av, ro2, to, plane - sp);
                    acc0 = __builtin_fma((double)v0[e1], (double)(own ? av : 0.0f), acc0);
                }
            } else {
                const float x = v0[e1] + mg_div(omega * (bv[e1] - av), d[e1]);
                v1[e1] = node[e1] ? x : 0.0f;
                s_v1[q1][c] = v1[e1];
                if constexpr (MODE == kMgDown)
                    if (in1) mg_st(v1[e1], ro, to, plane - sp);
                // plane k-2: the operator on v1
                float nc = (keep ? cx[e2] : s_cx[e2][c]) * s_v1[q0][c + 1];
                nc = mg_fma(s_cx[e2][c - 1], s_v1[q0][c - 1], nc);
                nc = mg_fma(keep ? cy[e2] : s_cy[e2][c], s_v1[q0][c + Tile::rx], nc);
                nc = mg_fma(s_cy[e2][c - Tile::rx], s_v1[q0][c - Tile::rx], nc);
                nc = mg_fma(cz[e2], v1[e1], nc);
                nc = mg_fma(cz[e3], v1[e3], nc);
                const float r = bv[e2] - mg_fma(d[e2], v1[e2], -nc);
                if constexpr (MODE == kMgUp) {
                    if ((unsigned)(k - 2 - z0) < (unsigned)nown) {
                        const float z = v1[e2] + mg_div(omega * r, d[e2]);
                        mg_st(z, ro, to, plane - 2 * sp);
                        if (partials) {
                            const double bd = (double)(own ? bv[e2] : 0.0f);
                            acc0 = __builtin_fma(bd, (double)(own ? z : 0.0f), acc0);
                            acc1 = __builtin_fma(bd, bd, acc1);
                        }
                    }
                } else {
                    s_r[q0][c] = node[e2] ? r : 0.0f;
                    // plane k-3: weights (1,2,1) in each direction, /64 in all
                    constexpr int ncol = (Tile::fx / 2) * (Tile::fy / 2);
                    const int m = k - 3;
                    if (m >= z0 && threadIdx.x < ncol) {
                        const float* q = &s_r[q1][cq];
                        float t = 0.0f;
#pragma unroll
                        for (int y = 0; y < 3; ++y) {
                            const float row = mg_fma(2.0f, q[y * Tile::rx + 1], q[y * Tile::rx] + q[y * Tile::rx + 2]);
                            t = mg_fma(y == 1 ? 2.0f : 1.0f, row, t);
                        }
                        t *= 0.015625f;
                        if (even) {   // m odd: the coarse plane's middle
                            rsum = mg_fma(2.0f, t, rsum);
                        } else {
                            const int K = (m >> 1) - 1;
                            if (m > z0 && K < G.ncz)
                                mg_st(rsum + t, mg_rsrc(out2, K * G.spc), toc, 0);
                            rsum = t;
                        }
                    }
                }
            }
            plane += sp;
        };
        for (int k = k0; k <= end; k += 4) {
            step(k, std::integral_constant<int, 0>{});
            if (k + 1 <= end) step(k + 1, std::integral_constant<int, 1>{});
            if (k + 2 <= end) step(k + 2, std::integral_constant<int, 2>{});
            if (k + 3 <= end) step(k + 3, std::integral_constant<int, 3>{});
        }
    }
    if (MODE != kMgDown && partials) {
        const double t0 = mg_block_sum<NT>(acc0, s_sum);
        const double t1 = MODE == kMgUp ? mg_block_sum<NT>(acc1, s_sum) : 0.0;
        if (threadIdx.x == 0) {
            double* dst = partials + (size_t)blockIdx.x * kMaxPartials;
            dst[0] = t0;
            if constexpr (MODE == kMgUp) dst[1] = t1;
        }
    }
}

// Planes per chunk: the even number for which the rounds of workgroups (two per
// compute unit) times the planes each marches, halo included, are fewest.
template <int MODE, int NT>
MgGeo march_geo(const Layout& L, const Layout* C) {
    using Tile = MgTile<MODE, NT>;
    MgGeo G{};
    G.nx = L.nx; G.ny = L.ny; G.nz = L.nz; G.sp = L.sp;
    if (C) { G.ncx = C->nx; G.ncy = C->ny; G.ncz = C->nz; G.spc = C->sp; }
    G.tx = (L.nx + Tile::fx - 1) / Tile::fx;
    G.ty = (L.ny + Tile::fy - 1) / Tile::fy;
    const int64_t tiles = (int64_t)G.tx * G.ty, cap = 2048 / NT * kMgCus;
    int64_t best = INT64_MAX;
    for (int chunk = 2; chunk <= L.nz + 1; chunk += 2) {
        const int64_t jobs = tiles * ((L.nz + chunk - 1) / chunk);
        const int64_t cost = (jobs + cap - 1) / cap * (chunk + 6);
        if (cost < best && jobs < (1ll << 30) && (chunk == 2 || 4 * (chunk + 7) * L.sp <= (int64_t)0x7fffffff)) {
            best = cost;
            G.chunk = chunk;
            G.jobs = (int)jobs;
        }
    }
    return G;
}
// Workgroups: as many as reside at once (multiples of eight: one run of tiles per XCD).
template <int NT>
unsigned march_grid(const MgGeo& G) { return (unsigned)std::min((G.jobs + 7) / 8 * 8, 2048 / NT * kMgCus); }

struct MgReader {
    bool coded;
    CodeCol cg;
    ArrCol ag;
};
// Levels of up to 2^20 nodes take tiles of 256 threads: more of them, and a
// quarter of the instructions in each step of the chain (64^3 down 12 us against 16,
// up 10 against 14); from there on the large tile's smaller halo wins (128^3 down
// 27 us against 36).
constexpr int64_t kMgSmallTile = 1 << 20;
// One pass of a level's leg; returns the number of workgroups (block sums).
template <int MODE>
unsigned march(const MgReader& rd, const Layout& L, const Layout* C, const float* b, const float* in, const float* in2,
               float* out, float* out2, float omega, double* partials, const SyncState* S, hipStream_t st) {
    auto run = [&](auto nt, auto r) {
        constexpr int NT = decltype(nt)::value;
        const MgGeo G = march_geo<MODE, NT>(L, C);
        const unsigned grid = march_grid<NT>(G);
        hipLaunchKernelGGL((k_mg_march<MODE, NT, decltype(r)>), dim3(grid), dim3(NT), 0, st, r, b, in, in2, out, out2,
                           G, omega, partials, S);
        return grid;
    };
    if (rd.coded)
        return L.n <= kMgSmallTile ? run(std::integral_constant<int, 256>{}, rd.cg)
                                   : run(std::integral_constant<int, 1024>{}, rd.cg);
    return L.n <= kMgSmallTile ? run(std::integral_constant<int, 256>{}, rd.ag)
                               : run(std::integral_constant<int, 1024>{}, rd.ag);
}

// ---- FP32: the bottom of the hierarchy
//
// The last two levels (the coarsest and, with at most 4096 nodes, the one
// above) in one workgroup: four nodes a thread above and one on the coarsest,
// operator and right-hand side in registers, iterates in LDS (natural order with
// a plane of zeros at both ends; couplings out of the grid are zero). Bound by the
// chain of sweeps, each an LDS round trip and a barrier. 16^3 and 8^3: 16 us, 36 in
// three launches.
struct MgBottomLevel {
    Op<float> op;
    int nx, ny, nz;
    int64_t sp;
};
constexpr int kMgBottomNodes = 4;   // per thread
struct MgRow {
    float cx, cxl, cy, cyl, cz, czl, d, b;
};
__device__ __forceinline__ MgRow mg_row(const MgBottomLevel& L, int n, int64_t& t) {
    MgRow r{0, 0, 0, 0, 0, 0, 1.0f, 0};
    t = -1;
    const int pl = L.nx * L.ny;
    if (n < pl * L.nz) {
        const int k = n / pl, q = n - k * pl;
        t = (int64_t)k * L.sp + q;
        r.cx = L.op.cx[t];
        r.cy = L.op.cy[t];
        r.cz = L.op.cz[t];
        r.d = L.op.d[t];
        r.cxl = q > 0 ? L.op.cx[t - 1] : 0.0f;
        r.cyl = q >= L.nx ? L.op.cy[t - L.nx] : 0.0f;
        r.czl = k > 0 ? L.op.cz[t - L.sp] : 0.0f;
    }
    return r;
}
// b - A x at the node of row r, x its place in LDS
__device__ __forceinline__ float mg_row_residual(const MgRow& r, const float* x, int nx, int pl) {
    float nb = r.cx * x[1];
    nb = mg_fma(r.cxl, x[-1], nb);
    nb = mg_fma(r.cy, x[nx], nb);
    nb = mg_fma(r.cyl, x[-nx], nb);
    nb = mg_fma(r.cz, x[pl], nb);
    nb = mg_fma(r.czl, x[-pl], nb);
    return r.b - mg_fma(r.d, x[0], -nb);
}
size_t mg_bottom_lds(const Layout& A, const Layout& C) {
    return sizeof(float) * 2 * (size_t)(A.n + 2 * A.plane + C.n + 2 * C.plane);
}
bool mg_bottom_fits(const Layout& A, const Layout& C) {
    return A.n <= 1024 * kMgBottomNodes && C.n <= 1024 && mg_bottom_lds(A, C) <= 64 * 1024;
}
__global__ __launch_bounds__(1024) void k_mg_bottom(MgBottomLevel A, MgBottomLevel C, const float* __restrict__ b,
                                                    float* __restrict__ out, float omega, int sweeps,
                                                    const SyncState* S) {
    if (S && stop(S)) return;
    extern __shared__ __align__(16) float bottom_lds[];
    const int pa = A.nx * A.ny, na = pa * A.nz, pc = C.nx * C.ny, nc = pc * C.nz;
    const int wa = na + 2 * pa, wc = nc + 2 * pc;
    float* xa = bottom_lds + pa;
    float* xb = xa + wa;
    float* ya = bottom_lds + 2 * wa + pc;
    float* yb = ya + wc;
    for (int i = threadIdx.x; i < 2 * (wa + wc); i += 1024) bottom_lds[i] = 0.0f;
    MgRow r[kMgBottomNodes];
    int64_t t[kMgBottomNodes], tc;
#pragma unroll
    for (int u = 0; u < kMgBottomNodes; ++u) {
        r[u] = mg_row(A, threadIdx.x + 1024 * u, t[u]);
        if (t[u] >= 0) r[u].b = b[t[u]];
    }
    MgRow rc = mg_row(C, threadIdx.x, tc);
    float x[kMgBottomNodes];
    const int n0 = threadIdx.x;
    // a sweep: from the values in `from` (x the node's own) into `to`
    auto sweep = [&](const float* from, float* to) {
#pragma unroll
        for (int u = 0; u < kMgBottomNodes; ++u)
            if (t[u] >= 0) {
                x[u] += mg_div(omega * mg_row_residual(r[u], from + n0 + 1024 * u, A.nx, pa), r[u].d);
                if (to) to[n0 + 1024 * u] = x[u];
            }
    };
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kMgBottomNodes; ++u) {
        x[u] = mg_div(omega * r[u].b, r[u].d);
        if (t[u] >= 0) xa[n0 + 1024 * u] = x[u];
    }
    __syncthreads();
    sweep(xa, xb);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kMgBottomNodes; ++u)
        if (t[u] >= 0) xa[n0 + 1024 * u] = mg_row_residual(r[u], xb + n0 + 1024 * u, A.nx, pa);
    __syncthreads();
    // restriction to the thread's coarse node, (1,2,1)/4 in each direction
    if (tc >= 0) {
        const int K = n0 / pc, J = (n0 - K * pc) / C.nx, I = n0 - K * pc - J * C.nx;
        float sum = 0.0f;
        for (int c = 0; c < 3; ++c)
            for (int v = 0; v < 3; ++v)
                for (int u = 0; u < 3; ++u) {
                    const int i = 2 * I + u, j = 2 * J + v, k = 2 * K + c;
                    const float w = (u == 1 ? 2.0f : 1.0f) * (v == 1 ? 2.0f : 1.0f) * (c == 1 ? 2.0f : 1.0f);
                    if (i < A.nx && j < A.ny && k < A.nz) sum = mg_fma(w, xa[(k * A.ny + j) * A.nx + i], sum);
                }
        rc.b = sum * 0.015625f;
    }
    float y = mg_div(omega * rc.b, rc.d);
    if (tc >= 0) ya[n0] = y;
    const float wd = mg_div(omega, rc.d);
    for (int s = 1; s < sweeps; ++s) {
        const float* from = (s & 1) ? ya : yb;
        float* to = (s & 1) ? yb : ya;
        __syncthreads();
        if (tc >= 0) {
            y = mg_fma(wd, mg_row_residual(rc, from + n0, C.nx, pc), y);
            to[n0] = y;
        }
    }
    __syncthreads();
    const float* ys = (sweeps - 1) & 1 ? yb : ya;
#pragma unroll
    for (int u = 0; u < kMgBottomNodes; ++u)
        if (t[u] >= 0) {
            const int n = n0 + 1024 * u, k = n / pa, j = (n - k * pa) / A.nx, i = n - k * pa - j * A.nx;
            const int I = (i - 1) >> 1, J = (j - 1) >> 1, K = (k - 1) >> 1;
            float add = 0.0f;
            for (int v = 0; v < 8; ++v) {   // an odd coordinate's node counts twice
                const int ci = I + ((v & 1) & ~i), cj = J + ((v >> 1 & 1) & ~j), ck = K + ((v >> 2) & ~k);
                if (ci >= 0 && ci < C.nx && cj >= 0 && cj < C.ny && ck >= 0 && ck < C.nz)
                    add += ys[(ck * C.ny + cj) * C.nx + ci];
            }
            x[u] = mg_fma(0.125f, add, x[u]);
            xb[n] = x[u];
        }
    __syncthreads();
    sweep(xb, xa);
    __syncthreads();
    sweep(xa, nullptr);
#pragma unroll
    for (int u = 0; u < kMgBottomNodes; ++u)
        if (t[u] >= 0) out[t[u]] = x[u];
}

// One V-cycle on level l from zero; returns the buffer holding the result.
// In FP64 the first two pre-smoothing sweeps run as one pass (k_mg_jacobi2z);
// FP32 takes each leg in one (k_mg_march; the flat kernels where a plane is too
// large for its offsets). With `fuse` the finest level's last
// post-smoothing sweep also stores the block sums of r.z and r.r. A single-level
// hierarchy has no such sweep; its caller takes those sums with k_mg_dot2.
// `rd0`: level 0's reader (FP32).
constexpr size_t kMgCoarseLds = 60 * 1024;   // dynamic LDS for the coarsest level's copies
static_assert(kMgNu == 2, "k_mg_jacobi2z and k_mg_march take two sweeps");

template <typename T>
T* vcycle(std::vector<MgLevel<T>>& lv, size_t l, const SyncState* S, hipStream_t st, DotFuse* fuse,
          const MgReader* rd0) {
    MgLevel<T>& m = lv[l];
    const Layout& L = m.L;
    const T om = (T)kMgOmega;
    if (l + 1 == lv.size()) {
        const size_t lds = 7 * sizeof(T) * (size_t)L.npad;
        const int use_lds = lds <= kMgCoarseLds ? 1 : 0;
        hipLaunchKernelGGL(k_mg_coarse<T>, dim3(1), dim3(1024), use_lds ? lds : 0, st, m.op, (const T*)m.b, m.xa,
                           m.xb, L.nx, L.sp, L.npad, om, kMgCoarseSweeps, use_lds, S);
        return ((kMgCoarseSweeps - 1) & 1) ? m.xb : m.xa;
    }
    MgLevel<T>& c = lv[l + 1];
    if constexpr (sizeof(T) == 4) if (march_fits(lv[0].L)) {
        if (l > 0 && l + 2 == lv.size() && mg_bottom_fits(L, c.L)) {
            auto level = [](const MgLevel<T>& v) { return MgBottomLevel{v.op, v.L.nx, v.L.ny, v.L.nz, v.L.sp}; };
            hipLaunchKernelGGL(k_mg_bottom, dim3(1), dim3(1024), mg_bottom_lds(L, c.L), st, level(m), level(c),
                               (const float*)m.b, m.xb, om, kMgCoarseSweeps, S);
            return m.xb;
        }
        const MgReader rd = l == 0 ? *rd0 : MgReader{false, {}, {m.op.cx, m.op.cy, m.op.cz, m.op.d}};
        march<kMgDown>(rd, L, &c.L, m.b, nullptr, nullptr, m.xa, c.b, om, nullptr, S, st);
        const float* zc = vcycle<T>(lv, l + 1, S, st, nullptr, nullptr);
        const unsigned sums = march<kMgUp>(rd, L, &c.L, m.b, m.xa, zc, m.xb, nullptr, om,
                                           fuse ? fuse->partials : nullptr, S, st);
        if (fuse) fuse->sums = (int)sums;
        return m.xb;
    }
    const unsigned g = mg_grid(L.npad);
    T* z = m.xa;
    hipLaunchKernelGGL(k_mg_jacobi2z<T>, dim3(g), dim3(kBS), 0, st, m.op, (const T*)m.b, z, L.nx, L.sp, L.npad,
                       om, S);
    hipLaunchKernelGGL(k_mg_residual<T>, dim3(g), dim3(kBS), 0, st, m.op, (const T*)m.b, (const T*)z, m.r, L.nx,
                       L.sp, L.npad, S);
    hipLaunchKernelGGL(k_mg_restrict<T>, plane_grid(c.L.sp, c.L.nz), dim3(kBS), 0, st, (const T*)m.r, L.nx, L.ny,
                       L.nz, L.sp, c.b, c.L.nx, c.L.ny, c.L.nz, c.L.sp, S);
    T* zc = vcycle<T>(lv, l + 1, S, st, nullptr, nullptr);
    hipLaunchKernelGGL(k_mg_prolong_add<T>, plane_grid((int64_t)(c.L.nx + 1) * (c.L.ny + 1), c.L.nz + 1),
                       dim3(kBS), 0, st, (const T*)zc, c.L.nx, c.L.ny, c.L.nz, c.L.sp, z, L.nx, L.ny, L.nz, L.sp,
                       S);
    hipLaunchKernelGGL(k_mg_jacobi<T>, dim3(g), dim3(kBS), 0, st, m.op, (const T*)m.b, (const T*)z, m.xb, L.nx,
                       L.sp, L.npad, om, S);
    if (fuse)
        hipLaunchKernelGGL(k_mg_jacobi_dot2<T>, dim3(fuse->nblk), dim3(kBS), 0, st, m.op, (const T*)m.b,
                           (const T*)m.xb, z, L.nx, L.sp, L.npad, om, fuse->per, fuse->partials, S);
    else
        hipLaunchKernelGGL(k_mg_jacobi<T>, dim3(g), dim3(kBS), 0, st, m.op, (const T*)m.b, (const T*)m.xb, z,
                           L.nx, L.sp, L.npad, om, S);
    return z;
}

}  // namespace

size_t mg_workspace_bytes(const Layout& L0, int prec) {
    return prec == PB_F64 ? mg_carve<double>(nullptr, L0, 1.0, nullptr) : mg_carve<float>(nullptr, L0, 1.0, nullptr);
}

// Multigrid-preconditioned CG. `ex..k2` are the caller's FP64 edge arrays
// (level 0 of the hierarchy); s.op is level 0's operator in T.
template <typename T>
pb_status mg_pcg_impl(const Layout& L0, double h, const double* ex, const double* ey, const double* ez,
                      const double* k2, const SolveBufs<T>& s, void* mgws, SyncState* S, double* partials,
                      double tol, int maxiter, hipStream_t st, SolveResult* res) {
    std::vector<MgLevel<T>> lv;
    mg_carve<T>(mgws, L0, h, &lv);
    lv[0].op = s.op;
    lv[0].ex = (double*)ex; lv[0].ey = (double*)ey; lv[0].ez = (double*)ez; lv[0].k2 = (double*)k2;
    lv[0].xa = s.z;      // (lv[0].b, the V-cycle's input, is the outer residual; set per iteration)
    const bool built = res && res->mg_built;
    for (size_t l = 1; l < lv.size() && !built; ++l) {
        const MgLevel<T>& f = lv[l - 1];
        MgLevel<T>& c = lv[l];
        const int64_t tot = (int64_t)(c.L.nx + 1) * c.L.ny * c.L.nz + (int64_t)c.L.nx * (c.L.ny + 1) * c.L.nz +
                            (int64_t)c.L.nx * c.L.ny * (c.L.nz + 1) + c.L.n;
        hipLaunchKernelGGL(k_mg_coarsen, dim3(mg_grid(tot)), dim3(kBS), 0, st, (const double*)f.ex, (const double*)f.ey,
                           (const double*)f.ez, (const double*)f.k2, f.L.nx, f.L.ny, f.L.nz, c.ex, c.ey, c.ez, c.k2,
                           c.L.nx, c.L.ny, c.L.nz);
        hipLaunchKernelGGL(k_mg_op<T>, dim3(mg_grid(c.L.npad)), dim3(kBS), 0, st, (const double*)c.ex,
                           (const double*)c.ey, (const double*)c.ez, (const double*)c.k2, c.L.nx, c.L.ny, c.L.nz,
                           c.L.sp, c.h * c.h, c.op);
    }
    PB_HIP(hipGetLastError());
    // level 0 in FP32 reads its operator as code words when the values fit
    // the dictionary (the same words and dictionary as the fused solver's)
    MgReader rd0{};
    const bool flat = sizeof(T) == 8 || !march_fits(L0);
    if constexpr (sizeof(T) == 4) if (!flat) {
        rd0.ag = {s.op.cx, s.op.cy, s.op.cz, s.op.d};
        if (built) {
            rd0.coded = res->mg_coded != 0;
            rd0.cg = {lv[0].codes, res->mg_tab, nullptr};
        } else if (coded_coefficients() && lv[0].codes) {
            bool fits = false;
            const float* tab = nullptr;
            const pb_status e = build_codes(s.op, L0.npad, lv[0].code_scratch, lv[0].codes, st, fits, &tab);
            if (e != PB_OK) return e;
            rd0.coded = fits;
            rd0.cg = {lv[0].codes, tab, nullptr};
        }
        if (res) {
            res->mg_coded = rd0.coded ? 1 : 0;
            res->mg_tab = rd0.cg.dict;
        }
        // the pad slots, which k_mg_march does not write and the flat kernels read
        auto zero_pads = [&](T* a, const Layout& L) {
            if (L.sp > L.plane)
                hipLaunchKernelGGL(k_mg_zero_pads<T>, dim3(mg_grid((L.sp - L.plane) * L.nz)), dim3(kBS), 0, st, a,
                                   L.plane, L.sp, (L.sp - L.plane) * L.nz);
        };
        if (!built) {
            zero_pads(lv[0].xb, L0);
            zero_pads(s.p1, L0);
            for (size_t l = 1; l < lv.size(); ++l) zero_pads(lv[l].b, lv[l].L);
        }
    }
    if (res) res->mg_built = 1;

    const int64_t npad = L0.npad;
    const Ranges R = ranges_for(npad);
    const unsigned g = stream_grid(npad);
    if (launch_fill<int>((int*)S, (int64_t)(sizeof(SyncState) / sizeof(int)), 0, st) != PB_OK) return PB_ERR_HIP;
    hipEvent_t ev[2] = {nullptr, nullptr};
    const bool timed = !(res && res->untimed);
    if (timed) {
        PB_HIP(hipEventCreate(&ev[0]));
        PB_HIP(hipEventCreate(&ev[1]));
    }
    if (timed) PB_HIP(hipEventRecord(ev[0], st));
    // r = b - A x0, z = M r, p = z. The residual and the direction
    // alternate between two buffers each: the fused kernels read the old
    // values around a node while writing the new ones.
    T* rb[2] = {s.r, s.r2};
    T* pb_[2] = {s.p0, s.p1};
    hipLaunchKernelGGL(k_mg_apply<T>, dim3(g), dim3(kBS), 0, st, s.op, (const T*)s.x, s.q, L0.nx, L0.sp, npad,
                       (const SyncState*)nullptr);
    hipLaunchKernelGGL(k_mg_sub<T>, dim3(g), dim3(kBS), 0, st, s.b, (const T*)s.q, rb[0], npad);
    lv[0].b = rb[0];
    T* z = vcycle<T>(lv, 0, nullptr, st, nullptr, &rd0);
    hipLaunchKernelGGL(k_mg_init_dots<T>, dim3(R.nblk), dim3(kBS), 0, st, (const T*)rb[0], (const T*)z, s.b, pb_[0],
                       npad, R.per, partials);
    hipLaunchKernelGGL(k_scalar_init, dim3(1), dim3(kBS), 0, st, S, (const double*)partials, R.nblk, tol, maxiter);
    PB_HIP(hipGetLastError());
    // Per iteration: p = z + beta p and q = A p with p.q (beta is 0 before the
    // first); alpha; x and r updated; the V-cycle, its last sweep with r.z and
    // r.r; beta.
    DotFuse fuse{partials, R.nblk, R.per, R.nblk};
    int it = 0;
    SyncState hs{};
    for (;;) {
        for (int u = 0; u < kPoll && it < maxiter; ++u, ++it) {
            T* pold = pb_[it & 1];
            T* pnew = pb_[(it + 1) & 1];
            T* rold = rb[it & 1];
            T* rnew = rb[(it + 1) & 1];
            int npq = R.nblk;   // block sums of p.q
            if constexpr (sizeof(T) == 4) {
                if (!flat)
                    npq = (int)march<kMgDir>(rd0, L0, nullptr, nullptr, z, pold, pnew, s.q, 0.0f, partials, S, st);
            }
            if (flat)
                hipLaunchKernelGGL(k_mg_direction_apply<T>, dim3(R.nblk), dim3(kBS), 0, st, s.op, (const T*)z,
                                   (const T*)pold, pnew, s.q, L0.nx, L0.sp, npad, R.per, partials,
                                   (const SyncState*)S);
            hipLaunchKernelGGL(k_scalar_alpha, dim3(1), dim3(kBS), 0, st, S, (const double*)partials, npq);
            lv[0].b = rnew;
            hipLaunchKernelGGL(k_mg_update<T>, dim3(g), dim3(kBS), 0, st, s.x, (const T*)pnew, (const T*)rold,
                               (const T*)s.q, rnew, npad, (const SyncState*)S);
            z = vcycle<T>(lv, 0, S, st, lv.size() > 1 ? &fuse : nullptr, &rd0);
            if (lv.size() == 1)
                hipLaunchKernelGGL(k_mg_dot2<T>, dim3(R.nblk), dim3(kBS), 0, st, (const T*)rnew, (const T*)z, npad,
                                   R.per, partials, (const SyncState*)S);
            hipLaunchKernelGGL(k_scalar_beta, dim3(1), dim3(kBS), 0, st, S, (const double*)partials,
                               fuse.sums, tol, maxiter);
        }
        PB_HIP(hipGetLastError());
        PB_HIP(hipMemcpyAsync(&hs, S, sizeof(SyncState), hipMemcpyDeviceToHost, st));
        PB_HIP(hipStreamSynchronize(st));
        if (hs.done || it >= maxiter) break;
    }
    if (timed) PB_HIP(hipEventRecord(ev[1], st));
    hipLaunchKernelGGL(k_zero_if_zero_rhs<T>, dim3(g), dim3(kBS), 0, st, s.x, npad, (const SyncState*)S);
    PB_HIP(hipGetLastError());
    PB_HIP(hipMemcpyAsync(&hs, S, sizeof(SyncState), hipMemcpyDeviceToHost, st));
    PB_HIP(hipStreamSynchronize(st));
    float ms = 0.0f;
    if (timed) {
        PB_HIP(hipEventElapsedTime(&ms, ev[0], ev[1]));
        (void)hipEventDestroy(ev[0]);
        (void)hipEventDestroy(ev[1]);
    }
    if (res) {
        res->kernel_seconds = 1e-3 * ms;
        res->status = hs.done ? hs.status : (int)PB_NOT_CONVERGED;
        res->iters = hs.iters;
        res->rr = hs.rr;
        res->bb = hs.bb;
    }
    return PB_OK;
}

template pb_status mg_pcg_impl<float>(const Layout&, double, const double*, const double*, const double*,
                                      const double*, const SolveBufs<float>&, void*, SyncState*, double*, double, int,
                                      hipStream_t, SolveResult*);
template pb_status mg_pcg_impl<double>(const Layout&, double, const double*, const double*, const double*,
                                       const double*, const SolveBufs<double>&, void*, SyncState*, double*, double,
                                       int, hipStream_t, SolveResult*);

}  // namespace pb
