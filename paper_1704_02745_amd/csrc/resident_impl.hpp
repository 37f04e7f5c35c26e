// Host side of the resident Jacobi-CG for one precision: the kernel variants,
// the choice of bricks and the launch. Included by one source file per
// precision, which lists its variants.
#pragma once

#include "resident_device.hpp"

#include <algorithm>
#include <mutex>
#include <vector>

namespace pb {
namespace {

struct ResVariant {
    int bs, nz;
    const void* fn[2];   // free, periodic
};
#define PB_RES_VARIANT(T, BS, NZ) \
    ResVariant { BS, NZ, { (const void*)k_jpcg_resident<T, BS, NZ, false>, (const void*)k_jpcg_resident<T, BS, NZ, true> } }

struct ResPlan {
    int bs, nz, tx, ty, nxt, nyt, nzc, grid;
    size_t lds;
    const void* fn;
};

struct ResDevice {
    int cus = 0, wallclock_khz = 0;
    size_t lds = 0;
};
ResDevice res_device() {
    static std::mutex mu;
    static std::vector<ResDevice> cache;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return ResDevice{};
    std::lock_guard<std::mutex> lk(mu);
    if ((int)cache.size() <= dev) cache.resize(dev + 1);
    if (cache[dev].cus == 0) {
        ResDevice d;
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess) d.cus = v;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeWallClockRate, dev) == hipSuccess) d.wallclock_khz = v;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess) d.lds = (size_t)v;
        cache[dev] = d;
    }
    return cache[dev];
}

template <typename T>
const std::vector<ResVariant>& res_variants();

// The bricks of a grid: the cheapest feasible (block, planes, tile) by a model
// of one pass (see resident_cost); grid = 0 when the state does not fit.
template <typename T>
ResPlan resident_plan(const Layout& L, int per) {
    ResPlan best{};
    const ResDevice di = res_device();
    const int cap = std::min(di.cus, kMaxResidentGroups);
    if (cap <= 0 || L.npad * (int64_t)sizeof(T) >= ((int64_t)1 << 31)) return best;
    double best_cost = 1e300;
    for (const ResVariant& v : res_variants<T>()) {
        const int nzc = (L.nz + v.nz - 1) / v.nz;
        if (nzc > cap) continue;
        for (int nxt = 1; nxt <= cap / nzc; ++nxt) {
            if (nxt > 1 && L.nx / nxt < 2) break;
            const int tx = (L.nx + nxt - 1) / nxt;
            if (tx > v.bs) continue;
            const int nyt = (L.ny + v.bs / tx - 1) / (v.bs / tx);
            if (nyt > 1 && L.ny / nyt < 2) continue;
            const int ty = (L.ny + nyt - 1) / nyt;
            const int64_t grid = (int64_t)nxt * nyt * nzc;
            if (grid > cap) continue;
            const size_t lds = resident_lds_bytes<T>(v.bs, v.nz, tx, ty);
            if (lds > 160 * 1024) continue;
            // published faces fit five of the six state arrays of the streaming
            // form (a warm start's residual takes the sixth)
            if ((grid > 1 || per) && 2 * grid * face_len(v.bs, v.nz, tx, ty) > 5 * L.npad) continue;
            const int halo = (nxt > 1 ? 2 * ty * v.nz : 0) + (nyt > 1 ? 2 * tx * v.nz : 0);
            // microseconds of one pass beyond its fixed part, fitted to sweeps of
            // block, planes and tile at 33^3-129^3: the planes of a thread (0.15
            // each with 512 threads), the halo nodes, the slots every workgroup
            // polls, and the strided x-faces
            const double cost = 0.149 * v.nz * v.bs / 512 + 0.1 * halo / v.bs + 0.0107 * grid + (nxt > 1 ? 0.2 : 0.0);
            if (cost < best_cost) {
                best_cost = cost;
                best = ResPlan{v.bs, v.nz, tx, ty, nxt, nyt, nzc, (int)grid, lds, v.fn[per ? 1 : 0]};
            }
        }
    }
    if (best.grid > 0) {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, best.fn, best.bs, best.lds) != hipSuccess ||
            nb * di.cus < best.grid)
            return ResPlan{};
    }
    return best;
}

// Initial residual b - A x0 of a warm start in the padded layout.
template <typename T>
__global__ void k_resident_start(Op<T> op, const T* __restrict__ b, const T* __restrict__ X, T* __restrict__ r, int nx,
                                 int ny, int nz, int64_t sp, int per) {
    const int64_t npad = sp * nz;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < npad; t += (int64_t)gridDim.x * blockDim.x) {
        const int k = (int)(t / sp);
        const int p = (int)(t - (int64_t)k * sp);
        const int j = p / nx, i = p - j * nx;
        if (j >= ny) {
            r[t] = T(0);
            continue;
        }
        auto at = [&](bool in, int64_t wrapped, int64_t there) { return in ? there : (per ? wrapped : (int64_t)-1); };
        const int64_t xr = at(i < nx - 1, t - (nx - 1), t + 1), xl = at(i > 0, t + (nx - 1), t - 1);
        const int64_t yu = at(j < ny - 1, t - (int64_t)(ny - 1) * nx, t + nx);
        const int64_t yd = at(j > 0, t + (int64_t)(ny - 1) * nx, t - nx);
        const int64_t zu = at(k < nz - 1, t - (int64_t)(nz - 1) * sp, t + sp);
        const int64_t zd = at(k > 0, t + (int64_t)(nz - 1) * sp, t - sp);
        T sum = xr >= 0 ? op.cx[t] * X[xr] : T(0);
        sum += xl >= 0 ? op.cx[xl] * X[xl] : T(0);
        sum += yu >= 0 ? op.cy[t] * X[yu] : T(0);
        sum += yd >= 0 ? op.cy[yd] * X[yd] : T(0);
        sum += zu >= 0 ? op.cz[t] * X[zu] : T(0);
        sum += zd >= 0 ? op.cz[zd] * X[zd] : T(0);
        r[t] = b[t] - (op.d[t] * X[t] - sum);
    }
}

template <typename T>
pb_status resident_solve(const Layout& L, const SolveBufs<T>& s, SyncState* sync, double* partials, double tol,
                         int maxiter, hipStream_t st, SolveResult* res, int periodic, bool& ran) {
    ran = false;
    // the state arrays of the streaming form, r to q2, hold the published faces
    if (!s.r || !s.q2 || s.q2 - s.r != 5 * L.npad) return PB_OK;
    const ResPlan p = resident_plan<T>(L, periodic);
    if (p.grid <= 0) return PB_OK;
    const ResDevice di = res_device();
    RArgs<T> a{};
    a.op = s.op;
    a.b = s.b;
    a.r0 = s.b;
    a.x = s.x;
    const int64_t half = (int64_t)p.grid * face_len(p.bs, p.nz, p.tx, p.ty);
    a.faces[0] = s.r;
    a.faces[1] = s.r + half;
    a.nx = L.nx; a.ny = L.ny; a.nz = L.nz;
    a.sp = L.sp;
    a.tx = p.tx; a.ty = p.ty;
    a.nxt = p.nxt; a.nyt = p.nyt; a.nzc = p.nzc;
    a.tol = tol;
    a.maxiter = maxiter;
    a.warm = s.warm;
    a.S = sync;
    a.slots = (unsigned long long*)partials;
    a.timeout_ticks = (long long)(di.wallclock_khz > 0 ? di.wallclock_khz : 100000) * 1000LL * 20LL;
    if (s.warm) {
        const unsigned nb = (unsigned)std::min<int64_t>((L.npad + 255) / 256, 8192);
        hipLaunchKernelGGL(k_resident_start<T>, dim3(nb), dim3(256), 0, st, s.op, s.b, (const T*)s.x, s.q2, L.nx, L.ny,
                           L.nz, L.sp, periodic);
        PB_HIP(hipGetLastError());
        a.r0 = s.q2;
    }
    if (launch_fill<int>((int*)sync, (int64_t)(sizeof(SyncState) / sizeof(int)), 0, st) != PB_OK) return PB_ERR_HIP;
    if (launch_fill<int>((int*)partials, (int64_t)2 * p.grid * kSlotWords * 2, 0, st) != PB_OK) return PB_ERR_HIP;
    hipEvent_t ev[2] = {nullptr, nullptr};
    const bool timed = res && !res->untimed;
    if (timed) {
        PB_HIP(hipEventCreate(&ev[0]));
        PB_HIP(hipEventCreate(&ev[1]));
        PB_HIP(hipEventRecord(ev[0], st));
    }
    void* args[] = {&a};
    const hipError_t e = hipLaunchCooperativeKernel(p.fn, dim3(p.grid), dim3(p.bs), args, p.lds, st);
    if (e != hipSuccess) {
        if (ev[0]) (void)hipEventDestroy(ev[0]);
        if (ev[1]) (void)hipEventDestroy(ev[1]);
        set_error("resident JPCG launch failed: %s (grid %d, block %d, lds %zu)", hipGetErrorString(e), p.grid, p.bs,
                  p.lds);
        return PB_ERR_HIP;
    }
    if (timed) PB_HIP(hipEventRecord(ev[1], st));
    ran = true;
    if (res) {
        SyncState h;
        PB_HIP(hipMemcpyAsync(&h, sync, sizeof(SyncState), hipMemcpyDeviceToHost, st));
        PB_HIP(hipStreamSynchronize(st));
        float ms = 0.0f;
        if (timed) {
            PB_HIP(hipEventElapsedTime(&ms, ev[0], ev[1]));
            (void)hipEventDestroy(ev[0]);
            (void)hipEventDestroy(ev[1]);
        }
        res->status = h.status;
        res->iters = h.iters;
        res->rr = h.rr;
        res->bb = h.bb;
        res->kernel_seconds = 1e-3 * ms;
        res->tiling = Tiling{};
        res->coded = 0;
        res->ctab = nullptr;
    }
    return PB_OK;
}

}  // namespace

template <typename T>
pb_status resident_jpcg(const Layout& L, const SolveBufs<T>& s, SyncState* sync, double* partials, double tol,
                        int maxiter, hipStream_t st, SolveResult* res, int periodic, bool& ran) {
    return resident_solve<T>(L, s, sync, partials, tol, maxiter, st, res, periodic, ran);
}
template <typename T>
bool resident_fits(const Layout& L, int periodic) {
    return resident_plan<T>(L, periodic).grid > 0;
}

}  // namespace pb
