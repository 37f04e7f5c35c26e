// Host side of the resident Jacobi-CG for one precision: the kernel variants,
// the choice of bricks and the launch. Included by one source file per
// precision, which lists its variants.
#pragma once

#include "resident_device.hpp"

#include <algorithm>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

namespace pb {
namespace {

struct ResVariant {
    int bs, nz;
    const void* fn[2];   // free, periodic
};
// compact: free and periodic kernels of the compact form
#define PB_RES_COMPACT(NZ)                                                     \
    ResVariant {                                                               \
        512, NZ, {                                                             \
            (const void*)k_jpcg_resident<float, 512, NZ, false, true>,         \
                (const void*)k_jpcg_resident<float, 512, NZ, true, true>       \
        }                                                                      \
    }
#define PB_RES_VARIANT(T, BS, NZ) \
    ResVariant { BS, NZ, { (const void*)k_jpcg_resident<T, BS, NZ, false>, (const void*)k_jpcg_resident<T, BS, NZ, true> } }

struct ResPlan {
    int bs, nz, tx, ty, nxt, nyt, nzc, grid;
    size_t lds;
    const void* fn;
    double us;   // modelled microseconds of a pass
};

struct ResDevice {
    int dev = -1, cus = 0, wallclock_khz = 0;
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
        d.dev = dev;
        cache[dev] = d;
    }
    return cache[dev];
}

template <typename T>
const std::vector<ResVariant>& res_variants();

template <typename T>
const void* batch_kernel(bool compact) {
    if constexpr (sizeof(T) == 4)
        if (compact) return (const void*)k_resident_batch<T, true, false>;
    return (const void*)k_resident_batch<T, false, false>;
}

// Microseconds of one pass, fitted to sweeps of block, planes and tile at
// 33^3-141^3: the barrier (its two memory latencies and the slots every workgroup
// polls, or two rounds of polling), the planes of a thread (0.15 each with 512
// threads), the halo nodes, and the strided x-faces.
double resident_pass_us(int bs, int nzb, int halo, int grid, bool split_x, bool compact) {
    const double barrier = slot_groups(nzb, grid, false) > 0 ? 3.8 : 2.4 + 0.0107 * grid;
    return barrier + (compact ? 0.19 : 0.149) * nzb * bs / 512 + 0.1 * halo / bs + (split_x ? 0.2 : 0.0);
}

// Every feasible way to cut a grid into bricks of `bs` threads and `nzb`
// planes, the cheapest by `cost` kept in `best`.
template <typename T, typename Cost>
void resident_search(const Layout& L, int per, int bs, int nzb, bool compact, int cap, int64_t face_room,
                     const void* fn, Cost&& cost, double& best_cost, ResPlan& best) {
    const int nzc = (L.nz + nzb - 1) / nzb;
    if (nzc > cap) return;
    // faces of one parity: both fit r where x takes p0 and p1 
    if (x_in_memory<T>(nzb, compact)) face_room = L.npad / 2;
    for (int nxt = 1; nxt <= cap / nzc; ++nxt) {
        if (nxt > 1 && L.nx / nxt < 2) break;   // a column is on one x-face at most
        const int tx = (L.nx + nxt - 1) / nxt;
        if (tx > bs) continue;
        const int nyt = (L.ny + bs / tx - 1) / (bs / tx);
        if (nyt > 1 && L.ny / nyt < 2) continue;
        const int ty = (L.ny + nyt - 1) / nyt;
        const int64_t grid = (int64_t)nxt * nyt * nzc;
        if (grid > cap) continue;
        // every halo column needs a thread; x by brick fits two state arrays
        if ((nxt > 1 ? 2 * ty : 0) + (nyt > 1 ? 2 * tx : 0) > bs) continue;
        if (x_in_memory<T>(nzb, compact) && grid * nzb * bs > 2 * L.npad) continue;
        const size_t lds = resident_lds_bytes<T>(bs, nzb, tx, ty, compact);
        if (lds + (compact ? sizeof(T) * 2 * kCodedTableSize : 0) > 160 * 1024) continue;
        if ((grid > 1 || per) && grid * face_len(bs, nzb, tx, ty) > face_room) continue;
        const int halo = (nxt > 1 ? 2 * ty * nzb : 0) + (nyt > 1 ? 2 * tx * nzb : 0);
        const double us = resident_pass_us(bs, nzb, halo, (int)grid, nxt > 1, compact), c = cost(us, (int)grid);
        if (c < best_cost) {
            best_cost = c;
            best = ResPlan{bs, nzb, tx, ty, nxt, nyt, nzc, (int)grid, lds, fn, us};
        }
    }
}

// The bricks of a grid; grid = 0 when its state does not fit the device. For a
// solve of its own the fastest pass counts; in a batch (batch = true, one
// kernel for all) the device time a pass takes, workgroups times microseconds:
// problems share the device, and each keeps its bricks in any mix. Plans are
// kept per device and shape (a host-side search of a few microseconds).
template <typename T>
ResPlan resident_plan(const Layout& L, int per, bool batch, bool compact) {
    ResPlan best{};
    const ResDevice di = res_device();
    const int cap = std::min(di.cus, kMaxResidentGroups);
    if (cap <= 0 || L.npad * (int64_t)sizeof(T) >= ((int64_t)1 << 31)) return best;
    using Key = std::tuple<int, int, int, int, int, bool, bool>;
    static std::mutex mu;
    static std::map<Key, ResPlan> kept;
    const Key key(di.dev, L.nx, L.ny, L.nz, per, batch, compact);
    {
        std::lock_guard<std::mutex> lk(mu);
        const auto it = kept.find(key);
        if (it != kept.end()) return it->second;
    }
    double best_cost = 1e300;
    if (batch) {
        // the faces of one parity in r, of the other in r2
        if (sizeof(T) == 4 || !compact)
            resident_search<T>(L, 0, 512, batch_planes<T>(compact), compact, cap, L.npad, batch_kernel<T>(compact),
                               [](double us, int grid) { return us * grid; }, best_cost, best);
    } else {
        // both parities in five of the six state arrays of the streaming form (a
        // warm start's residual takes the sixth)
        for (const ResVariant& v : res_variants<T>())
            if (compact == (v.nz >= kCompactFrom))
                resident_search<T>(L, per, v.bs, v.nz, compact, cap, 5 * L.npad / 2,
                                   v.fn[per ? 1 : 0], [](double us, int) { return us; }, best_cost, best);
    }
    if (best.grid > 0) {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, best.fn, best.bs, best.lds) != hipSuccess ||
            nb * di.cus < best.grid)
            best = ResPlan{};
    }
    std::lock_guard<std::mutex> lk(mu);
    if (kept.size() >= 4096) kept.clear();
    kept[key] = best;
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
RArgs<T> resident_args(const Layout& L, const SolveBufs<T>& s, const ResPlan& p, SyncState* sync,
                       unsigned long long* slots, double tol, int maxiter) {
    const ResDevice di = res_device();
    RArgs<T> a{};
    a.op = s.op;
    a.b = s.b;
    a.r0 = s.b;
    a.x = s.x;
    a.nx = L.nx; a.ny = L.ny; a.nz = L.nz;
    a.sp = L.sp;
    a.tx = p.tx; a.ty = p.ty;
    a.nxt = p.nxt; a.nyt = p.nyt; a.nzc = p.nzc;
    a.tol = tol;
    a.maxiter = maxiter;
    a.warm = s.warm;
    a.S = sync;
    a.slots = slots;
    // every wait is bounded: 20 s of the constant-rate clock
    a.timeout_ticks = (long long)(di.wallclock_khz > 0 ? di.wallclock_khz : 100000) * 1000LL * 20LL;
    a.first_timeout_ticks = a.timeout_ticks;
    return a;
}

// Bound of the wait in the first barrier of one of `problems` in a launch, in ticks:
// a workgroup may come to it from all the others, each of which may take a bounded
// wait and all its passes (by the model, which the real ones exceed up to twofold, more
// where the device is shared: ten times), and must not give up on them.
long long first_wait_ticks(long long wait_ticks, int problems, double pass_us, double ticks_per_us) {
    const double t = (double)wait_ticks * (1.0 + problems) + 10.0 * pass_us * ticks_per_us;
    return t < 4e18 ? (long long)t : (long long)4e18;
}

template <typename T>
pb_status launch_resident_start(const Layout& L, const Op<T>& op, const T* b, const T* x, T* r, int periodic,
                                hipStream_t st) {
    const unsigned nb = (unsigned)std::min<int64_t>((L.npad + 255) / 256, 8192);
    hipLaunchKernelGGL(k_resident_start<T>, dim3(nb), dim3(256), 0, st, op, b, x, r, L.nx, L.ny, L.nz, L.sp, periodic);
    PB_HIP(hipGetLastError());
    return PB_OK;
}

// cw, ctab: the compact form on these code words (null: the full form).
template <typename T>
pb_status resident_solve(const Layout& L, const SolveBufs<T>& s, SyncState* sync, double* partials, double tol,
                         int maxiter, hipStream_t st, SolveResult* res, int periodic, const uint32_t* cw,
                         const float* ctab, bool& ran) {
    ran = false;
    // the state arrays of the streaming form, r to q2, hold the published faces
    if (!s.r || !s.q2 || s.q2 - s.r != 5 * L.npad || s.p1 - s.p0 != L.npad) return PB_OK;
    const ResPlan p = resident_plan<T>(L, periodic, false, cw != nullptr);
    if (p.grid <= 0) return PB_OK;
    RArgs<T> a = resident_args<T>(L, s, p, sync, (unsigned long long*)partials, tol, maxiter);
    const int64_t half = (int64_t)p.grid * face_len(p.bs, p.nz, p.tx, p.ty);
    a.faces[0] = s.r;
    a.faces[1] = s.r + half;
    a.cw = cw;
    a.ctab = ctab;
    a.xs = s.p0;
    a.refuse = res ? res->refuse : nullptr;
    if (s.warm) {
        T* r0 = x_in_memory<T>(p.nz, cw != nullptr) ? s.r2 : s.q2;   // q2 holds the code words
        if (launch_resident_start<T>(L, s.op, s.b, s.x, r0, periodic, st) != PB_OK) return PB_ERR_HIP;
        a.r0 = r0;
    }
    if (launch_clear2((int*)sync, (int64_t)(sizeof(SyncState) / sizeof(int)), (int*)partials,
                      (int64_t)2 * slot_words(p.nz, p.grid, false), st) != PB_OK)
        return PB_ERR_HIP;
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
        res->coded = cw ? 1 : 0;
        res->ctab = ctab;
    }
    return PB_OK;
}

}  // namespace

template <typename T>
pb_status resident_jpcg(const Layout& L, const SolveBufs<T>& s, SyncState* sync, double* partials, double tol,
                        int maxiter, hipStream_t st, SolveResult* res, int periodic, const uint32_t* cw,
                        const float* ctab, bool& ran) {
    return resident_solve<T>(L, s, sync, partials, tol, maxiter, st, res, periodic, cw, ctab, ran);
}
template <typename T>
bool resident_fits(const Layout& L, int periodic, bool compact) {
    return resident_plan<T>(L, periodic, false, compact).grid > 0;
}

// ---- batch support (see solver.hpp)

template <typename T>
ResBatchPlan resident_batch_plan(const Layout& L) {
    ResPlan p = resident_plan<T>(L, 0, true, false);
    const bool compact = p.grid <= 0;
    if (compact) p = resident_plan<T>(L, 0, true, true);
    ResBatchPlan b{};
    b.grid = p.grid;
    b.compact = compact && p.grid > 0;
    b.groups = std::min(res_device().cus, kMaxResidentGroups);
    b.us = p.us;
    b.lds = p.lds;
    b.slot_bytes = (size_t)slot_words(p.nz, p.grid, true) * sizeof(unsigned long long);
    return b;
}
template <typename T>
size_t resident_batch_args_bytes() {
    return sizeof(RArgs<T>);
}
template <typename T>
pb_status resident_batch_fill(void* dst, const Layout& L, const SolveBufs<T>& s, SyncState* S, void* slots, double tol,
                              int maxiter, int problems, double pass_us, const float* cw, const float* ctab,
                              const int* fit) {
    ResPlan p = resident_plan<T>(L, 0, true, false);
    const bool compact = p.grid <= 0;
    if (compact) p = resident_plan<T>(L, 0, true, true);
    RArgs<T> a = resident_args<T>(L, s, p, S, (unsigned long long*)slots, tol, maxiter);
    a.faces[0] = s.r;
    const bool xmem = x_in_memory<T>(p.nz, compact);
    a.faces[1] = xmem ? s.r + (int64_t)p.grid * face_len(p.bs, p.nz, p.tx, p.ty) : s.r2;
    a.xs = s.p0;
    if (s.warm) a.r0 = xmem ? s.r2 : s.p0;
    a.first_timeout_ticks = first_wait_ticks(a.timeout_ticks, problems, pass_us, (double)a.timeout_ticks / 20e6);
    a.cw = (const uint32_t*)cw;
    a.ctab = ctab;
    a.fit = fit;
    std::memcpy(dst, &a, sizeof(a));
    return PB_OK;
}
template <typename T>
pb_status resident_batch_start(const Layout& L, const SolveBufs<T>& s, hipStream_t st) {
    ResPlan p = resident_plan<T>(L, 0, true, false);
    const bool compact = p.grid <= 0;
    if (compact) p = resident_plan<T>(L, 0, true, true);
    T* r0 = x_in_memory<T>(p.nz, compact) ? s.r2 : s.p0;
    return s.warm ? launch_resident_start<T>(L, s.op, s.b, s.x, r0, 0, st) : PB_OK;
}
template <typename T>
pb_status resident_batch_launch(const void* d_args, const int* d_off, const void* d_jobs, int grid, size_t lds,
                                bool compact, hipStream_t st, bool cooperative) {
    const RArgs<T>* ap = (const RArgs<T>*)d_args;
    const int2* jp = (const int2*)d_jobs;
    void* args[] = {&ap, &d_off, &jp};
    const void* fn = batch_kernel<T>(compact);
    const hipError_t e = cooperative ? hipLaunchCooperativeKernel(fn, dim3(grid), dim3(512), args, lds, st)
                                     : hipLaunchKernel(fn, dim3(grid), dim3(512), args, lds, st);
    if (e != hipSuccess) {
        set_error("resident batch launch failed: %s (grid %d, lds %zu)", hipGetErrorString(e), grid, lds);
        return PB_ERR_HIP;
    }
    return PB_OK;
}
#define PB_RES_INSTANCES(T)                                                                                       \
    template pb_status resident_jpcg<T>(const Layout&, const SolveBufs<T>&, SyncState*, double*, double, int,     \
                                        hipStream_t, SolveResult*, int, const uint32_t*, const float*, bool&);    \
    template bool resident_fits<T>(const Layout&, int, bool);                                                     \
    template ResBatchPlan resident_batch_plan<T>(const Layout&);                                                  \
    template size_t resident_batch_args_bytes<T>();                                                               \
    template pb_status resident_batch_fill<T>(void*, const Layout&, const SolveBufs<T>&, SyncState*, void*, double, \
                                              int, int, double, const float*, const float*, const int*);          \
    template pb_status resident_batch_start<T>(const Layout&, const SolveBufs<T>&, hipStream_t);                  \
    template pb_status resident_batch_launch<T>(const void*, const int*, const void*, int, size_t, bool, hipStream_t, \
                                                bool);

}  // namespace pb
