// The resident Jacobi-CG in FP32: kernel variants.
#include "resident_impl.hpp"

namespace pb {
namespace {
template <>
const std::vector<ResVariant>& res_variants<float>() {
    static const std::vector<ResVariant> v = {
        PB_RES_VARIANT(float, 256, 2),  PB_RES_VARIANT(float, 256, 4),  PB_RES_VARIANT(float, 512, 4),
        PB_RES_VARIANT(float, 512, 6),  PB_RES_VARIANT(float, 512, 8),  PB_RES_VARIANT(float, 512, 10),
        PB_RES_VARIANT(float, 512, 12), PB_RES_VARIANT(float, 512, 14), PB_RES_VARIANT(float, 512, 19),
        PB_RES_COMPACT(24),             PB_RES_COMPACT(32),             PB_RES_COMPACT(43),
    };
    return v;
}
}  // namespace
PB_RES_INSTANCES(float)

// A request of the solve server: as in a batch, in chunks. r is kept where a warm
// start's residual is; q, or where x by brick takes both direction arrays p, in
// the place of b, which only the first launch reads, and q then in that of x.
pb_status resident_serve_fill(void* dst, const Layout& L, const SolveBufs<float>& s, SyncState* S, void* slots,
                              double tol, int maxiter, int problems, double pass_us, const float* cw,
                              const float* ctab, int chunk, bool resume) {
    const pb_status e =
        resident_batch_fill<float>(dst, L, s, S, slots, tol, maxiter, problems, pass_us, cw, ctab, nullptr);
    RArgs<float>& a = *(RArgs<float>*)dst;
    const bool compact = resident_batch_plan<float>(L).compact;
    a.keep_r = compact ? s.r2 : s.p0;
    a.keep_q = compact ? s.x : const_cast<float*>(s.b);
    a.keep_p = compact ? const_cast<float*>(s.b) : s.p1;
    a.chunk = chunk;
    a.resume = resume ? 1 : 0;
    if (resume) {
        a.r0 = a.keep_r;
        a.warm = 1;
    }
    return e;
}
pb_status resident_serve_launch(const void* d_args, const int* d_off, const void* d_jobs, int grid, size_t lds,
                                bool compact, hipStream_t st) {
    const RArgs<float>* ap = (const RArgs<float>*)d_args;
    const int2* jp = (const int2*)d_jobs;
    void* args[] = {&ap, &d_off, &jp};
    const void* fn = compact ? (const void*)k_resident_batch<float, true, true>
                             : (const void*)k_resident_batch<float, false, true>;
    const hipError_t e = hipLaunchKernel(fn, dim3(grid), dim3(512), args, lds, st);
    if (e != hipSuccess) {
        set_error("served resident launch failed: %s (grid %d, lds %zu)", hipGetErrorString(e), grid, lds);
        return PB_ERR_HIP;
    }
    return PB_OK;
}
namespace {
__global__ void k_serve_digests(const RArgs<float>* __restrict__ probs, int n, StateDigest* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const SyncState* S = probs[i].S;
    out[i] = StateDigest{S->rr, S->bb, S->iters, S->done, S->status, 0};
}
}  // namespace
pb_status resident_serve_digests(const void* d_args, int n, StateDigest* out, hipStream_t st) {
    hipLaunchKernelGGL(k_serve_digests, dim3((n + 255) / 256), dim3(256), 0, st, (const RArgs<float>*)d_args, n, out);
    PB_HIP(hipGetLastError());
    return PB_OK;
}
}  // namespace pb
