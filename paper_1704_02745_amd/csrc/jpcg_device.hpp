// Device helpers shared by the persistent Jacobi-CG kernels: agent-scope
// loads, cross-lane sums, the Jacobi scaling and the operator at one node.
// Both kernels evaluate the operator and the scaling through these functions
// only, so their iterates differ by the order of the reductions alone.
#pragma once

#include "pb_internal.hpp"

namespace pb {
namespace {

__device__ __forceinline__ double ld_agent_d(const double* p) {
    unsigned long long v = __hip_atomic_load((const unsigned long long*)p, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
    return __longlong_as_double((long long)v);
}
__device__ __forceinline__ int ld_agent_i(const int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Workgroup barrier for the LDS hand-off between planes.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Cross-lane moves of a double through DPP (two 32-bit halves).
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
    const long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)u, CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double readlane_d(double v, int lane) {
    const long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)u, lane);
    const int hi = __builtin_amdgcn_readlane((int)(u >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
constexpr int kDppXor1 = 0xB1;         // quad permute [1,0,3,2]
constexpr int kDppXor2 = 0x4E;         // quad permute [2,3,0,1]
constexpr int kDppHalfMirror = 0x141;  // lane i of 8 reads lane 7-i
constexpr int kDppMirror = 0x140;      // lane i of 16 reads lane 15-i
constexpr int kDppRor8 = 0x128;        // lane i of 16 reads lane (i+8) mod 16

// Sum over the 64 lanes of a wave (every lane active) in a fixed order: a
// butterfly inside each 16-lane row, then (row0 + row1) + (row2 + row3).
__device__ __forceinline__ double wave_sum(double v) {
    v += dpp_d<kDppXor1>(v);
    v += dpp_d<kDppXor2>(v);
    v += dpp_d<kDppHalfMirror>(v);
    v += dpp_d<kDppMirror>(v);
    return (readlane_d(v, 0) + readlane_d(v, 16)) + (readlane_d(v, 32) + readlane_d(v, 48));
}

// Jacobi scaling 1/d: the hardware reciprocal in FP32 (about 1 ulp), an
// exact division in FP64. Every use of M^-1 in a solve goes through this one
// function, so the preconditioner is the same fixed positive diagonal in the
// direction update and in the dot products.
__device__ __forceinline__ float jacobi_inv(float d) { return __builtin_amdgcn_rcpf(d); }
__device__ __forceinline__ uint32_t bits(float f) { return __float_as_uint(f); }
__device__ __forceinline__ double jacobi_inv(double d) { return 1.0 / d; }

// (A v) at one node: d v minus the six couplings times the neighbour values,
// summed in one fixed order (x, then y, then z). Every evaluation of the
// operator in the 40-byte pass goes through this function, so a node's value
// recomputed in a tile's halo is the one its own tile computes.
// (A v)_n at one node. The rounding is fixed by explicit fused multiply-adds
// (no compiler contraction), so every kernel variant computes the same value.
template <typename T>
__device__ __forceinline__ T apply_point(T d, T v, T cr, T vr, T cl, T vl, T cu, T vu, T cd, T vd, T ca, T va, T cb,
                                         T vb) {
#pragma clang fp contract(off)
    T nb = cr * vr;
    nb = fma(cl, vl, nb);
    nb = fma(cu, vu, nb);
    nb = fma(cd, vd, nb);
    nb = fma(ca, va, nb);
    nb = fma(cb, vb, nb);
    return fma(d, v, -nb);
}

}  // namespace
}  // namespace pb
