// The resident Jacobi-CG: a persistent kernel for grids whose whole iteration
// state fits the registers and LDS of the device.
//
// Each workgroup owns a brick: a tile of columns (one per thread) times NZ
// planes. A thread keeps r, x, q = A p and the operator of its NZ nodes in
// registers; p of the brick sits in LDS with a halo of one node around the tile.
// Between iterations nothing of the state touches memory except the q of the
// nodes on the brick's faces, which the neighbours need.
//
// The iteration is that of the streaming form (one grid barrier per
// iteration, r.z and ||r||^2 of the next step from the expansion of this step's
// sums; see the comment at the head of jpcg.hip). It lets the halo travel one
// barrier behind: pass l needs p_{l-1} = r_{l-1}/d + beta p_{l-2} on the halo,
// with r_{l-1} = r_{l-2} - alpha q_{l-1}. A brick keeps r, 1/d and p of its halo
// nodes itself, so it reads only q_{l-1} there, which the owner published before
// the barrier that gave alpha and beta: the exchange needs no second barrier.
// The halo's values are computed by the owner's own operations, so they are
// bitwise the owner's.
//
// Barrier: every workgroup stores its sums into its own slot as 8-byte words
// (half of a double, barrier tag), and every workgroup polls all slots until
// the tags match, then adds them in one fixed order; with many workgroups
// (slot_groups) the first of every 16 polls these and stores their sums into a
// group slot, and all poll the group slots. A word carries its own
// tag, so there is no arrival counter, no second round trip for the data and no
// order to keep between words. The face values of q, stored before, are waited
// for (vmcnt) before the slot is written. All cross-workgroup accesses go past
// the L2 of the XCD (agent scope).
#pragma once

#include "jpcg_device.hpp"
#include "solver.hpp"

#include <vector>

namespace pb {
namespace {

template <typename T>
struct RArgs {
    Op<T> op;
    const T* b;
    const T* r0;          // initial residual: b, or b - A x0 with a warm start
    T* x;
    T* faces[2];          // published q by pass parity: per workgroup x-, x+, y-, y+, z-, z+ (face_len elements)
    int nx, ny, nz;
    int64_t sp;
    int tx, ty;           // largest tile (columns per workgroup: tx * ty <= block)
    int nxt, nyt, nzc;    // bricks per axis
    double tol;
    int maxiter;
    int warm;
    SyncState* S;
    unsigned long long* slots;   // slot_words, cleared before the launch
    long long timeout_ticks;
    long long first_timeout_ticks;   // of the first barrier (a batch's workgroups come to it from earlier problems)
    T* xs;                // forms with x in memory: x by brick (one value per thread and plane)
    // batch: the operator as code words and their dictionary, read instead of
    // its arrays when given and (fit given) *fit == 1
    const uint32_t* cw;
    const float* ctab;
    const int* fit;
    const int* refuse;    // given (a solve of its own): nothing to do when it holds a bit of kRefused
    // a solve in chunks (KEEPS): r, q and p between launches, the iterations of this
    // launch, and whether it goes on from them
    T *keep_r, *keep_q, *keep_p;
    int chunk, resume;
};

constexpr int kSlotWords = 16;            // two words per sum (low half, high half), 8 sums
// Barrier words are reached through global-memory instructions also where the
// compiler cannot see the pointer's origin (a batch's argument table).
typedef __attribute__((address_space(1))) unsigned long long GlobalWord;
constexpr int kMaxResidentGroups = 256;   // workgroups of a problem at most
constexpr int kSlotGroup = 16;            // slots that one wave polls
static_assert(kMaxResidentGroups <= kSlotGroup * kSlotGroup, "two rounds of polling");
// Group slots of a barrier over G workgroups, 0 where each polls all the slots.
// One round costs a latency less, two rounds a fraction of the traffic: with 99
// workgroups (65 x 57 x 61) 4.24 us a pass against 4.66, with 143 (81 x 77 x 85) 5.27
// against 5.04, with 200 (97^3) 6.30 against 5.51, with 210 (97 x 105 x 89 FP64) 7.61
// against 6.43, with 252 (24 planes, 141^3) 12.2 against 10.4, with 225 and 250 (32
// planes, 145^3 and 159^3) 14.1 against 13.1 and 14.3 against 12.7. Two kernels are
// slower with two rounds, those whose registers are full (256, and some spilled): 19
// planes 6.96 against 7.0 to 7.3 (129^3), 43 planes 15.1 against 15.6 (161^3). Those of
// up to 6 planes, whose plans have fewer workgroups, go without the choice (0.09 us
// a pass).
//
// The kernels over many problems always take two rounds (one for up to 16
// workgroups): polling all slots needs eight more registers, which they have only
// by spilling, and the spilled values' loads stood in the barrier's path (129^3
// 9.1 us a pass against 7.0, 97^3 7.5 against 7.0, 161^3 16.4 against 16.1; 65^3 6.6
// against 6.8).
__host__ __device__ constexpr int slot_groups(int nzb, int G, bool many) {
    if (many) return G > kSlotGroup ? (G + kSlotGroup - 1) / kSlotGroup : 0;
    return nzb > 6 && (nzb <= 14 || nzb == 24 || nzb == 32) && G > 128 ? (G + kSlotGroup - 1) / kSlotGroup : 0;
}
// Barrier words of a problem, both parities.
__host__ __device__ constexpr int slot_words(int nzb, int G, bool many) {
    return 2 * (G + slot_groups(nzb, G, many)) * kSlotWords;
}

// The value, unknown to the optimizer: keeps what is derived from it (1/d,
// offsets) from being hoisted out of the iteration into registers of its own.
__device__ __forceinline__ int opaque_v(int v) {
    asm volatile("" : "+v"(v));
    return v;
}
__device__ __forceinline__ int opaque_s(int v) {   // v uniform over the wave
    v = __builtin_amdgcn_readfirstlane(v);
    asm volatile("" : "+s"(v));
    return v;
}
__device__ __forceinline__ uint32_t opaque_v(uint32_t v) { return (uint32_t)opaque_v((int)v); }
__device__ __forceinline__ float opaque_v(float v) {
    asm volatile("" : "+v"(v));
    return v;
}
__device__ __forceinline__ double opaque_v(double v) {
    asm volatile("" : "+v"(v));
    return v;
}

constexpr int kDppRor4 = 0x124;   // lane i of 16 reads a lane 4 away (cyclic)

// Sums of eight values over each row of 16 lanes by exchange: afterwards lane
// l holds the row's sum of value l & 7. Fixed order; every lane active.
__device__ __forceinline__ double row_sum8(const double (&v)[8]) {
    const int lane = threadIdx.x & 63;
    const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4;
    double w[4], u[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const double keep = b0 ? v[2 * j + 1] : v[2 * j], send = b0 ? v[2 * j] : v[2 * j + 1];
        w[j] = keep + dpp_d<kDppXor1>(send);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const double keep = b1 ? w[2 * j + 1] : w[2 * j], send = b1 ? w[2 * j] : w[2 * j + 1];
        u[j] = keep + dpp_d<kDppXor2>(send);
    }
    const double keep = b2 ? u[1] : u[0], send = b2 ? u[0] : u[1];
    const double t = keep + dpp_d<kDppRor4>(send);
    return t + dpp_d<kDppRor8>(t);
}
// Sum of `rows` partial rows of eight values in LDS (a multiple of 8), made by
// every wave for itself: lane l returns the total of value l & 7.
__device__ __forceinline__ double lds_rows_sum8(const double* red, int rows) {
    const int lane = threadIdx.x & 63;
    double t = 0.0;
    for (int g = lane >> 3; g < rows; g += 8) t += red[g * 8 + (lane & 7)];
    t += dpp_d<kDppRor8>(t);
    t += __shfl_xor(t, 16);
    t += __shfl_xor(t, 32);
    return t;
}

using Rsrc = __amdgpu_buffer_rsrc_t;
constexpr int kRawWord3 = 0x00020000;       // raw (unformatted, unswizzled) buffer
constexpr int kAgentScope = 16;             // sc1: past the XCD's L2
constexpr uint32_t kNowhere = 0x80000000u;  // past the end of every resource: loads return 0, stores are dropped
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

template <typename T>
__device__ __forceinline__ Rsrc rsrc_of(const T* base, int64_t elems) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(base), 0, (int)(elems * (int64_t)sizeof(T)), kRawWord3);
}
template <int AUX>
__device__ __forceinline__ float bload(Rsrc r, uint32_t off, float) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, AUX));
}
template <int AUX>
__device__ __forceinline__ double bload(Rsrc r, uint32_t off, double) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, AUX));
}
__device__ __forceinline__ uint32_t word_load(Rsrc r, uint32_t off) {
    return __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0);
}
__device__ __forceinline__ void agent_store(Rsrc r, uint32_t off, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, (int)off, 0, kAgentScope);
}
// x by brick: one address register per thread, the plane in the scalar offset.
__device__ __forceinline__ float x_get(Rsrc r, uint32_t off, int plane, float) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, plane, 0));
}
__device__ __forceinline__ void x_put(Rsrc r, uint32_t off, int plane, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, (int)off, plane, 0);
}
__device__ __forceinline__ double x_get(Rsrc r, uint32_t off, int plane, double) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, plane, 0));
}
__device__ __forceinline__ void x_put(Rsrc r, uint32_t off, int plane, double v) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, (int)off, plane, 0);
}
__device__ __forceinline__ void agent_store(Rsrc r, uint32_t off, double v) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, (int)off, 0, kAgentScope);
}

// Published face values of one workgroup, in elements: two x-faces of ty * NZ,
// two y-faces of tx * NZ, two z-faces of one value per thread.
__host__ __device__ constexpr int face_len(int bs, int nzb, int tx, int ty) { return 2 * (tx + ty) * nzb + 2 * bs; }

// Whether the couplings to the lower x and y neighbours sit in LDS (each thread
// its own) instead of registers: from 15 planes of FP32 or 7 of FP64 on, where the
// rest of the state fills the 256 registers of a thread and they would spill (129^3,
// 19 planes: 13.1 us per iteration with the spills, 7.5 without). Beside the line it
// matters little: 8 planes of FP64 (97 x 105 x 89) 6.50 us in LDS and 6.52 in registers,
// 9 (101 x 99 x 97) 6.94 and 6.86, 14 of FP32 (113 x 111 x 112, 117 x 117 x 113) 6.22 and
// 6.45 in LDS and 6.27 and 6.79 in registers.
template <typename T>
__host__ __device__ constexpr bool lower_in_lds(int bs, int nzb) { return nzb > (sizeof(T) == 4 ? 14 : 6); }
// Whether x goes to memory by brick instead of registers (each thread reads and
// writes its own values once per pass; they stay in the XCD's L2): the compact
// form, and FP64 from 7 planes on (97 x 105 x 89, 8 planes: 14.0 us per
// iteration with x in registers and 36 of them spilled).
template <typename T>
__host__ __device__ constexpr bool x_in_memory(int nzb, bool compact) {
    return compact || (sizeof(T) == 8 && nzb > 6);
}
// LDS of one workgroup, in bytes: the reduction scratch, p by columns (the NZ
// values of a column together, at an odd stride, so that a lane's accesses
// are one address plus constants and the lanes fall into different banks) over
// the tile and its halo, and r and 1/d of the halo.
template <typename T>
__host__ __device__ constexpr size_t resident_lds_bytes(int bs, int nzb, int tx, int ty, bool compact) {
    return (!compact && lower_in_lds<T>(bs, nzb) ? sizeof(T) * 2 * (size_t)bs * nzb : 0) +
           sizeof(double) * (size_t)(bs / 64) * 4 * 8 * 2 + 256 +
           sizeof(T) * ((size_t)(nzb | 1) * (tx + 2) * (ty + 2) + (size_t)nzb * 4 * (tx + ty));
}

// The whole solve of one problem by workgroup `w` of its nxt * nyt * nzc.
//
// CP, the compact form (FP32, operator given as code words): for bricks whose
// state does not fit the registers. A node keeps r, q and six bytes of codes
// there, decoded through the dictionary in LDS where they are used; x goes to
// memory (x_in_memory). The operations and their order are the same.
//
// KEEPS: the launch ends after a.chunk iterations of an unfinished solve, with r,
// q, p, x and the scalars in memory as the next pass expects them, and the next
// launch goes on with that pass, so the iterates are those of one launch, bit for
// bit. The last pass stores them before its barrier, from inside the loop: with
// r and q alive past it the compiler spilled 74 (compact: 170) registers.
// MANY: in a launch over many problems. A: RArgs<T>, as a kernel argument or in
// constant memory.
template <typename T, int BS, int NZ, bool PER, bool CP, bool MANY, bool KEEPS, typename A>
__device__ void resident_problem(const A& a, int w, unsigned char* lds_raw) {
#pragma clang fp contract(off)
    constexpr int ROWS = BS / 64 * 4;
    constexpr int E = (int)sizeof(T);
    // 1/d kept beside d where the registers allow
    static_assert(!CP || E == 4, "code words are FP32");
    constexpr bool LL = !CP && lower_in_lds<T>(BS, NZ);
    constexpr bool XM = x_in_memory<T>(NZ, CP);
    constexpr bool KEEP = E == 8 || NZ <= (LL ? 17 : 12);
    constexpr int SZ = NZ | 1;   // LDS stride of a column
    if (!MANY && a.refuse && (*a.refuse & kRefused)) return;
    const int G = a.nxt * a.nyt * a.nzc;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int64_t sp = a.sp;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // the brick: columns [x0, x1) x [y0, y1), planes [k0, k0 + nk)
    const int bx = w % a.nxt, by = w / a.nxt % a.nyt, bz = w / (a.nxt * a.nyt);
    const int x0 = (int)((int64_t)bx * nx / a.nxt), x1 = (int)((int64_t)(bx + 1) * nx / a.nxt);
    const int y0 = (int)((int64_t)by * ny / a.nyt), y1 = (int)((int64_t)(by + 1) * ny / a.nyt);
    const int k0 = bz * NZ, nk = min(NZ, nz - k0);
    const int wx = x1 - x0, wy = y1 - y0, row = a.tx + 2;
    const int cxx = tid % a.tx, cyy = tid / a.tx;
    const bool valid = cxx < wx && cyy < wy;
    const int i = x0 + cxx, j = y0 + cyy, pos = j * nx + i;

    double* red = reinterpret_cast<double*>(lds_raw);
    double* red2 = red + ROWS * 8;
    int* s_flag = reinterpret_cast<int*>(red2 + ROWS * 8);
    T* const P = reinterpret_cast<T*>(lds_raw + sizeof(double) * ROWS * 16 + 256);
    T* const RH = P + (size_t)SZ * row * (a.ty + 2);
    T* const IH = RH + (size_t)NZ * 2 * (a.tx + a.ty);
    T* const CL = IH + (size_t)NZ * 2 * (a.tx + a.ty) + tid;   // LL: x and y of plane kk at 2kk, 2kk+1
    // CP: dictionary and 1/dictionary, at an address known to the compiler (a
    // lookup is one shift of a code byte and one LDS read)
    T *tv = nullptr, *ti = nullptr;
    if constexpr (CP) {
        __shared__ T s_dict[2 * kCodedTableSize];
        tv = s_dict;
        ti = s_dict + kCodedTableSize;
        if (a.fit && *a.fit != 1) return;   // the operator does not fit the dictionary: the streaming form solves it
        for (int n = tid; n < kCodedTableSize; n += BS) {
            const T c = (T)a.ctab[n];
            tv[n] = c;
            ti[n] = c == T(0) ? T(0) : jacobi_inv(c);   // 0 is read for the diagonal where there is no node
        }
        __syncthreads();
    }

    // p of this thread's column and of the four around it. With one brick
    // along a periodic axis the neighbour across the end is in the tile itself.
    // Threads without a column share the halo's corner, which stays zero.
    const bool wrap_x = PER && a.nxt == 1, wrap_y = PER && a.nyt == 1;
    T* const pl = P + SZ * (valid ? (cyy + 1) * row + cxx + 1 : 0);
    const T* const pR = !valid ? pl : wrap_x && i == nx - 1 ? pl - SZ * (nx - 1) : pl + SZ;
    const T* const pL = !valid ? pl : wrap_x && i == 0 ? pl + SZ * (nx - 1) : pl - SZ;
    const T* const pU = !valid ? pl : wrap_y && j == ny - 1 ? pl - SZ * row * (ny - 1) : pl + SZ * row;
    const T* const pD = !valid ? pl : wrap_y && j == 0 ? pl + SZ * row * (ny - 1) : pl - SZ * row;

    const bool coded = CP || (E == 4 && a.cw && (!a.fit || *a.fit == 1));
    auto decode = [&](uint32_t c, int byte) -> T { return (T)a.ctab[(c >> (8 * byte)) & 255u]; };
    auto diag_at = [&](int64_t g) -> T { return coded ? decode(a.cw[g], 3) : a.op.d[g]; };
    // ---- the operator and the state of the own nodes
    constexpr int NR = CP ? 1 : NZ;   // held in registers by the full form alone
    T r[NZ], q[NZ];
    T x[XM ? 1 : NZ], cx[NR], cy[NR], cz[NR], d[NR], iv[KEEP && !CP ? NZ : 1], cxm[LL ? 1 : NR], cym[LL ? 1 : NR];
    uint32_t w1[CP ? NZ : 1], w2[CP ? (NZ + 1) / 2 : 1];   // codes: x+, x-, y+, y-; z+, d of two planes
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    // XM: x of plane kk at xoff + kk * BS elements
    const Rsrc xs = rsrc_of(XM ? a.xs + (size_t)w * NZ * BS : a.x, XM ? NZ * BS : 0);
    const uint32_t xoff = (uint32_t)tid * E;
    const bool resume = KEEPS && a.resume;
    {
        // positions without a node and planes past nk read as zero
        auto from = [&](const void* p) { return rsrc_of((const T*)p + (int64_t)k0 * sp, (int64_t)nk * sp); };
        const Rsrc rcx = from(a.op.cx), rcy = from(a.op.cy), rcz = from(a.op.cz), rd = from(a.op.d), rr0 = from(a.r0),
                   rb0 = from(a.b), rx = from(a.x), rcw = from(a.cw), rkq = from(KEEPS ? a.keep_q : a.x);
        const bool keeps_x = resume;   // by brick, from the launch before
        auto at = [&](bool in, int p) { return valid && in ? (uint32_t)p * E : kNowhere; };
        uint32_t o = at(true, pos), ox = at(i > 0 || PER, i > 0 ? pos - 1 : pos + nx - 1),
                 oy = at(j > 0 || PER, j > 0 ? pos - nx : pos + (ny - 1) * nx);
        const uint32_t plane_bytes = (uint32_t)(sp * E);
#pragma unroll
        for (int kk = 0; kk < NZ; ++kk) {
            if constexpr (CP) {   // words at kNowhere read as 0, the code of 0
                const uint32_t c = word_load(rcw, o), cl = word_load(rcw, ox), cd = word_load(rcw, oy);
                w1[kk] = (c & 0xffu) | (cl & 0xffu) << 8 | (c & 0xff00u) << 8 | (cd & 0xff00u) << 16;
                if (kk % 2 == 0) w2[kk / 2] = c >> 16;
                else w2[kk / 2] |= c & 0xffff0000u;
            } else {
                T cxl, cyl;
                if (coded) {
                    const uint32_t c = word_load(rcw, o);
                    cx[kk] = decode(c, 0);
                    cy[kk] = decode(c, 1);
                    cz[kk] = decode(c, 2);
                    d[kk] = decode(c, 3);
                    cxl = decode(word_load(rcw, ox), 0);
                    cyl = decode(word_load(rcw, oy), 1);
                } else {
                    cx[kk] = bload<0>(rcx, o, T());
                    cy[kk] = bload<0>(rcy, o, T());
                    cz[kk] = bload<0>(rcz, o, T());
                    d[kk] = bload<0>(rd, o, T());
                    cxl = bload<0>(rcx, ox, T());
                    cyl = bload<0>(rcy, oy, T());
                }
                if constexpr (LL) {
                    CL[2 * kk * BS] = cxl;
                    CL[(2 * kk + 1) * BS] = cyl;
                } else {
                    cxm[kk] = cxl;
                    cym[kk] = cyl;
                }
                if (d[kk] == T(0)) d[kk] = T(1);
                if constexpr (KEEP) iv[kk] = jacobi_inv(d[kk]);
            }
            const T xv = bload<0>(rx, a.warm ? o : kNowhere, T());
            if constexpr (XM) x_put(xs, keeps_x ? kNowhere : xoff, kk * BS * E, xv);
            else x[kk] = xv;
            r[kk] = bload<0>(rr0, o, T());
            q[kk] = KEEPS ? bload<0>(rkq, resume ? o : kNowhere, T()) : T(0);
            const T bv = bload<0>(rb0, o, T());
            acc[0] = fma((double)r[kk], (double)r[kk], acc[0]);
            acc[1] = fma((double)bv, (double)bv, acc[1]);
            o += plane_bytes;
            ox += plane_bytes;
            oy += plane_bytes;
            if (kk % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
    }
    auto inv = [&](int kk) -> T {
        if constexpr (CP) return ti[(w2[kk / 2] >> (kk % 2 ? 24 : 8)) & 255u];
        else if constexpr (KEEP) return iv[kk];
        else return jacobi_inv(opaque_v(d[kk]));
    };
    // planes below and above the brick, in this thread's column
    const bool has_b = PER || bz > 0, has_t = PER || bz + 1 < a.nzc;
    const int kb = k0 > 0 ? k0 - 1 : nz - 1, kt = k0 + nk < nz ? k0 + nk : 0;
    T czb = T(0), rb = T(0), ib = T(0), pb_ = T(0), rt = T(0), it_ = T(0), pt = T(0);
    if (valid && has_b) {
        const int64_t g = (int64_t)kb * sp + pos;
        czb = coded ? decode(a.cw[g], 2) : a.op.cz[g];
        rb = a.r0[g];
        ib = jacobi_inv(diag_at(g));
    }
    if (valid && has_t) {
        const int64_t g = (int64_t)kt * sp + pos;
        rt = a.r0[g];
        it_ = jacobi_inv(diag_at(g));
    }
    // ---- where the faces of this brick are published and the halo's are read
    // (byte offsets); kNowhere where no neighbour reads or is
    const int FX = a.ty * NZ, FY = a.tx * NZ;
    const uint32_t face_bytes = (uint32_t)face_len(BS, NZ, a.tx, a.ty) * E;
    auto brick = [&](int ux, int uy, int uz) -> uint32_t {   // wrapped coordinates
        ux = ux < 0 ? ux + a.nxt : (ux >= a.nxt ? ux - a.nxt : ux);
        uy = uy < 0 ? uy + a.nyt : (uy >= a.nyt ? uy - a.nyt : uy);
        uz = uz < 0 ? uz + a.nzc : (uz >= a.nzc ? uz - a.nzc : uz);
        return (uint32_t)((uz * a.nyt + uy) * a.nxt + ux) * face_bytes;
    };
    const uint32_t mine = (uint32_t)w * face_bytes;
    const bool face_x = a.nxt > 1, face_y = a.nyt > 1;
    const uint32_t pub_x = !valid || !face_x ? kNowhere
                           : cxx == 0        ? mine + (uint32_t)cyy * E
                           : cxx == wx - 1   ? mine + (uint32_t)(FX + cyy) * E
                                             : kNowhere;
    const uint32_t pub_y = !valid || !face_y ? kNowhere
                           : cyy == 0        ? mine + (uint32_t)(2 * FX + cxx) * E
                           : cyy == wy - 1   ? mine + (uint32_t)(2 * FX + FY + cxx) * E
                                             : kNowhere;
    const uint32_t zlo = (uint32_t)(2 * FX + 2 * FY + tid) * E, zhi = zlo + (uint32_t)BS * E;
    const bool face_z = PER || a.nzc > 1;
    const uint32_t pub_zlo = valid && face_z ? mine + zlo : kNowhere, pub_zhi = valid && face_z ? mine + zhi : kNowhere;
    const uint32_t off_b = valid && has_b ? brick(bx, by, bz - 1) + zhi : kNowhere;
    const uint32_t off_t = valid && has_t ? brick(bx, by, bz + 1) + zlo : kNowhere;
    const int64_t face_elems = (int64_t)G * face_len(BS, NZ, a.tx, a.ty);
    // in-plane halo: column c of hc (x-, x+, y-, y+ neighbours) is kept by the
    // threads c + hc * m, planes m, m + hgroups, ... each
    const int hxc = face_x ? 2 * a.ty : 0, hc = hxc + (face_y ? 2 * a.tx : 0);
    const int hgroups = hc > 0 ? BS / hc : 0;   // at least 1 (host)
    const int hk0 = hc > 0 ? tid / hc : 0, hcol = tid - hk0 * hc;
    bool hon = hc > 0 && hk0 < hgroups;
    uint32_t hfrom = kNowhere;   // byte offset of plane 0's value in the faces
    int hpos = 0;                // plane position of the column's nodes
    T* hP = P;
    if (hon) {
        const bool alongx = hcol < hxc;
        const int side = alongx ? a.ty : a.tx, g = alongx ? hcol : hcol - hxc, hi = g >= side ? 1 : 0, c = g - hi * side;
        int hi_i, hi_j, col;
        if (alongx) {
            hon = c < wy && (PER || (hi ? x1 < nx : x0 > 0));
            hi_i = hi ? (x1 < nx ? x1 : 0) : (x0 > 0 ? x0 - 1 : nx - 1);
            hi_j = y0 + c;
            col = (c + 1) * row + (hi ? wx + 1 : 0);
            hfrom = brick(bx + (hi ? 1 : -1), by, bz) + (uint32_t)((hi ? 0 : FX) + c) * E;
        } else {
            hon = c < wx && (PER || (hi ? y1 < ny : y0 > 0));
            hi_j = hi ? (y1 < ny ? y1 : 0) : (y0 > 0 ? y0 - 1 : ny - 1);
            hi_i = x0 + c;
            col = (hi ? wy + 1 : 0) * row + c + 1;
            hfrom = brick(bx, by + (hi ? 1 : -1), bz) + (uint32_t)(2 * FX + (hi ? 0 : FY) + c) * E;
        }
        hpos = hi_j * nx + hi_i;
        hP = P + SZ * col;
    }
    const uint32_t hstride = (uint32_t)((hcol < hxc ? a.ty : a.tx) * E);   // bytes from plane to plane
    for (int h = tid; h < SZ * row * (a.ty + 2); h += BS) P[h] = T(0);
    if (hon)
        for (int kk = hk0; kk < nk; kk += hgroups) {
            const int64_t g = (int64_t)(k0 + kk) * sp + hpos;
            RH[kk * hc + hcol] = a.r0[g];
            IH[kk * hc + hcol] = jacobi_inv(diag_at(g));
        }
    if constexpr (KEEPS) {
        if (resume) {
            __syncthreads();   // p is cleared
            const T* const kp = a.keep_p;
            if (valid)
                for (int kk = 0; kk < nk; ++kk) pl[kk] = kp[(int64_t)(k0 + kk) * sp + pos];
            if (hon)
                for (int kk = hk0; kk < nk; kk += hgroups) hP[kk] = kp[(int64_t)(k0 + kk) * sp + hpos];
            if (valid && has_b) pb_ = kp[(int64_t)kb * sp + pos];
            if (valid && has_t) pt = kp[(int64_t)kt * sp + pos];
        }
    }

    // ---- grid barrier with the reduction of the sums in acc; the totals in
    // every thread
    int b = 0;
    auto reduce = [&](double (&out)[8]) -> bool {
        const double t = row_sum8(acc);
        if ((lane & 15) < 8) red[(wave * 4 + (lane >> 4)) * 8 + (lane & 7)] = t;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's face values have arrived
        __syncthreads();
        const unsigned tag = (unsigned)(b + 1);
        GlobalWord* slots = (GlobalWord*)(uintptr_t)a.slots + (size_t)(b & 1) * (G + slot_groups(NZ, G, MANY)) * kSlotWords;
        auto put = [&](int slot, double v) {   // lane n's sum n
            if (lane < 8) {
                const unsigned long long u = (unsigned long long)__double_as_longlong(v);
                GlobalWord* m = slots + (size_t)slot * kSlotWords + 2 * lane;
                __hip_atomic_store(m, (u << 32) | tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(m + 1, (u & 0xffffffff00000000ull) | tag, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
        };
        double tot;
        if (MANY || slot_groups(NZ, G, MANY) > 0) {
            if (wave == 0) {
                // the sums of up to kSlotGroup slots: lane n polls sum n & 7 of slots n / 8 and
                // n / 8 + 8, and gets the total of that sum
                auto get = [&](int first, int count) -> double {
                    const int s0 = opaque_v(lane >> 3);
                    const bool on0 = s0 < count, on1 = s0 + 8 < count;
                    const GlobalWord* p0 = slots + (size_t)(first + (on0 ? s0 : 0)) * kSlotWords + 2 * (lane & 7);
                    const GlobalWord* p1 = slots + (size_t)(first + (on1 ? s0 + 8 : 0)) * kSlotWords + 2 * (lane & 7);
                    unsigned long long l0, h0, l1, h1;
                    long long t0 = 0;
                    while (true) {
                        l0 = __hip_atomic_load(p0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        h0 = __hip_atomic_load(p0 + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        l1 = __hip_atomic_load(p1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        h1 = __hip_atomic_load(p1 + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        if ((((unsigned)l0 ^ tag) | ((unsigned)h0 ^ tag) | ((unsigned)l1 ^ tag) | ((unsigned)h1 ^ tag)) == 0)
                            break;
                        const long long now = wall_clock64();
                        if (t0 == 0) t0 = now;
                        if (now - t0 > (b == 0 ? a.first_timeout_ticks : a.timeout_ticks)) {
                            s_flag[0] = 1;
                            break;
                        }
                    }
                    const double v0 = __longlong_as_double((long long)((h0 & 0xffffffff00000000ull) | (l0 >> 32)));
                    const double v1 = __longlong_as_double((long long)((h1 & 0xffffffff00000000ull) | (l1 >> 32)));
                    double t = on0 ? v0 : 0.0;
                    t += on1 ? v1 : 0.0;
                    t += dpp_d<kDppRor8>(t);
                    t += __shfl_xor(t, 16);
                    t += __shfl_xor(t, 32);
                    return t;
                };
                put(w, lds_rows_sum8(red, ROWS));
                const int ng = slot_groups(NZ, G, MANY);
                if (ng > 0 && w % kSlotGroup == 0) put(G + w / kSlotGroup, get(w, min(kSlotGroup, G - w)));
                const double t = ng > 0 ? get(G, ng) : get(0, G);
                if (lane < 8) red2[lane] = t;
            }
            __syncthreads();
            tot = red2[lane & 7];
        } else {
            if (wave == 0) put(w, lds_rows_sum8(red, ROWS));
            // thread n polls the sum n & 7 of slots n/8, n/8 + BS/8, ...
            constexpr int M = (kMaxResidentGroups * 8 + BS - 1) / BS;
            double part = 0.0;
            if (opaque_v(tid >> 3) < G) {
                unsigned long long lo[M], hi[M];
                long long t0 = 0;
                while (true) {
                    unsigned bad = 0;
#pragma unroll
                    for (int m = 0; m < M; ++m) {
                        if (m > 0 && m * (BS / 8) >= G) break;   // uniform
                        const int slot = min((tid >> 3) + m * (BS / 8), G - 1);
                        const GlobalWord* p = slots + (size_t)slot * kSlotWords + 2 * (tid & 7);
                        lo[m] = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        hi[m] = __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
#pragma unroll
                    for (int m = 0; m < M; ++m) {
                        if (m > 0 && m * (BS / 8) >= G) break;
                        bad |= ((unsigned)lo[m] ^ tag) | ((unsigned)hi[m] ^ tag);
                    }
                    if (bad == 0) break;
                    const long long now = wall_clock64();
                    if (t0 == 0) t0 = now;
                    if (now - t0 > (b == 0 ? a.first_timeout_ticks : a.timeout_ticks)) {
                        s_flag[0] = 1;
                        break;
                    }
                }
#pragma unroll
                for (int m = 0; m < M; ++m)
                    if ((tid >> 3) + m * (BS / 8) < G)
                        part += __longlong_as_double((long long)((hi[m] & 0xffffffff00000000ull) | (lo[m] >> 32)));
            }
            asm volatile("" ::: "memory");
            part += dpp_d<kDppRor8>(part);
            if ((lane & 15) < 8) red2[(wave * 4 + (lane >> 4)) * 8 + (lane & 7)] = part;
            __syncthreads();
            tot = lds_rows_sum8(red2, ROWS);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) out[k] = readlane_d(tot, k);
        ++b;
        return s_flag[0] == 0;
    };
    auto timed_out = [&] {
        if (tid == 0) __hip_atomic_store(&a.S->status, (int)PB_ERR_TIMEOUT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (KEEPS && tid == 0) __hip_atomic_store(&a.S->done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };

    if (tid == 0) s_flag[0] = 0;
    __syncthreads();
    double v[8];
    double alpha = 0.0, beta = 0.0, rr, bb;
    int done = 0, status = PB_OK, zero = 0, iters = 0;
    if (!reduce(v)) return timed_out();   // also: every halo is read before any state is stored
    if (resume) {
        rr = a.S->rr;
        bb = a.S->bb;
        alpha = a.S->alpha;
        beta = a.S->beta;
        iters = a.S->iters;
    } else {
        rr = v[0];
        bb = v[1];
    }
    const double sqrt_bb = sqrt(bb);
    const int stop_at = KEEPS ? iters + a.chunk : 0;
    if (resume) {
    } else if (!(bb - bb == 0.0) || !(rr - rr == 0.0)) { done = 1; status = PB_ERR_NONFINITE; }
    else if (bb == 0.0) { done = 1; zero = 1; }
    else if (sqrt(rr) / sqrt_bb < a.tol) { done = 1; }
    else if (a.maxiter <= 0) { done = 1; status = PB_NOT_CONVERGED; }

    T last = T(0);   // XM: step of the last x update
    for (int pass = KEEPS ? iters : 0; !done && !(KEEPS && iters >= stop_at); ++pass) {
        const T al = (T)alpha, be = (T)beta;
        // ---- q of the halo, on its way while the own nodes are updated (the
        // first pass has alpha = 0 and reads nothing)
        const uint32_t none = pass > 0 ? 0u : kNowhere;
        const Rsrc qo = rsrc_of((pass & 1) ? a.faces[0] : a.faces[1], face_elems);
        const T qb = bload<kAgentScope>(qo, off_b | none, T());
        const T qt = bload<kAgentScope>(qo, off_t | none, T());
        constexpr int U = E == 4 ? 4 : 2;   // halo nodes in flight per thread
        T qh[U];
        const uint32_t hbytes = (uint32_t)hgroups * hstride;
        uint32_t hoff = hon ? (hfrom + (uint32_t)hk0 * hstride) | none : kNowhere;
        int hk = hon ? hk0 : nk;
        auto fetch = [&] {
#pragma unroll
            for (int u = 0; u < U; ++u) qh[u] = bload<kAgentScope>(qo, hoff + (uint32_t)u * hbytes, T());
            hoff += U * hbytes;
        };
        fetch();
        // ---- r, p, x of the own nodes
        if constexpr (XM) {
            constexpr int C = 32 / E;   // x values in flight
            T xv[C];
#pragma unroll
            for (int u = 0; u < C && u < NZ; ++u) xv[u] = x_get(xs, xoff, u * BS * E, T());
#pragma unroll
            for (int k8 = 0; k8 < NZ; k8 += C) {
                T xn[C];
#pragma unroll
                for (int u = 0; u < C; ++u)
                    if (k8 + C + u < NZ) xn[u] = x_get(xs, xoff, (k8 + C + u) * BS * E, T());
#pragma unroll
                for (int u = 0; u < C; ++u) {
                    const int kk = k8 + u < NZ ? k8 + u : 0;
                    if (k8 + u >= NZ) continue;
                    const T po = pl[kk];
                    r[kk] = fma(-al, q[kk], r[kk]);
                    if constexpr (CP)
                        if (kk % 2 == 0) asm volatile("" : "+v"(w2[kk / 2]));
                    x_put(xs, xoff, kk * BS * E, fma(al, po, xv[u]));
                    pl[kk] = fma(be, po, r[kk] * inv(kk));
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < C; ++u) xv[u] = xn[u];
            }
        } else {
#pragma unroll
            for (int kk = 0; kk < NZ; ++kk) {
                const T po = pl[kk];
                r[kk] = fma(-al, q[kk], r[kk]);
                x[kk] = fma(al, po, x[kk]);
                pl[kk] = fma(be, po, r[kk] * inv(kk));
            }
        }
        // ---- r and p of the halo
        while (hk < nk) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (hk < nk) {
                    const int h = hk * hc + hcol;
                    const T rh = fma(-al, qh[u], RH[h]);
                    RH[h] = rh;
                    hP[hk] = fma(be, hP[hk], rh * IH[h]);
                }
                hk += hgroups;
            }
            if (hk < nk) fetch();
        }
        rb = fma(-al, qb, rb);
        pb_ = fma(be, pb_, rb * ib);
        rt = fma(-al, qt, rt);
        pt = fma(be, pt, rt * it_);
        __syncthreads();
        // ---- q = A p and the sums
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[k] = 0.0;
        const Rsrc qn = rsrc_of((pass & 1) ? a.faces[1] : a.faces[0], face_elems);
        T pm = pb_, pc = pl[0], cbelow = T(0);
        uint32_t ox = opaque_v(pub_x), oy = opaque_v(pub_y);
        const int nkv = opaque_s(nk);   // compared in place, not kept as NZ masks
        // the operator and the neighbours' p of a plane, read from LDS one plane
        // ahead of their use; the forms that fill the registers hold the scheduler
        // to that with a barrier after each plane (it would pull the reads of many
        // planes ahead and spill), the others leave it free: with two waves per
        // SIMD they need the planes' chains interleaved
        struct Ops {
            T right, left, up, down, above, cr, cl, cu, cd, ca, d, iv;
        };
        auto ops_of = [&](int kk) -> Ops {
            Ops o;
            o.right = pR[kk];
            o.left = pL[kk];
            o.up = pU[kk];
            o.down = pD[kk];
            o.above = kk + 1 < NZ ? pl[kk + 1 < NZ ? kk + 1 : 0] : T(0);
            if constexpr (CP) {
                // (in place: no copy, and no address kept across iterations)
                asm volatile("" : "+v"(w1[kk]), "+v"(w2[kk / 2]));
                const uint32_t c1 = w1[kk], c2 = w2[kk / 2];
                o.cr = tv[c1 & 255u];
                o.cl = tv[c1 >> 8 & 255u];
                o.cu = tv[c1 >> 16 & 255u];
                o.cd = tv[c1 >> 24];
                o.ca = tv[(kk % 2 ? c2 >> 16 : c2) & 255u];
                o.d = tv[(kk % 2 ? c2 >> 24 : c2 >> 8) & 255u];
                o.iv = ti[(kk % 2 ? c2 >> 24 : c2 >> 8) & 255u];
            } else {
                o.cr = cx[kk];
                o.cl = LL ? CL[2 * kk * BS] : cxm[LL ? 0 : kk];
                o.cu = cy[kk];
                o.cd = LL ? CL[(2 * kk + 1) * BS] : cym[LL ? 0 : kk];
                o.ca = cz[kk];
                o.d = d[kk];
                o.iv = E == 8 ? opaque_v(inv(kk)) : inv(kk);   // FP64: r/d is formed again, not kept
            }
            return o;
        };
        Ops cur = ops_of(0);
#pragma unroll
        for (int kk = 0; kk < NZ; ++kk) {
            Ops nxt;
            if (kk + 1 < NZ) nxt = ops_of(kk + 1 < NZ ? kk + 1 : kk);
            const T pu = kk + 1 == NZ || kk + 1 == nkv ? pt : cur.above;
            T cb = kk == 0 ? czb : cbelow;
            if (PER && kk > 0) cb = kk < nkv ? cb : T(0);
            cbelow = cur.ca;
            const T qq = apply_point(cur.d, pc, cur.cr, cur.right, cur.cl, cur.left, cur.cu, cur.up, cur.cd, cur.down,
                                     cur.ca, pu, cb, pm);
            q[kk] = qq;
            agent_store(qn, ox, qq);   // dropped at kNowhere
            agent_store(qn, oy, qq);
            if (kk == 0) agent_store(qn, pub_zlo, qq);
            if (kk + 1 == nkv) agent_store(qn, pub_zhi, qq);
            ox += (uint32_t)(a.ty * E);
            oy += (uint32_t)(a.tx * E);
            const T ivk = cur.iv;
            const double pd = (double)pc, qd = (double)qq, rd = (double)r[kk];
            const double zd = (double)(r[kk] * ivk), wd = (double)(qq * ivk);
            acc[0] = fma(pd, qd, acc[0]);
            acc[1] = fma(rd, zd, acc[1]);
            acc[2] = fma(rd, wd, acc[2]);
            acc[3] = fma(qd, wd, acc[3]);
            acc[4] = fma(rd, rd, acc[4]);
            acc[5] = fma(rd, qd, acc[5]);
            acc[6] = fma(qd, qd, acc[6]);
            if constexpr (CP || (LL && E == 4)) {
                // the sums are otherwise sunk below the loop, with p and 1/d of
                // every plane kept until then
#pragma unroll
                for (int k = 0; k < 7; ++k) asm volatile("" : "+v"(acc[k]));
                __builtin_amdgcn_sched_barrier(0);
            }
            pm = pc;
            pc = cur.above;
            cur = nxt;
        }
        if constexpr (KEEPS) {
            if (iters + 1 >= stop_at) {   // the launch's last pass
                const Rsrc kr = rsrc_of(a.keep_r + (int64_t)k0 * sp, (int64_t)nk * sp),
                           kq = rsrc_of(a.keep_q + (int64_t)k0 * sp, (int64_t)nk * sp),
                           kp = rsrc_of(a.keep_p + (int64_t)k0 * sp, (int64_t)nk * sp);
                uint32_t o = opaque_v(valid ? (uint32_t)pos * E : kNowhere);
#pragma unroll
                for (int kk = 0; kk < NZ; ++kk) {
                    x_put(kr, o, 0, r[kk]);
                    x_put(kq, o, 0, q[kk]);
                    x_put(kp, o, 0, pl[kk]);
                    o += (uint32_t)(sp * E);
                }
            }
        }
        if (!reduce(v)) return timed_out();
        const double pq = v[0], rrd = v[1], rqd = v[2], qqd = v[3];
        if (!(pq > 0.0) || !(pq - pq == 0.0) || !(rrd > 0.0)) {
            done = 1;
            status = PB_ERR_BREAKDOWN;   // x holds the last good iterate
        } else {
            const double alp = rrd / pq;
            const double rho = fmax(rrd - 2.0 * alp * rqd + alp * alp * qqd, 0.0);
            rr = fmax(v[4] - 2.0 * alp * v[5] + alp * alp * v[6], 0.0);
            ++iters;
            alpha = alp;
            beta = rho / rrd;
            const double rel = sqrt(rr) / sqrt_bb;
            if (!(rel - rel == 0.0)) { done = 1; status = PB_ERR_BREAKDOWN; }
            else if (rel < a.tol) { done = 1; }
            else if (iters >= a.maxiter) { done = 1; status = PB_NOT_CONVERGED; }
            if (done && status != PB_ERR_BREAKDOWN) {
                // last x update with the final alpha and direction
                if constexpr (!XM)
#pragma unroll
                    for (int kk = 0; kk < NZ; ++kk) x[kk] = fma((T)alpha, pl[kk], x[kk]);
                last = (T)alpha;
            }
        }
    }
    if (valid && !(KEEPS && XM && !done))   // (x by brick stays there)
#pragma unroll
        for (int kk = 0; kk < NZ; ++kk)
            if (kk < nk) {
                T xk;
                if constexpr (XM) xk = fma(last, pl[kk], x_get(xs, xoff, kk * BS * E, T()));
                else xk = x[kk];
                a.x[(int64_t)(k0 + kk) * sp + pos] = zero ? T(0) : xk;
            }
    if (w == 0 && tid == 0) {
        a.S->rr = rr;
        a.S->bb = bb;
        a.S->alpha = alpha;
        a.S->beta = beta;
        a.S->iters = iters;
        a.S->done = done;
        a.S->status = status;
        a.S->zero_rhs = zero;
    }
}

template <typename T, int BS, int NZ, bool PER, bool CP = false>
__global__ __launch_bounds__(BS) void k_jpcg_resident(RArgs<T> a) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    resident_problem<T, BS, NZ, PER, CP, false, false>(a, blockIdx.x, lds_raw);
}

constexpr int kCompactFrom = 24;   // planes per brick from which a kernel is the compact form's
// Planes per brick of a batch: the largest that leave the registers unspilled,
// so that a problem takes few workgroups and the barrier's latency is shared by
// many nodes. One number per form: a kernel that chose between four inlined
// forms spilled, and gave wrong potentials in the last bricks of one of them (the
// cause is not known; nothing here was found to depend on the number of forms, and
// partial last bricks are held to the streaming form's potentials by tests).
template <typename T>
constexpr int batch_planes(bool compact) { return sizeof(T) == 8 ? 8 : (compact ? 43 : 19); }

template <typename T>
using ConstArgs = __attribute__((address_space(4))) RArgs<T>;

// Many problems in one launch: workgroup g runs the jobs [off[g], off[g + 1]) of
// its list one after the other, job (problem, its workgroup number there). Jobs
// are listed in one global order, so a workgroup that waits in a problem's
// first barrier waits only for workgroups whose earlier jobs come before that
// problem in every list: no cycle.
template <typename T, bool CP, bool KEEPS>
__global__ __launch_bounds__(512) void k_resident_batch(const RArgs<T>* __restrict__ probs, const int* __restrict__ off,
                                                        const int2* __restrict__ jobs) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int end = off[blockIdx.x + 1];
    for (int n = off[blockIdx.x]; n < end; ++n) {
        const int2 job = jobs[n];
        // the arguments through the constant address space: known uniform, and read
        // again by scalar loads where a register is short (as copies in registers
        // they made the server's kernels spill 28 and 125 vector registers, full and
        // compact, 6 and 77 like this; the batch's 3 and 6)
        const ConstArgs<T>* a = (const ConstArgs<T>*)(uintptr_t)(probs + __builtin_amdgcn_readfirstlane(job.x));
        resident_problem<T, 512, batch_planes<T>(CP), false, CP, true, KEEPS>(*a, __builtin_amdgcn_readfirstlane(job.y),
                                                                        lds_raw);
        __syncthreads();
    }
}

}  // namespace
}  // namespace pb
