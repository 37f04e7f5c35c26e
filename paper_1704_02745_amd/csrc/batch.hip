// Batched solves: many independent systems of uneven size in one persistent
// launch per kernel form (and the same work recorded once in a HIP graph for
// replay).
//
// Each problem is prepared into its own padded operator and state and runs in the
// resident form where its state fits the device (bricks that depend on its shape
// only, workgroups working through job lists), else in the streaming one: a tiling
// that depends on its shape only, and a share of the co-resident workgroups
// proportional to its expected work (nodes x max edge, since the Jacobi-CG
// iteration count grows with the grid edge). Workgroups of one problem
// synchronise only with each other, and every problem's result is bitwise the same
// alone or in any mix.
#include "solver.hpp"

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <memory>
#include <vector>

namespace pb {

// Problems in order of decreasing width (the longer first among equals), each on
// the workgroups that are free first.
void resident_schedule(const std::vector<int>& grid, const std::vector<double>& cost, int groups,
                       std::vector<int>& off, std::vector<int>& jobs) {
    const int n = (int)grid.size();
    std::vector<int> order(n);
    for (int k = 0; k < n; ++k) order[k] = k;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
        return grid[a] != grid[b] ? grid[a] > grid[b] : cost[a] > cost[b];
    });
    std::vector<std::vector<int>> list(groups);
    std::vector<double> free_at(groups, 0.0);
    std::vector<int> by(groups);
    for (int g = 0; g < groups; ++g) by[g] = g;
    for (int k : order) {
        const int G = grid[k];
        std::stable_sort(by.begin(), by.end(), [&](int a, int b) { return free_at[a] < free_at[b]; });
        const double end = free_at[by[G - 1]] + cost[k];
        std::vector<int> gang(by.begin(), by.begin() + G);
        std::sort(gang.begin(), gang.end());
        for (int w = 0; w < G; ++w) {
            list[gang[w]].push_back(k);
            list[gang[w]].push_back(w);
            free_at[gang[w]] = end;
        }
    }
    off.assign(1, 0);
    jobs.clear();
    for (int g = 0; g < groups; ++g) {
        jobs.insert(jobs.end(), list[g].begin(), list[g].end());
        off.push_back((int)jobs.size() / 2);
    }
}

namespace {

struct ProbRec {            // per-problem host-visible results in the workspace
    int flags;
    int pad;
    double rr, bb;          // true FP64 residual sums
    double pad2[5];
};

template <typename T>
struct Plan {
    int nprob = 0;
    size_t bytes = 0;
    size_t lds = 0;
    char* table = nullptr;          // device: KArgs records
    int* first = nullptr;           // device: workgroup offsets of the streaming launches
    SyncState* sync = nullptr;      // device: one per problem
    ProbRec* rec = nullptr;         // device: one per problem
    int* fit = nullptr;             // device: one per problem (coded coefficients fit the dictionary)
    // problems whose state fits the device run in the resident form, full or
    // compact, the others in the streaming form, one launch each (choose_forms);
    // `fall`: compact problems of a recorded batch, whose operator may turn out
    // not to fit its dictionary, in a streaming launch of their own
    struct Form {
        std::vector<int> of;        // indices of its problems
        size_t lds = 0;
        char* table = nullptr;      // device: RArgs records
        int* job_off = nullptr;     // device: job list offsets per workgroup
        char* jobs = nullptr;       // device: (index in of, workgroup) pairs
    };
    Form res[2];                    // full, compact
    std::vector<int> str, fall;
    size_t fall_lds = 0;
    int fall_grid = 0;              // workgroups of that launch
    std::vector<int> words;         // per problem: code words given: 0 no, 1 yes, 2 as its fit flag says
    std::vector<ResBatchPlan> rp;   // per problem (grid 0: streaming)
    std::vector<char*> slots;       // device: barrier words per problem
    char* all_slots = nullptr;      // and the range that holds them all
    size_t slot_bytes = 0;
    int groups = 0;                 // workgroups of a resident launch
    size_t str_lds = 0;             // LDS of the streaming form over every problem of the batch
    std::vector<Layout> L;
    std::vector<Tiling> t;
    std::vector<SolveBufs<T>> s;
    std::vector<Op<double>> op64;
    std::vector<double*> b64, x64, resp;
    std::vector<double*> partials;
};

bool problem_ok(const pb_problem& p) {
    return p.nx >= 1 && p.ny >= 1 && p.nz >= 1 && (int64_t)p.nx * p.ny * p.nz < (int64_t(1) << 36) &&
           std::isfinite(p.h) && p.h > 0 && std::isfinite(p.tol) && p.tol > 0 && p.eps_x && p.eps_y &&
           p.eps_z && p.kappa2 && p.rhs && p.x;
}

// Which problems run in which form, from each problem's shape and code words
// alone, so that its arithmetic does not depend on the others. A problem that
// only the compact form takes runs in it where it has code words, else in the
// streaming form. Where the device decides (words 2) it is in both launches, one
// of which skips it. The second is apart from the streaming launch: workgroups
// shared out to a problem that is then skipped would be lost to the others.
template <typename T>
void choose_forms(Plan<T>& P) {
    for (auto& f : P.res) {
        f.of.clear();
        f.lds = 0;
    }
    P.str.clear();
    P.fall.clear();
    P.lds = P.fall_lds = 0;
    for (int i = 0; i < P.nprob; ++i) {
        const ResBatchPlan& rp = P.rp[i];
        if (rp.grid <= 0 || (rp.compact && !P.words[i])) {
            P.str.push_back(i);
            P.lds = std::max(P.lds, P.t[i].lds);
            continue;
        }
        auto& f = P.res[rp.compact ? 1 : 0];
        f.of.push_back(i);
        f.lds = std::max(f.lds, rp.lds);
        if (rp.compact && P.words[i] == 2) {
            P.fall.push_back(i);
            P.fall_lds = std::max(P.fall_lds, P.t[i].lds);
        }
    }
}

// Carve the workspace (base may be null to size it). Returns false with an
// error set if a problem cannot be tiled.
template <typename T>
bool carve_batch(void* base, int nprob, const pb_problem* probs, Plan<T>& P, int zchunk = 0, bool resident = true) {
    size_t off = 0;
    auto take = [&](size_t bytes) -> void* {
        const size_t o = off;
        off = align_up(off + bytes, 256);
        return base ? (void*)((char*)base + o) : nullptr;
    };
    P.nprob = nprob;
    P.table = (char*)take(batch_kargs_bytes<T>() * (size_t)nprob);
    P.first = (int*)take(sizeof(int) * (size_t)(nprob + 2));
    P.sync = (SyncState*)take(sizeof(SyncState) * (size_t)nprob);
    P.rec = (ProbRec*)take(sizeof(ProbRec) * (size_t)nprob);
    P.fit = (int*)take(sizeof(int) * (size_t)nprob);
    size_t nres[2] = {0, 0}, njobs[2] = {0, 0};
    for (int i = 0; i < nprob; ++i) {
        const Layout L = make_layout(probs[i].nx, probs[i].ny, probs[i].nz);
        const Tiling t = batch_tiling<T>(L, zchunk);
        if (t.ntiles <= 0) {
            set_error("batch: problem %d (nx = %d) is too wide for the batch kernel's in-plane halo", i, L.nx);
            return false;
        }
        const ResBatchPlan rp = resident ? resident_batch_plan<T>(L) : ResBatchPlan{};
        P.rp.push_back(rp);
        P.str_lds = std::max(P.str_lds, t.lds);
        if (rp.grid > 0) {
            ++nres[rp.compact ? 1 : 0];
            njobs[rp.compact ? 1 : 0] += (size_t)rp.grid;
            P.groups = rp.groups;
        }
        const size_t n8 = sizeof(double) * (size_t)L.npad, nT = sizeof(T) * (size_t)L.npad;
        P.L.push_back(L);
        P.t.push_back(t);
        P.partials.push_back((double*)take(2 * sizeof(double) * kMaxPartials * (size_t)t.ntiles));
        P.resp.push_back((double*)take(sizeof(double) * 2 * (size_t)residual_blocks(L)));
        Op<double> o64;
        o64.cx = (double*)take(n8);
        o64.cy = (double*)take(n8);
        o64.cz = (double*)take(n8);
        o64.d = (double*)take(n8);
        P.op64.push_back(o64);
        P.b64.push_back((double*)take(n8));
        P.x64.push_back((double*)take(n8));
        SolveBufs<T> s{};
        if constexpr (sizeof(T) == sizeof(double)) {
            s.op = o64;
            s.b = P.b64.back();
            s.x = P.x64.back();
        } else {
            s.op.cx = (T*)take(nT); s.op.cy = (T*)take(nT); s.op.cz = (T*)take(nT); s.op.d = (T*)take(nT);
            s.b = (T*)take(nT);
            s.x = (T*)take(nT);
        }
        s.r = (T*)take(nT); s.r2 = (T*)take(nT);
        s.q = (T*)take(nT); s.q2 = (T*)take(nT);
        s.p0 = (T*)take(nT); s.p1 = (T*)take(nT);
        s.warm = probs[i].warm_start ? 1 : 0;
        P.s.push_back(s);
    }
    P.all_slots = base ? (char*)base + off : nullptr;
    const size_t slots0 = off;
    for (int i = 0; i < nprob; ++i) {
        P.slots.push_back(P.rp[i].grid > 0 ? (char*)take(P.rp[i].slot_bytes) : nullptr);
    }
    P.slot_bytes = off - slots0;
    for (int c = 0; c < 2; ++c)
        if (nres[c]) {
            P.res[c].table = (char*)take(resident_batch_args_bytes<T>() * nres[c]);
            P.res[c].job_off = (int*)take(sizeof(int) * (size_t)(P.groups + 1));
            P.res[c].jobs = (char*)take(2 * sizeof(int) * njobs[c]);
        }
    P.bytes = off;
    P.words.assign(nprob, 0);
    choose_forms(P);
    return true;
}

// Jacobi-CG iterations of a problem relative to others (the count grows about
// with the root of the edge once the salt screens the long waves).
double expected_iterations(const Layout& L) { return std::sqrt((double)std::max(L.nx, std::max(L.ny, L.nz))); }

// Workgroups per problem, proportional to nodes x max edge, at least one,
// at most the problem's tile count; returns the offsets (size nprob + 1).
std::vector<int> share_workgroups(const std::vector<Layout>& L, const std::vector<Tiling>& t, int capacity) {
    const int n = (int)L.size();
    std::vector<double> w(n);
    double tot = 0;
    for (int i = 0; i < n; ++i) {
        w[i] = (double)L[i].n * std::max(L[i].nx, std::max(L[i].ny, L[i].nz));
        tot += w[i];
    }
    std::vector<int> g(n, 1);
    int used = n;
    // hand out the remaining workgroups one at a time to the problem with the
    // largest work per workgroup that can still take one
    std::vector<double> load(n);
    for (int i = 0; i < n; ++i) load[i] = w[i] / g[i];
    while (used < capacity) {
        int best = -1;
        for (int i = 0; i < n; ++i)
            if (g[i] < t[i].ntiles && (best < 0 || load[i] > load[best])) best = i;
        if (best < 0) break;
        ++g[best];
        ++used;
        load[best] = w[best] / g[best];
    }
    std::vector<int> first(n + 1, 0);
    for (int i = 0; i < n; ++i) first[i + 1] = first[i] + g[i];
    (void)tot;
    return first;
}

template <typename T>
pb_status enqueue_prepare(const Plan<T>& P, const pb_problem* probs, hipStream_t st) {
    for (int i = 0; i < P.nprob; ++i) {
        const Op<float>* op32 = nullptr;
        float *b32 = nullptr, *x32 = nullptr;
        if constexpr (sizeof(T) == sizeof(float)) {
            op32 = &P.s[i].op;
            b32 = (float*)P.s[i].b;
            x32 = P.s[i].x;
        }
        pb_status e = launch_prepare64(probs[i].eps_x, probs[i].eps_y, probs[i].eps_z, probs[i].kappa2, probs[i].rhs,
                                       probs[i].x, probs[i].warm_start ? 1 : 0, 0, P.L[i], probs[i].h, P.op64[i],
                                       P.b64[i], P.x64[i], &P.rec[i].flags, st, op32, b32, x32);
        if (e != PB_OK) return e;
    }
    return PB_OK;
}

template <typename T>
pb_status enqueue_finish(const Plan<T>& P, const pb_problem* probs, hipStream_t st) {
    for (int i = 0; i < P.nprob; ++i) {
        pb_status e = PB_OK;
        if constexpr (sizeof(T) == sizeof(float)) e = launch_f32_to_f64(P.s[i].x, P.x64[i], P.L[i].npad, st);
        if (e != PB_OK) return e;
        e = launch_residual64(P.op64[i], P.b64[i], P.x64[i], P.L[i], 0, nullptr, nullptr, P.resp[i], &P.rec[i].rr, st);
        if (e != PB_OK) return e;
        e = launch_unpad<double>(P.x64[i], P.L[i], probs[i].x, st);
        if (e != PB_OK) return e;
    }
    return PB_OK;
}

template <typename T>
pb_status launch_solves(const Plan<T>& P, int grid, hipStream_t st, bool cooperative, int coded);

// Dynamic LDS of the streaming launch.
template <typename T>
size_t streaming_lds(const Plan<T>& P, int coded) {
    return P.lds + (coded ? kCodedLdsBytes : 0);
}

// The whole batch on `st`: clear flags and barrier state, prepare, solve,
// finish; nothing is read back to the host, so it can be recorded in a graph.
// Where P.words says 2 (FP32), the problem's dictionary, fit flag and code words
// are rebuilt on the device before the launches, whose kernels read the flag (the
// argument tables must carry the code words, dictionaries and flags).
template <typename T>
pb_status enqueue_batch(const Plan<T>& P, const pb_problem* probs, int grid, bool cooperative, hipStream_t st,
                        int coded = 0) {
    pb_status e = launch_fill<int>((int*)P.rec, (int64_t)(sizeof(ProbRec) / sizeof(int)) * P.nprob, 0, st);
    if (e != PB_OK) return e;
    e = launch_fill<int>((int*)P.sync, (int64_t)(sizeof(SyncState) / sizeof(int)) * P.nprob, 0, st);
    if (e != PB_OK) return e;
    e = enqueue_prepare<T>(P, probs, st);
    if (e != PB_OK) return e;
    if constexpr (sizeof(T) == sizeof(float)) {
        for (int i = 0; i < P.nprob; ++i)
            if (P.words[i] == 2) {
                e = enqueue_dictionary(P.s[i].op, P.L[i].npad, (void*)P.s[i].q, P.fit + i, st);
                if (e != PB_OK) return e;
                e = enqueue_encode(P.s[i].op, P.L[i].npad, P.s[i].q, (uint32_t*)P.s[i].q2, st, P.fit + i);
                if (e != PB_OK) return e;
            }
    }
    e = launch_solves<T>(P, grid, st, cooperative, coded);
    if (e != PB_OK) return e;
    return enqueue_finish<T>(P, probs, st);
}

// Write the per-problem kernel arguments (with each problem's code words and
// dictionary as P.words says). The streaming launches' records follow one
// another in one table.
template <typename T>
pb_status fill_table(const Plan<T>& P, const pb_problem* probs, hipStream_t st) {
    auto limit = [&](int i) {
        return probs[i].maxiter > 0 ? probs[i].maxiter : 10 * std::max(probs[i].nx, std::max(probs[i].ny, probs[i].nz));
    };
    auto args = [&](int i, auto&& fill) {
        const int words = P.words[i];
        fill(limit(i), words ? (const float*)P.s[i].q2 : nullptr, words ? dictionary_table(P.s[i].q) : nullptr,
             words == 2 ? (const int*)(P.fit + i) : nullptr);
    };
    const size_t nstr = P.str.size();
    std::vector<char> host(batch_kargs_bytes<T>() * (nstr + P.fall.size())), rhost[2];
    for (size_t k = 0; k < nstr + P.fall.size(); ++k) {
        const bool fall = k >= nstr;
        const int i = fall ? P.fall[k - nstr] : P.str[k];
        args(i, [&](int maxiter, const float* cw, const float* tab, const int* fit) {
            batch_fill_kargs<T>(host.data() + batch_kargs_bytes<T>() * k, P.L[i], P.s[i], &P.sync[i], P.partials[i],
                                P.t[i], probs[i].tol, maxiter, 0, 0, cw, tab, fit, fall);
        });
    }
    for (int c = 0; c < 2; ++c) {
        const auto& f = P.res[c];
        rhost[c].resize(resident_batch_args_bytes<T>() * f.of.size());
        double pass_us = 0.0;
        for (int i : f.of) pass_us += P.rp[i].us * limit(i);
        for (size_t k = 0; k < f.of.size(); ++k) {
            const int i = f.of[k];
            args(i, [&](int maxiter, const float* cw, const float* tab, const int* fit) {
                resident_batch_fill<T>(rhost[c].data() + resident_batch_args_bytes<T>() * k, P.L[i], P.s[i], &P.sync[i],
                                       P.slots[i], probs[i].tol, maxiter, (int)f.of.size(), pass_us, cw, tab, fit);
            });
        }
        if (!f.of.empty())
            PB_HIP(hipMemcpyAsync(f.table, rhost[c].data(), rhost[c].size(), hipMemcpyHostToDevice, st));
    }
    if (!host.empty()) PB_HIP(hipMemcpyAsync(P.table, host.data(), host.size(), hipMemcpyHostToDevice, st));
    PB_HIP(hipStreamSynchronize(st));
    return PB_OK;
}

// The solves: a launch of each resident form, then the streaming ones, each over
// the problems of its form. grid, coded: workgroups and kernel of the streaming
// launch (the compact problems' fallback runs uncoded: it has no dictionary).
template <typename T>
pb_status launch_solves(const Plan<T>& P, int grid, hipStream_t st, bool cooperative, int coded) {
    pb_status e = PB_OK;
    if (P.slot_bytes > 0) e = launch_fill<int>((int*)P.all_slots, (int64_t)(P.slot_bytes / sizeof(int)), 0, st);
    if (e != PB_OK) return e;
    for (int c = 0; c < 2; ++c) {
        const auto& f = P.res[c];
        if (f.of.empty()) continue;
        for (int i : f.of)
            if ((e = resident_batch_start<T>(P.L[i], P.s[i], st)) != PB_OK) return e;
        e = resident_batch_launch<T>(f.table, f.job_off, f.jobs, P.groups, f.lds, c == 1, st, cooperative);
        if (e != PB_OK) return e;
    }
    const int nstr = (int)P.str.size(), nfall = (int)P.fall.size();
    if (nstr > 0) e = batch_launch<T>(P.table, P.first, nstr, grid, streaming_lds(P, coded), st, cooperative, coded);
    if (e == PB_OK && nfall > 0)
        e = batch_launch<T>(P.table + batch_kargs_bytes<T>() * nstr, P.first + nstr + 1, nfall, P.fall_grid, P.fall_lds,
                            st, cooperative, 0);
    return e;
}

// A batch holds at most as many problems as the streaming form has co-resident
// workgroups, whatever form its problems run in.
template <typename T>
pb_status check_count(const Plan<T>& P) {
    const int most = batch_capacity<T>(P.str_lds);
    if (most >= P.nprob) return PB_OK;
    set_error("batch: %d problems but only %d co-resident workgroups; split the batch", P.nprob, most);
    return PB_ERR_ARG;
}

// Settle the forms (choose_forms, from P.words) and upload the per-problem kernel
// arguments, the workgroup offsets and the job lists. coded: the streaming
// launch's kernel; grid: its workgroups.
template <typename T>
pb_status upload_table(Plan<T>& P, const pb_problem* probs, int& grid, int coded, hipStream_t st) {
    grid = 0;
    choose_forms(P);
    if (const pb_status e = check_count(P); e != PB_OK) return e;
    auto share = [&](const std::vector<int>& of, int cap) {
        std::vector<Layout> L;
        std::vector<Tiling> t;
        for (int i : of) {
            L.push_back(P.L[i]);
            t.push_back(P.t[i]);
        }
        return share_workgroups(L, t, cap);
    };
    std::vector<int> first, ffirst;
    if (!P.str.empty()) {
        first = share(P.str, batch_capacity<T>(streaming_lds(P, coded), coded));
        grid = first.back();
        PB_HIP(hipMemcpyAsync(P.first, first.data(), sizeof(int) * first.size(), hipMemcpyHostToDevice, st));
    }
    if (!P.fall.empty()) {
        ffirst = share(P.fall, batch_capacity<T>(P.fall_lds));
        P.fall_grid = ffirst.back();
        PB_HIP(hipMemcpyAsync(P.first + P.str.size() + 1, ffirst.data(), sizeof(int) * ffirst.size(),
                              hipMemcpyHostToDevice, st));
    }
    std::vector<int> off[2], jobs[2];
    for (int c = 0; c < 2; ++c) {
        const auto& f = P.res[c];
        if (f.of.empty()) continue;
        std::vector<int> grids;
        std::vector<double> cost;
        for (int i : f.of) {
            grids.push_back(P.rp[i].grid);
            cost.push_back(P.rp[i].us * expected_iterations(P.L[i]));
        }
        resident_schedule(grids, cost, P.groups, off[c], jobs[c]);
        PB_HIP(hipMemcpyAsync(f.job_off, off[c].data(), sizeof(int) * off[c].size(), hipMemcpyHostToDevice, st));
        PB_HIP(hipMemcpyAsync(f.jobs, jobs[c].data(), sizeof(int) * jobs[c].size(), hipMemcpyHostToDevice, st));
    }
    return fill_table<T>(P, probs, st);
}

// Whether every problem of the batch can have code words: the arrays that hold
// them are large enough, and the coded streaming kernel takes as many problems.
template <typename T>
bool can_code(const Plan<T>& P, int coded) {
    if (sizeof(T) != sizeof(float) || !coded_coefficients()) return false;
    for (const Layout& L : P.L)
        if (!coded_layout_ok(L)) return false;
    return batch_capacity<T>(P.str_lds + kCodedLdsBytes, coded) >= P.nprob;
}

// Whether a problem runs in the compact form if its operator fits a dictionary
// (whatever pb_set_coded_coefficients says, as in a solve of its own).
template <typename T>
bool wants_words(const Plan<T>& P, int i) {
    return sizeof(T) == sizeof(float) && P.rp[i].grid > 0 && P.rp[i].compact && coded_layout_ok(P.L[i]);
}

// The direct (not graph-recorded) batch: as enqueue_batch, with the fit flags
// read back to the host once, after the preparation. The compact problems whose
// operator fits get code words; every problem does where all fit and the coded
// kernel keeps the grid co-resident (coded). The code words go to a problem's q2
// and the dictionary to its q (the batch's pass form uses neither).
template <typename T>
pb_status enqueue_batch_direct(Plan<T>& P, const pb_problem* probs, hipStream_t st) {
    pb_status e = launch_fill<int>((int*)P.rec, (int64_t)(sizeof(ProbRec) / sizeof(int)) * P.nprob, 0, st);
    if (e != PB_OK) return e;
    e = launch_fill<int>((int*)P.sync, (int64_t)(sizeof(SyncState) / sizeof(int)) * P.nprob, 0, st);
    if (e != PB_OK) return e;
    e = enqueue_prepare<T>(P, probs, st);
    if (e != PB_OK) return e;
    bool coded = can_code(P, 1);
    if constexpr (sizeof(T) == sizeof(float)) {
        std::vector<int> fit(P.nprob, 0);
        bool any = false;
        for (int i = 0; i < P.nprob; ++i) {
            if (!coded && !wants_words(P, i)) continue;
            any = true;
            e = enqueue_dictionary(P.s[i].op, P.L[i].npad, (void*)P.s[i].q, P.fit + i, st);
            if (e != PB_OK) return e;
        }
        if (any) {
            PB_HIP(hipMemcpyAsync(fit.data(), P.fit, sizeof(int) * P.nprob, hipMemcpyDeviceToHost, st));
            PB_HIP(hipStreamSynchronize(st));
        }
        for (int i = 0; i < P.nprob; ++i) coded = coded && fit[i] == 1;
        for (int i = 0; i < P.nprob; ++i) {
            P.words[i] = coded || (wants_words(P, i) && fit[i] == 1) ? 1 : 0;
            if (!P.words[i]) continue;
            e = enqueue_encode(P.s[i].op, P.L[i].npad, P.s[i].q, (uint32_t*)P.s[i].q2, st);
            if (e != PB_OK) return e;
        }
    }
    int grid = 0;
    e = upload_table<T>(P, probs, grid, coded ? 1 : 0, st);
    if (e != PB_OK) return e;
    e = launch_solves<T>(P, grid, st, true, coded ? 1 : 0);
    if (e != PB_OK) return e;
    return enqueue_finish<T>(P, probs, st);
}

// Read back per-problem results; returns the batch status (first error, else
// PB_NOT_CONVERGED if any problem did not converge, else PB_OK).
template <typename T>
pb_status collect(const Plan<T>& P, hipStream_t st, pb_info* infos, double seconds) {
    std::vector<SyncState> S(P.nprob);
    std::vector<ProbRec> R(P.nprob);
    PB_HIP(hipMemcpyAsync(S.data(), P.sync, sizeof(SyncState) * P.nprob, hipMemcpyDeviceToHost, st));
    PB_HIP(hipMemcpyAsync(R.data(), P.rec, sizeof(ProbRec) * P.nprob, hipMemcpyDeviceToHost, st));
    PB_HIP(hipStreamSynchronize(st));
    pb_status worst = PB_OK;
    for (int i = 0; i < P.nprob; ++i) {
        int status = S[i].status;
        if (R[i].flags & FLAG_BAD_COEF) status = PB_ERR_ARG;
        else if (R[i].flags & (FLAG_BAD_RHS | FLAG_BAD_GUESS)) status = PB_ERR_NONFINITE;
        if (infos) {
            pb_info& f = infos[i];
            std::memset(&f, 0, sizeof(f));
            f.iters = S[i].iters;
            f.status = status;
            f.kernel_launches = 1;
            f.relres_recur = S[i].bb > 0 ? std::sqrt(S[i].rr) / std::sqrt(S[i].bb) : 0.0;
            f.relres_true = R[i].bb > 0 ? std::sqrt(R[i].rr) / std::sqrt(R[i].bb) : 0.0;
            f.seconds = seconds;
        }
        if (status < 0 && worst >= 0) worst = (pb_status)status;
        if (status == PB_NOT_CONVERGED && worst == PB_OK) worst = PB_NOT_CONVERGED;
    }
    if (worst < 0) set_error("batch: at least one problem failed (see its pb_info.status)");
    return worst;
}

template <typename T>
pb_status solve_batch_impl(int nprob, const pb_problem* probs, void* ws, size_t wsb, hipStream_t st, pb_info* infos) {
    const auto t0 = std::chrono::steady_clock::now();
    Plan<T> P;
    if (!carve_batch<T>(ws, nprob, probs, P)) return PB_ERR_ARG;
    if (wsb < P.bytes) {
        set_error("pb_solve_batch: workspace of %zu bytes, %zu needed", wsb, P.bytes);
        return PB_ERR_NOMEM;
    }
    hipEvent_t ev[2];
    PB_HIP(hipEventCreate(&ev[0]));
    PB_HIP(hipEventCreate(&ev[1]));
    PB_HIP(hipEventRecord(ev[0], st));
    pb_status e = enqueue_batch_direct<T>(P, probs, st);
    if (e != PB_OK) {
        (void)hipEventDestroy(ev[0]);
        (void)hipEventDestroy(ev[1]);
        return e;
    }
    PB_HIP(hipEventRecord(ev[1], st));
    PB_HIP(hipStreamSynchronize(st));
    float ms = 0;
    PB_HIP(hipEventElapsedTime(&ms, ev[0], ev[1]));
    (void)hipEventDestroy(ev[0]);
    (void)hipEventDestroy(ev[1]);
    const double secs = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    const pb_status st_all = collect<T>(P, st, infos, secs);
    if (infos)
        for (int i = 0; i < nprob; ++i) {
            infos[i].kernel_seconds = 1e-3 * ms;
            infos[i].coded_launches = P.words[i] ? 1 : 0;
        }
    return st_all;
}

// z-chunks the batch autotuner times.
constexpr int kBatchZCandidates[] = {16, 24, 32, 48, 64};

// Time the streaming batch kernel for each candidate z-chunk, each problem capped
// at `iters` iterations (state cleared and prepared as for a solve, but no
// hand-back: the problems' x arrays are not written), and make the fastest the
// device's batch z-chunk. The problems that stream are timed (the z-chunk is of no
// effect on the others); all of them where none does.
template <typename T>
pb_status batch_autotune_impl(int nprob, const pb_problem* probs, int iters, void* ws, size_t wsb, hipStream_t st,
                              int* best_z, double* best_seconds) {
    std::vector<pb_problem> trial;
    for (int i = 0; i < nprob; ++i)
        if (resident_batch_plan<T>(make_layout(probs[i].nx, probs[i].ny, probs[i].nz)).grid == 0)
            trial.push_back(probs[i]);
    if (trial.empty()) trial.assign(probs, probs + nprob);
    for (auto& p : trial) p.maxiter = iters;
    const int ntrial = (int)trial.size();
    hipEvent_t ev[2];
    PB_HIP(hipEventCreate(&ev[0]));
    PB_HIP(hipEventCreate(&ev[1]));
    double best = 1e300;
    int bz = 0;
    pb_status e = PB_OK;
    for (int z : kBatchZCandidates) {
        // (the whole batch as its solve would be checked)
        Plan<T> all, P;
        if (!carve_batch<T>(nullptr, nprob, probs, all, z, false)) { e = PB_ERR_ARG; break; }
        if (wsb < all.bytes) {
            set_error("pb_batch_autotune: workspace of %zu bytes, %zu needed", wsb, all.bytes);
            e = PB_ERR_NOMEM;
            break;
        }
        if ((e = check_count(all)) != PB_OK) break;
        if (!carve_batch<T>(ws, ntrial, trial.data(), P, z, false)) { e = PB_ERR_ARG; break; }
        int grid = 0;
        if ((e = upload_table<T>(P, trial.data(), grid, 0, st)) != PB_OK) break;
        if ((e = launch_fill<int>((int*)P.rec, (int64_t)(sizeof(ProbRec) / sizeof(int)) * ntrial, 0, st)) != PB_OK) break;
        if ((e = launch_fill<int>((int*)P.sync, (int64_t)(sizeof(SyncState) / sizeof(int)) * ntrial, 0, st)) != PB_OK) break;
        if ((e = enqueue_prepare<T>(P, trial.data(), st)) != PB_OK) break;
        // solves run coded where they can: time the kernel they will run (the
        // per-problem checked form, which needs no read-back here)
        int coded = 0;
        if constexpr (sizeof(T) == sizeof(float)) {
            bool can = coded_coefficients() != 0 && batch_capacity<T>(P.lds + kCodedLdsBytes, 2) >= grid;
            for (int i = 0; i < ntrial && can; ++i) can = coded_layout_ok(P.L[i]);
            if (can) {
                for (int i = 0; i < ntrial && e == PB_OK; ++i) {
                    e = enqueue_dictionary(P.s[i].op, P.L[i].npad, (void*)P.s[i].q, P.fit + i, st);
                    if (e == PB_OK) e = enqueue_encode(P.s[i].op, P.L[i].npad, P.s[i].q, (uint32_t*)P.s[i].q2, st,
                                                       P.fit + i);
                }
                P.words.assign(ntrial, 2);
                if (e != PB_OK || (e = fill_table<T>(P, trial.data(), st)) != PB_OK) break;
                coded = 2;
            }
        }
        if (hipEventRecord(ev[0], st) != hipSuccess) { e = PB_ERR_HIP; break; }
        if ((e = batch_launch<T>(P.table, P.first, ntrial, grid, coded ? P.lds + kCodedLdsBytes : P.lds, st, true,
                                 coded)) != PB_OK)
            break;
        if (hipEventRecord(ev[1], st) != hipSuccess || hipStreamSynchronize(st) != hipSuccess) { e = PB_ERR_HIP; break; }
        float ms = 0.0f;
        if (hipEventElapsedTime(&ms, ev[0], ev[1]) != hipSuccess) { e = PB_ERR_HIP; break; }
        if (ms < best) {
            best = ms;
            bz = z;
        }
    }
    (void)hipEventDestroy(ev[0]);
    (void)hipEventDestroy(ev[1]);
    if (e != PB_OK) return e;
    set_batch_zchunk(bz);
    if (best_z) *best_z = bz;
    if (best_seconds) *best_seconds = 1e-3 * best;
    return PB_OK;
}

bool batch_args_ok(int nprob, const pb_problem* probs, int precision) {
    if (nprob < 1 || !probs || (precision != PB_F32 && precision != PB_F64)) return false;
    for (int i = 0; i < nprob; ++i)
        if (!problem_ok(probs[i])) return false;
    return true;
}

}  // namespace

struct BatchGraph {
    int precision = 0;
    int nprob = 0;
    std::vector<pb_problem> probs;
    std::unique_ptr<Plan<float>> p32;
    std::unique_ptr<Plan<double>> p64;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    bool cooperative = true;
    int coded = 0;   // 2: every problem's dictionary is built and the streaming kernel reads its fit flag
    hipEvent_t ev[2] = {nullptr, nullptr};
};

}  // namespace pb

using namespace pb;

struct pb_batch_graph : public pb::BatchGraph {};

extern "C" size_t pb_batch_workspace_bytes(int32_t nprob, const pb_problem* probs, int32_t precision) {
    if (!batch_args_ok(nprob, probs, precision)) return 0;
    if (precision == PB_F64) {
        Plan<double> P;
        return carve_batch<double>(nullptr, nprob, probs, P) ? P.bytes : 0;
    }
    Plan<float> P;
    return carve_batch<float>(nullptr, nprob, probs, P) ? P.bytes : 0;
}

extern "C" pb_status pb_solve_batch(int32_t nprob, const pb_problem* probs, int32_t precision, void* workspace,
                                    size_t workspace_bytes, void* stream, pb_info* infos) {
    PB_ARG(batch_args_ok(nprob, probs, precision),
           "pb_solve_batch: need nprob >= 1, valid problems (dims >= 1, h > 0, tol > 0, non-null arrays), "
           "precision PB_F32 or PB_F64");
    PB_ARG(workspace != nullptr && ((uintptr_t)workspace & 255) == 0, "pb_solve_batch: null or misaligned workspace");
    hipStream_t st = (hipStream_t)stream;
    if (precision == PB_F64) return solve_batch_impl<double>(nprob, probs, workspace, workspace_bytes, st, infos);
    return solve_batch_impl<float>(nprob, probs, workspace, workspace_bytes, st, infos);
}

extern "C" pb_status pb_batch_set_zchunk(int32_t zchunk) {
    PB_ARG(zchunk >= 1 && zchunk <= 4096, "pb_batch_set_zchunk: zchunk in [1, 4096]");
    set_batch_zchunk(zchunk);
    return PB_OK;
}

extern "C" int32_t pb_batch_get_zchunk(void) { return batch_zchunk(); }

extern "C" size_t pb_batch_autotune_workspace_bytes(int32_t nprob, const pb_problem* probs, int32_t precision) {
    if (!batch_args_ok(nprob, probs, precision)) return 0;
    size_t most = 0;
    for (int z : kBatchZCandidates) {
        size_t b = 0;
        if (precision == PB_F64) {
            Plan<double> P;
            b = carve_batch<double>(nullptr, nprob, probs, P, z, false) ? P.bytes : 0;
        } else {
            Plan<float> P;
            b = carve_batch<float>(nullptr, nprob, probs, P, z, false) ? P.bytes : 0;
        }
        if (b == 0) return 0;
        most = std::max(most, b);
    }
    return most;
}

extern "C" pb_status pb_batch_autotune(int32_t nprob, const pb_problem* probs, int32_t precision,
                                       int32_t iters_per_trial, void* workspace, size_t workspace_bytes, void* stream,
                                       int32_t* best_zchunk, double* best_seconds) {
    PB_ARG(batch_args_ok(nprob, probs, precision),
           "pb_batch_autotune: need nprob >= 1, valid problems, precision PB_F32 or PB_F64");
    PB_ARG(iters_per_trial >= 1, "pb_batch_autotune: iters_per_trial >= 1");
    PB_ARG(workspace != nullptr && ((uintptr_t)workspace & 255) == 0,
           "pb_batch_autotune: null or misaligned workspace");
    hipStream_t st = (hipStream_t)stream;
    if (precision == PB_F64)
        return batch_autotune_impl<double>(nprob, probs, iters_per_trial, workspace, workspace_bytes, st,
                                           best_zchunk, best_seconds);
    return batch_autotune_impl<float>(nprob, probs, iters_per_trial, workspace, workspace_bytes, st, best_zchunk,
                                      best_seconds);
}

namespace {

template <typename T>
pb_status graph_build(pb_batch_graph* G, Plan<T>& P, void* ws, size_t wsb, hipStream_t st) {
    if (!carve_batch<T>(ws, G->nprob, G->probs.data(), P)) return PB_ERR_ARG;
    if (wsb < P.bytes) {
        set_error("pb_batch_graph_create: workspace of %zu bytes, %zu needed", wsb, P.bytes);
        return PB_ERR_NOMEM;
    }
    // coded coefficients, decided on the device at every replay (the
    // coefficients may change between replays)
    G->coded = can_code(P, 2) ? 2 : 0;
    for (int i = 0; i < P.nprob; ++i) P.words[i] = G->coded || wants_words(P, i) ? 2 : 0;
    int grid = 0;
    pb_status e = upload_table<T>(P, G->probs.data(), grid, G->coded, st);
    if (e != PB_OK) return e;
    hipStream_t cs;
    PB_HIP(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
    for (int attempt = 0; attempt < 2; ++attempt) {
        const bool coop = attempt == 0;
        if (hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal) != hipSuccess) break;
        const pb_status ee = enqueue_batch<T>(P, G->probs.data(), grid, coop, cs, G->coded);
        hipGraph_t g = nullptr;
        const hipError_t he = hipStreamEndCapture(cs, &g);
        if (ee == PB_OK && he == hipSuccess && g) {
            if (hipGraphInstantiate(&G->exec, g, nullptr, nullptr, 0) == hipSuccess) {
                G->graph = g;
                G->cooperative = coop;
                break;
            }
        }
        if (g) (void)hipGraphDestroy(g);
        (void)hipGetLastError();
    }
    (void)hipStreamDestroy(cs);
    if (!G->exec) {
        set_error("pb_batch_graph_create: could not capture the batch into a graph");
        return PB_ERR_HIP;
    }
    PB_HIP(hipEventCreate(&G->ev[0]));
    PB_HIP(hipEventCreate(&G->ev[1]));
    return PB_OK;
}

}  // namespace

extern "C" pb_status pb_batch_graph_create(int32_t nprob, const pb_problem* probs, int32_t precision, void* workspace,
                                           size_t workspace_bytes, void* stream, pb_batch_graph** out) {
    PB_ARG(out != nullptr, "pb_batch_graph_create: null output handle");
    *out = nullptr;
    PB_ARG(batch_args_ok(nprob, probs, precision), "pb_batch_graph_create: invalid problems or precision");
    PB_ARG(workspace != nullptr && ((uintptr_t)workspace & 255) == 0,
           "pb_batch_graph_create: null or misaligned workspace");
    std::unique_ptr<pb_batch_graph> G(new pb_batch_graph());
    G->precision = precision;
    G->nprob = nprob;
    G->probs.assign(probs, probs + nprob);
    hipStream_t st = (hipStream_t)stream;
    pb_status e;
    if (precision == PB_F64) {
        G->p64.reset(new Plan<double>());
        e = graph_build<double>(G.get(), *G->p64, workspace, workspace_bytes, st);
    } else {
        G->p32.reset(new Plan<float>());
        e = graph_build<float>(G.get(), *G->p32, workspace, workspace_bytes, st);
    }
    if (e != PB_OK) {
        if (G->exec) (void)hipGraphExecDestroy(G->exec);
        if (G->graph) (void)hipGraphDestroy(G->graph);
        return e;
    }
    *out = G.release();
    return PB_OK;
}

extern "C" pb_status pb_batch_graph_launch(pb_batch_graph* G, void* stream) {
    PB_ARG(G && G->exec, "pb_batch_graph_launch: null graph");
    hipStream_t st = (hipStream_t)stream;
    PB_HIP(hipEventRecord(G->ev[0], st));
    PB_HIP(hipGraphLaunch(G->exec, st));
    PB_HIP(hipEventRecord(G->ev[1], st));
    return PB_OK;
}

extern "C" pb_status pb_batch_graph_results(pb_batch_graph* G, void* stream, pb_info* infos) {
    PB_ARG(G && G->exec, "pb_batch_graph_results: null graph");
    hipStream_t st = (hipStream_t)stream;
    PB_HIP(hipStreamSynchronize(st));
    float ms = 0;
    PB_HIP(hipEventElapsedTime(&ms, G->ev[0], G->ev[1]));
    const pb_status s = G->precision == PB_F64 ? collect<double>(*G->p64, st, infos, 1e-3 * ms)
                                               : collect<float>(*G->p32, st, infos, 1e-3 * ms);
    std::vector<int> fit(G->nprob, 0);
    if (infos && G->p32) {
        PB_HIP(hipMemcpyAsync(fit.data(), G->p32->fit, sizeof(int) * G->nprob, hipMemcpyDeviceToHost, st));
        PB_HIP(hipStreamSynchronize(st));
    }
    if (infos)
        for (int i = 0; i < G->nprob; ++i) {
            infos[i].kernel_seconds = 1e-3 * ms;
            infos[i].coded_launches = G->p32 && G->p32->words[i] && fit[i] == 1 ? 1 : 0;
        }
    return s;
}

extern "C" int32_t pb_batch_graph_is_cooperative(const pb_batch_graph* G) { return G && G->cooperative ? 1 : 0; }

extern "C" void pb_batch_graph_destroy(pb_batch_graph* G) {
    if (!G) return;
    if (G->exec) (void)hipGraphExecDestroy(G->exec);
    if (G->graph) (void)hipGraphDestroy(G->graph);
    if (G->ev[0]) (void)hipEventDestroy(G->ev[0]);
    if (G->ev[1]) (void)hipEventDestroy(G->ev[1]);
    delete G;
}
