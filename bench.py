"""Benchmark: linear FDPB Jacobi-PCG on one MI355X.

One step = the whole hot path on the 257^3 workload (20,000-atom synthetic
globule, h = 0.5 A): GPU setup (classification, edge dielectrics, salt term,
charge spreading, Debye-Hueckel boundary), the mixed-precision solve (FP32
fused JPCG to 1e-4 inside an FP64 refinement loop to a 1e-9 relative
residual) and the energy. Inputs (atom arrays) are resident on the device
before the timed region; outputs stay on the device.

value = algorithmic HBM bytes of the fused JPCG launches in the timed steps /
wall time of the timed steps (GB/s), at 40 B per unknown per iteration
whichever pass form runs (the floor of any schedule that keeps the operator
as four FP32 arrays), so it scales with iterations per second: an effective
rate. The roofline block reports the fused kernel alone: the same bytes over
its own summed duration (HIP events on the solve stream, recorded by the
library), beside the bytes the running form itself moves (24.5 B on average with
coded coefficients, the default when the operator fits its dictionary:
form_achieved, form_frac), the counted HBM traffic (when the committed
counter summary matches the kernel source) and three streaming ceilings
measured in the same run: the runtime's device copy and the library's own
copy kernel with nontemporal and with cached accesses.
The CPU baseline is the FP64 NumPy oracle timed on a bounded sample of the
same workload.

python bench.py [--gpus 1] [--steps K] [--warmup W] [--no-cpu-baseline] [--coded 0|1]
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import resource
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "JPCG HBM GB/s (% peak) at 257^3; served solves/s + p99 latency at tol 1e-6"
PEAK_GBS = 8000.0
# Algorithmic bytes per unknown (FP32): the schedule-independent floor of one
# JPCG iteration, x, r and p each read and written (24 B) plus the four
# operator arrays read once (16 B) = 40 B, whatever pass form runs. Per
# launch add the initial pass (read b, write r and p: 12 B) and the final x
# update (read x, p, write x: 12 B), less the x update the first iteration
# skips (8 B). The pass forms themselves move 48 B (form 0, stores A.p),
# 40 B (form 1, recomputes it) or 28 B (form 1 with coded coefficients: the
# operator read as one 4-byte word of dictionary codes per unknown) per
# unknown per iteration. Form 1 reads and writes x (8 B) in every second pass
# where beta is at least 0.8, which leaves it out of some 44% of the passes of
# the refined 257^3 solve: 3.5 B less on average. That figure is reported beside
# the metric.
ITER_BYTES = 40
INIT_BYTES = 12 - 8 + 12
PASS_BYTES_BY_SCHEME = {0: 48, 1: 36.5}
CODED_PASS_BYTES = 24.5


def form_bytes(scheme: int, coded: bool):
    """Bytes per unknown and iteration of a pass form; None for the resident form (scheme + 2)."""
    if scheme >= 2:
        return None
    return CODED_PASS_BYTES if (scheme == 1 and coded) else PASS_BYTES_BY_SCHEME[scheme]
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "jpcg_fused_f32_257_traffic.txt")
KERNEL_SRC = os.path.join(ROOT, "paper_1704_02745_amd", "csrc", "jpcg.hip")


def launch_bytes(n: int, iters: int, launches: int) -> float:
    return float(n) * (ITER_BYTES * iters + INIT_BYTES * launches)


def measured_traffic():
    """Per-launch HBM bytes of the fused kernel from the committed rocprofv3
    counter summary, if it was taken on the current kernel source."""
    if not os.path.exists(TRAFFIC_FILE):
        return None
    kv = {}
    for line in open(TRAFFIC_FILE):
        if ":" in line and not line.startswith("#"):
            k, v = line.split(":", 1)
            kv[k.strip()] = v.strip()
    sha = hashlib.sha256(open(KERNEL_SRC, "rb").read()).hexdigest()
    if kv.get("kernel_source_sha256") != sha:
        return None
    try:
        return float(kv["hbm_bytes_per_launch"])
    except (KeyError, ValueError):
        return None


def cpu_model() -> str:
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def copy_ceiling(torch, dev, gib=1, reps=10):
    """Device-to-device copy rate (read + write bytes / time) of a `gib` GiB
    FP32 buffer, timed with HIP events: the plain-streaming ceiling measured
    beside the kernel."""
    n = (gib << 30) // 4
    src = torch.ones(n, dtype=torch.float32, device=dev)
    dst = torch.empty_like(src)
    dst.copy_(src)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record()
    for _ in range(reps):
        dst.copy_(src)
    e1.record()
    torch.cuda.synchronize()
    gbs = 2.0 * 4 * n * reps / (1e-3 * e0.elapsed_time(e1)) / 1e9
    del src, dst
    torch.cuda.empty_cache()
    return round(gbs, 1)


def stream_ceiling(pbgpu, torch, dev, gib=1, reps=10, nontemporal=True):
    """The library's own streaming kernel (pb_stream_copy: 16-byte vector
    loads and stores, nontemporal or cached, as the fused pass issues them)
    over a `gib` GiB FP32 buffer: read + write bytes / time, HIP events on the
    stream it runs on."""
    n = (gib << 30) // 4
    src = torch.ones(n, dtype=torch.float32, device=dev)
    dst = torch.empty_like(src)
    stream = torch.cuda.current_stream()
    pbgpu.stream_copy(src, dst, nontemporal, stream)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record(stream)
    for _ in range(reps):
        pbgpu.stream_copy(src, dst, nontemporal, stream)
    e1.record(stream)
    torch.cuda.synchronize()
    gbs = 2.0 * 4 * n * reps / (1e-3 * e0.elapsed_time(e1)) / 1e9
    del src, dst
    torch.cuda.empty_cache()
    return round(gbs, 1)


def cpu_baseline(prob, n_iters=40):
    """FP64 oracle Jacobi PCG at the full 257^3 size, bounded to n_iters
    iterations (about 10-15 s of host work). The sample system uses the oracle's own classification,
    edges, salt term and charges; its boundary values are zero (the boundary
    sum alone would take minutes in NumPy and does not change the iteration
    cost)."""
    import numpy as np
    from oracle import fdpb, pcg
    g = prob.grid
    mask = fdpb.classify(g.nx, g.ny, g.nz, g.h, g.origin, prob.mol.xyz, prob.mol.radius)
    ex, ey, ez = fdpb.dielectric_edges(mask, prob.eps_in, prob.eps_out)
    k2 = fdpb.salt_term(mask, prob.eps_out, prob.kappa_d2)
    q = fdpb.spread_charges(g.nx, g.ny, g.nz, g.h, g.origin, prob.mol.xyz, prob.mol.charge)
    s = fdpb.System(h=g.h, eps_x=ex, eps_y=ey, eps_z=ez, kappa2=k2, b=fdpb.FOUR_PI * q / g.h ** 3)
    r0 = resource.getrusage(resource.RUSAGE_SELF)
    t0 = time.perf_counter()
    res = pcg.pcg(lambda v: fdpb.apply(s, v), s.b, fdpb.diagonal(s), 1e-300, n_iters)
    wall = time.perf_counter() - t0
    r1 = resource.getrusage(resource.RUSAGE_SELF)
    cpu = (r1.ru_utime - r0.ru_utime) + (r1.ru_stime - r0.ru_stime)
    n = g.nx * g.ny * g.nz
    its = res.iters / wall
    return {"value": round(its * ITER_BYTES * n / 1e9, 3), "unit": "GB/s",
            "cores": max(1, int(round(cpu / wall))), "kind": "oracle",
            "sample": f"{res.iters} FP64 NumPy Jacobi-PCG iterations of the oracle at 257^3 "
                      f"(same operator, zero boundary), {wall:.1f} s wall; rate scaled by the "
                      f"metric's {ITER_BYTES} B/unknown per iteration",
            "iters_per_s": round(its, 4), "os_cpu_count": os.cpu_count(), "cpu_model": cpu_model()}


GOLDEN_C2 = os.path.join(ROOT, "tests", "golden", "c2_257_oracle.json")


def oracle_golden_errors(x, e):
    """phi and energy of the last step against the oracle's FP64 solution of
    the same workload (solved to 1e-12, stored at a seeded node sample by
    tests/golden/make_fullsize_golden.py)."""
    import numpy as np
    import torch
    if not os.path.exists(GOLDEN_C2):
        return None
    with open(GOLDEN_C2) as f:
        gold = json.load(f)
    nodes = torch.as_tensor(np.asarray(gold["sample_nodes"], np.int64), device=x.device)
    got = x.reshape(-1)[nodes].cpu().numpy()
    err = float(np.abs(got - np.asarray(gold["sample_phi"])).max() / gold["max_abs_phi"])
    return {"phi_max_rel_err": err, "sample_nodes": len(gold["sample_nodes"]),
            "energy_kcal_oracle": gold["energy_kcal"],
            "energy_rel_err": abs(e - gold["energy_kcal"]) / abs(gold["energy_kcal"]),
            "oracle_relres_true": gold["true_relres"]}


# DIA form: 7 diagonals (28 B) + p (4 B) read, q (4 B) written by the SpMV
# with p.q; x, r updated with r.(r/d), r.r (x, r read and written, p, q, d
# read: 28 B); p = r/d + beta p (r, d, p read, p written: 16 B).
DIA_ITER_BYTES = 80


def bench_c1(pbgpu, torch, synth, dev, reps=3):
    """Config 1: 129^3 FP32 to 1e-6, fused matrix-free stencil vs the DIA form."""
    p = synth.config1()
    g = p.grid
    sm = pbgpu.setup(g, p.mol.xyz, p.mol.radius, p.mol.charge, p.eps_in, p.eps_out, p.kappa_d2, device=dev)
    n = g.nx * g.ny * g.nz
    out = {}
    tun = pbgpu.autotune(sm, precision="f32", iters_per_trial=20)   # untimed: this shape's tiling
    sch = tun["scheme"]
    for op in ("stencil", "dia"):
        pbgpu.solve(sm, tol=1e-6, precision="f32", op=op)
        best = None
        for _ in range(reps):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            _, info = pbgpu.solve(sm, tol=1e-6, precision="f32", op=op)
            torch.cuda.synchronize()
            dt = time.perf_counter() - t0
            if best is None or dt < best[0]:
                best = (dt, info)
        dt, info = best
        coded = info["coded_launches"] > 0
        per = form_bytes(sch, coded) if op == "stencil" else DIA_ITER_BYTES
        out[op] = {"iters": info["iters"], "solve_ms": round(1e3 * dt, 3),
                   "iter_loop_ms": round(1e3 * info["kernel_seconds"], 3),
                   "us_per_iter": round(1e6 * info["kernel_seconds"] / max(info["iters"], 1), 2),
                   "algorithmic_gbs": round(ITER_BYTES * n * info["iters"] / info["kernel_seconds"] / 1e9, 1),
                   "form_gbs": per and round(per * n * info["iters"] / info["kernel_seconds"] / 1e9, 1),
                   "form_bytes_per_node_iter": per, "relres_true": info["relres_true"]}
        if op == "stencil":
            out[op]["pass_form"] = sch if sch < 2 else "resident"
            out[op]["coded"] = coded
    out["speedup_stencil_vs_dia"] = round(out["dia"]["iter_loop_ms"] / out["stencil"]["iter_loop_ms"], 2)
    del sm
    torch.cuda.empty_cache()
    return out


def bench_small(pbgpu, torch, synth, dev, reps=5):
    """Small grids (the served requests' range), FP32 to 1e-6: the fused
    kernel (one grid barrier and one reduction of all its sums per iteration,
    one launch per solve) against the DIA form (the listing's two reductions
    per iteration in separate kernels, host-driven): wall time per solve and
    per iteration."""
    out = {}
    for n, natoms in ((33, 40), (49, 120), (65, 300), (97, 900)):
        p = synth.small_problem(n, n, n, natoms, seed=900 + n, precision="f32", tol=1e-6)
        g = p.grid
        sm = pbgpu.setup(g, p.mol.xyz, p.mol.radius, p.mol.charge, p.eps_in, p.eps_out, p.kappa_d2, device=dev)
        row = {}
        for op in ("stencil", "dia"):
            pbgpu.solve(sm, tol=1e-6, precision="f32", op=op)
            best = None
            for _ in range(reps):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                _, info = pbgpu.solve(sm, tol=1e-6, precision="f32", op=op)
                torch.cuda.synchronize()
                dt = time.perf_counter() - t0
                if best is None or dt < best[0]:
                    best = (dt, info)
            dt, info = best
            row[op] = {"iters": info["iters"], "solve_ms": round(1e3 * dt, 3),
                       "us_per_iter_wall": round(1e6 * dt / max(info["iters"], 1), 2)}
        row["speedup_fused_vs_dia"] = round(row["dia"]["solve_ms"] / row["stencil"]["solve_ms"], 2)
        out[f"{n}^3"] = row
        del sm
    torch.cuda.empty_cache()
    return out


def bench_slab(pbgpu, torch, synth, dev, iters=200):
    """One GPU's share of an 8-way z-slab split of the 257^3 solve: the fused
    kernel alone on 257 x 257 x 33 nodes (the halo exchange and the all-reduce
    of a multi-GPU run are not part of it), FP32, a fixed iteration count."""
    p = synth.small_problem(257, 257, 33, 400, seed=11, precision="f32")
    g = p.grid
    sm = pbgpu.setup(g, p.mol.xyz, p.mol.radius, p.mol.charge, p.eps_in, p.eps_out, p.kappa_d2, device=dev)
    n = g.nx * g.ny * g.nz
    tun = pbgpu.autotune(sm, precision="f32", iters_per_trial=20)   # untimed: this shape's tiling
    best = None
    for _ in range(3):
        _, info = pbgpu.solve(sm, tol=1e-300, precision="f32", maxiter=iters, check=False)
        if best is None or info["kernel_seconds"] < best["kernel_seconds"]:
            best = info
    us = 1e6 * best["kernel_seconds"] / best["iters"]
    del sm
    torch.cuda.empty_cache()
    return {"grid": [g.nx, g.ny, g.nz], "iters": best["iters"], "us_per_iter": round(us, 2),
            "algorithmic_gbs": round(ITER_BYTES * n / us / 1e3, 1),
            "form_bytes_per_node_iter": form_bytes(tun["scheme"], best["coded_launches"] > 0), "tuning": tun}


def bench_solvation(pbgpu, torch, synth, dev, reps=2):
    """Solvation energy dG from two solves (solvent vs uniform eps_in) of the
    257^3 config-2 system, FP32 inner / FP64 refinement to 1e-9; and the Born
    ion (a = 2.1 A, 33^3, h = 0.5) against Born's formula."""
    import numpy as np
    p = synth.config2()
    best = None
    for _ in range(reps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        r = pbgpu.solvation_energy(p.grid, p.mol.xyz, p.mol.radius, p.mol.charge, p.eps_in, p.eps_out,
                                   p.kappa_d2, tol=1e-9, precision="f32_refine64", inner_tol=1e-4, device=dev)
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        if best is None or dt < best[0]:
            best = (dt, r)
    dt, r = best
    # the same two solves preconditioned by the multigrid V-cycle
    best_mg = None
    for _ in range(reps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        rm = pbgpu.solvation_energy(p.grid, p.mol.xyz, p.mol.radius, p.mol.charge, p.eps_in, p.eps_out,
                                    p.kappa_d2, tol=1e-9, precision="f32_refine64", inner_tol=1e-4, op="mg",
                                    device=dev)
        torch.cuda.synchronize()
        dtm = time.perf_counter() - t0
        if best_mg is None or dtm < best_mg[0]:
            best_mg = (dtm, rm)
    dtm, rm = best_mg
    n, h, a = 33, 0.5, 2.1
    g = pbgpu.make_grid(n, n, n, h, np.full(3, -(n - 1) / 2 * h))
    born = pbgpu.solvation_energy(g, np.zeros((1, 3)), np.array([a]), np.array([1.0]), 1.0, 80.0, 0.0,
                                  tol=1e-10, precision="f64", device=dev)
    born_exact = -0.5 * 332.0637133 * (1.0 - 1.0 / 80.0) / a
    torch.cuda.empty_cache()
    return {"dG_kcal": round(r["dG"], 4), "ms": round(1e3 * dt, 2),
            "iters": [r["info_solv"]["iters"], r["info_ref"]["iters"]],
            "relres_true": [r["info_solv"]["relres_true"], r["info_ref"]["relres_true"]],
            "multigrid": {"dG_kcal": round(rm["dG"], 4), "ms": round(1e3 * dtm, 2),
                          "iters": [rm["info_solv"]["iters"], rm["info_ref"]["iters"]],
                          "relres_true": [rm["info_solv"]["relres_true"], rm["info_ref"]["relres_true"]],
                          "dG_rel_diff_vs_jacobi": abs(rm["dG"] - r["dG"]) / abs(r["dG"]),
                          "speedup": round(dt / dtm, 2)},
            "born_ion_dG_kcal": round(born["dG"], 5), "born_formula_kcal": round(born_exact, 5),
            "born_rel_err": round(born["dG"] / born_exact - 1.0, 5)}


def bench_periodic(pbgpu, torch, synth, dev, reps=3):
    """Periodic boundary: the config-2 molecule in a 257^3 periodic box with
    salt, FP32 Jacobi-PCG to 1e-6, in both pass forms: the 40-byte pass on
    ghost-row copies (coded; the default) and the pass that stores A.p."""
    p = synth.config2()
    g = p.grid
    sm = pbgpu.setup(g, p.mol.xyz, p.mol.radius, p.mol.charge, p.eps_in, p.eps_out, p.kappa_d2, device=dev,
                     boundary="periodic")
    n = g.nx * g.ny * g.nz
    out, xs = {}, {}
    try:
        for form, name, scheme in ((1, "pass40", 1), (0, "pass48", 0)):
            pbgpu.set_periodic_pass(form)
            pbgpu.solve(sm, tol=1e-6, precision="f32")
            best = None
            for _ in range(reps):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                x, info = pbgpu.solve(sm, tol=1e-6, precision="f32")
                torch.cuda.synchronize()
                dt = time.perf_counter() - t0
                if best is None or dt < best[0]:
                    best = (dt, info)
            dt, info = best
            xs[name] = x
            us = 1e6 * info["kernel_seconds"] / max(info["iters"], 1)
            coded = info["coded_launches"] > 0
            out[name] = {"iters": info["iters"], "solve_ms": round(1e3 * dt, 3), "us_per_iter": round(us, 2),
                         "coded": coded, "algorithmic_gbs": round(ITER_BYTES * n / us / 1e3, 1),
                         "form_gbs": round(form_bytes(scheme, coded) * n / us / 1e3, 1),
                         "relres_true": info["relres_true"]}
    finally:
        pbgpu.set_periodic_pass(-1)
    out["phi_rel_diff_forms"] = float((xs["pass40"] - xs["pass48"]).abs().max() / xs["pass48"].abs().max())
    del sm, xs
    torch.cuda.empty_cache()
    return out


def bench_mg(pbgpu, torch, synth, dev, reps=3):
    """Config 2 solves with the multigrid-preconditioned CG against the fused
    Jacobi-PCG (same system, same tolerances), best of `reps`."""
    p = synth.config2()
    g = p.grid
    sm = pbgpu.setup(g, p.mol.xyz, p.mol.radius, p.mol.charge, p.eps_in, p.eps_out, p.kappa_d2, device=dev)
    out = {}
    for prec, tol in (("f32", 1e-6), ("f32_refine64", 1e-9)):
        row = {}
        for op in ("stencil", "mg"):
            best = None
            for _ in range(reps):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                _, info = pbgpu.solve(sm, tol=tol, precision=prec, op=op,
                                      inner_tol=1e-4 if prec == "f32_refine64" else 0.0)
                torch.cuda.synchronize()
                dt = time.perf_counter() - t0
                if best is None or dt < best[0]:
                    best = (dt, info)
            dt, info = best
            row[op] = {"iters": info["iters"], "outer": info["outer_iters"], "solve_ms": round(1e3 * dt, 2),
                       "relres_true": info["relres_true"]}
        row["speedup_mg"] = round(row["stencil"]["solve_ms"] / row["mg"]["solve_ms"], 2)
        out[f"{prec}_tol{tol:g}"] = row
    del sm
    torch.cuda.empty_cache()
    return out


def bench_batched(pbgpu, torch, synth, dev, nsnap=256, seq_sample=24):
    """Config 3: snapshots on {65,97,129,161}^3 grids solved to 1e-6 in FP32 in one
    persistent launch (and replayed from a HIP graph), against plain per-snapshot
    fused solves on a sample. The batch kernel's z-chunk is first autotuned on
    this batch (untimed)."""
    probs = synth.config3(nsnap)
    systems = [pbgpu.setup(p.grid, p.mol.xyz, p.mol.radius, p.mol.charge, p.eps_in, p.eps_out, p.kappa_d2,
                           device=dev) for p in probs]
    torch.cuda.synchronize()
    z_prev = pbgpu.get_batch_zchunk()
    tuned = pbgpu.batch_autotune(systems, precision="f32", iters_per_trial=20)   # untimed: the batch's z-chunk
    pbgpu.solve_batch(systems[:8], tol=1e-6, precision="f32")          # warm-up (code, allocator)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    xs, infos = pbgpu.solve_batch(systems, tol=1e-6, precision="f32")
    torch.cuda.synchronize()
    t_batch = time.perf_counter() - t0
    nodes = [p.grid.nx * p.grid.ny * p.grid.nz for p in probs]
    bytes_ = sum(ITER_BYTES * n * i["iters"] for n, i in zip(nodes, infos))
    ok = sum(1 for i in infos if i["status"] == 0)
    worst = max(i["relres_true"] for i in infos)
    del xs
    g = pbgpu.BatchGraph(systems, tol=1e-6, precision="f32")
    g.launch()
    g.results()
    t0 = time.perf_counter()
    g.launch()
    ginfos = g.results()
    t_graph = time.perf_counter() - t0
    coop = g.cooperative
    g.close()
    del g
    # plain fused FP32 solves, one after another, on a sample
    t_seq, n_seq = 0.0, 0
    for sm in systems[:seq_sample]:
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        pbgpu.solve(sm, tol=1e-6, precision="f32")
        torch.cuda.synchronize()
        t_seq += time.perf_counter() - t0
        n_seq += 1
    del systems
    torch.cuda.empty_cache()
    pbgpu.set_batch_zchunk(z_prev)   # the served form keeps its own (latency-oriented) setting
    return {"snapshots": nsnap, "batch_zchunk": tuned["zchunk"], "converged": ok, "worst_relres_true": worst,
            "total_unknowns": sum(nodes), "iters_mean": sum(i["iters"] for i in infos) / nsnap,
            "batch_s": round(t_batch, 4), "snapshots_per_s": round(nsnap / t_batch, 2),
            "batch_gbs": round(bytes_ / t_batch / 1e9, 1),
            "graph_s": round(t_graph, 4), "graph_snapshots_per_s": round(nsnap / t_graph, 2),
            "graph_cooperative": coop,
            "plain_fused_sequential_snapshots_per_s": round(n_seq / t_seq, 2),
            "plain_fused_sample": n_seq}


def bench_serving(pbgpu, torch, synth, dev, nreq=2200, warm=200, rate=200.0, chunk=32, arena_gb=64,
                  seq_sample=48):
    """Config 4: a seeded Poisson trace of PB requests (atom counts
    log-uniform 500-30,000, grids 49^3-193^3, tol 1e-4/1e-6/1e-8) served by
    the continuous-batching server. Every request is its own molecule (one of
    64 config-4 chains with its atoms moved by seeded 0.3 A noise) handed over
    as atoms, radii and charges: the server runs the setup at admission and
    the energy at completion, so latency = completion - arrival covers setup,
    solve and energy. Atom arrays are resident on the device before the trace."""
    import numpy as np
    reqs = [synth.config4_molecule(i) for i in range(nreq)]
    dev_atoms = [tuple(torch.as_tensor(a, dtype=torch.float64, device=dev).contiguous()
                       for a in (p.mol.xyz.reshape(-1), p.mol.radius, p.mol.charge)) for p in reqs]
    outs = {}
    torch.cuda.synchronize()

    def out_for(p):
        key = (p.grid.nx, p.grid.ny, p.grid.nz)
        if key not in outs:
            outs[key] = torch.empty((p.grid.nz, p.grid.ny, p.grid.nx), dtype=torch.float64, device=dev)
        return outs[key]

    def run(nr, rate_, seed):
        arrivals = synth.config4_arrivals(nr, rate=rate_, seed=seed)
        srv = pbgpu.Server(int(arena_gb * (1 << 30)), max_slots=96, device=dev, keep_outputs=False)
        done_at, submitted = {}, {}
        k = 0
        t0 = time.perf_counter()
        while len(done_at) < nr:
            now = time.perf_counter() - t0
            while k < nr and arrivals[k] <= now:
                p = reqs[k]
                xyz, rad, q = dev_atoms[k]
                # each request writes its own potential tensor (recycled per grid shape once reported)
                rid = srv.submit_atoms(p.grid, xyz, rad, q, p.eps_in, p.eps_out, p.kappa_d2, tol=p.tol,
                                       precision=p.precision,
                                       out=torch.empty((p.grid.nz, p.grid.ny, p.grid.nx), dtype=torch.float64,
                                                       device=dev))
                submitted[rid] = k
                k += 1
            st = srv.stats()
            if st["active"] == 0 and st["pending"] == 0:
                if k < nr:
                    time.sleep(max(0.0, min(arrivals[k] - (time.perf_counter() - t0), 0.01)))
                continue
            for rid, info in srv.step(chunk=chunk):
                done_at[submitted[rid]] = (time.perf_counter() - t0, info, srv.energies.pop(rid, None))
        span = time.perf_counter() - t0
        stats = srv.stats()
        srv.close()
        w0 = warm if nr > warm else 0
        lat = np.array([done_at[i][0] - arrivals[i] for i in range(w0, nr)])
        fin = np.array([done_at[i][0] for i in range(w0, nr)])
        okc = sum(1 for i in range(nr) if done_at[i][1]["status"] == 0)
        thr = len(lat) / max(fin.max() - min(arrivals[w0], fin.min()), 1e-9)
        return {"requests": nr, "offered_per_s": rate_, "solves_per_s": round(float(thr), 2),
                "p50_ms": round(1e3 * float(np.percentile(lat, 50)), 2),
                "p99_ms": round(1e3 * float(np.percentile(lat, 99)), 2),
                "converged": okc, "span_s": round(span, 3), "launches": stats["launches"],
                "device_s": round(stats["device_seconds"], 3),
                "energies_returned": sum(1 for i in range(nr) if done_at[i][2] is not None)}

    def one(i):   # one request alone: setup + fused solve + energy
        p = reqs[i]
        xyz, rad, q = dev_atoms[i]
        sysm = pbgpu.setup(p.grid, xyz, rad, q, p.eps_in, p.eps_out, p.kappa_d2, device=dev)
        x, _ = pbgpu.solve(sysm, tol=p.tol, precision=p.precision, out=out_for(p))
        pbgpu.energy(p.grid, xyz, q, x)
        torch.cuda.synchronize()

    def run_fifo(nr, rate_, seed):
        """The same arrival trace served one request at a time in arrival order."""
        arrivals = synth.config4_arrivals(nr, rate=rate_, seed=seed)
        done = np.zeros(nr)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for i in range(nr):
            wait = arrivals[i] - (time.perf_counter() - t0)
            if wait > 0:
                time.sleep(wait)
            one(i)
            done[i] = time.perf_counter() - t0
        w0 = warm if nr > warm else 0
        lat = done[w0:] - arrivals[w0:nr]
        thr = len(lat) / max(done[w0:].max() - min(arrivals[w0], done[w0:].min()), 1e-9)
        return {"requests": nr, "offered_per_s": rate_, "solves_per_s": round(float(thr), 2),
                "p50_ms": round(1e3 * float(np.percentile(lat, 50)), 2),
                "p99_ms": round(1e3 * float(np.percentile(lat, 99)), 2)}

    full = run(nreq, rate, 4999)
    # the same requests one at a time, back to back: the service time alone
    lat_seq = []
    for i in range(seq_sample):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        one(i)
        lat_seq.append(time.perf_counter() - t0)
    lat_seq = np.array(lat_seq)
    seq_rate = float(len(lat_seq) / lat_seq.sum())
    # latency under load, the server against a sequential FIFO server on the
    # same arrival traces: at 0.7x the server's saturated rate (beyond what
    # the sequential server can sustain) and at half the sequential rate
    light_rate = round(0.7 * full["solves_per_s"], 1)
    nl = max(400, nreq // 4)
    light = run(nl, light_rate, 5999)
    light["sequential_fifo"] = run_fifo(nl, light_rate, 5999)
    half_rate = round(0.5 * seq_rate, 1)
    half = run(nl, half_rate, 6999)
    half["sequential_fifo"] = run_fifo(nl, half_rate, 6999)
    del dev_atoms, outs
    torch.cuda.empty_cache()
    return {"trace": full, "at_0.7x_capacity": light, "at_0.5x_sequential_rate": half,
            "plain_fused_sequential": {"solves_per_s": round(seq_rate, 2),
                                       "p50_ms": round(1e3 * float(np.percentile(lat_seq, 50)), 2),
                                       "p99_ms": round(1e3 * float(np.percentile(lat_seq, 99)), 2),
                                       "sample": len(lat_seq)},
            "requests_from": "molecules: setup at admission and energy at completion inside each request",
            "chunk": chunk}


# Forms reported beside the main line (also runnable alone with --forms-only).
FORMS = {"c1": bench_c1, "small": bench_small, "mg": bench_mg, "f1_solvation": bench_solvation, "f2_periodic": bench_periodic,
         "slab": bench_slab, "batched": bench_batched, "served": bench_serving}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-forms", action="store_true",
                    help="skip the batched (config 3) and served (config 4) measurements")
    ap.add_argument("--tuning", default="",
                    help="block,groups,zchunk,grid,scheme[,streaming[,segments]]: use this tiling instead of "
                         "autotuning (profiled runs; streaming 1/0 = nontemporal/cached, default the shape's own; "
                         "segments = in-plane segments, default any)")
    ap.add_argument("--coded", type=int, default=1, choices=(0, 1),
                    help="coded-coefficient 40-byte pass (1, the library default) or the uncoded pass (0)")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="run one untimed 512 MiB device copy first (counter calibration under rocprofv3)")
    ap.add_argument("--forms-only", default="",
                    help="comma-separated forms to run alone, one JSON line each, without the main step "
                         "(profiling): " + ", ".join(sorted(FORMS)))
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py: the benchmark runs on one GPU only (asked for --gpus {args.gpus}); independent "
              "solves would shard across GPUs without communication, one process per GPU.", file=sys.stderr)
        sys.exit(2)

    import torch
    import paper_1704_02745_amd as pbgpu
    import synth

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    dev = "cuda:0"
    torch.cuda.set_device(0)
    pbgpu.set_coded_coefficients(bool(args.coded))
    if args.forms_only:
        for name in args.forms_only.split(","):
            print(json.dumps({"form": name, "result": FORMS[name](pbgpu, torch, synth, dev)}), flush=True)
        teardown(torch)
        return
    prob = synth.config2()
    g = prob.grid
    n = g.nx * g.ny * g.nz
    xyz = torch.as_tensor(prob.mol.xyz, dtype=torch.float64, device=dev).contiguous()
    rad = torch.as_tensor(prob.mol.radius, dtype=torch.float64, device=dev)
    chg = torch.as_tensor(prob.mol.charge, dtype=torch.float64, device=dev)
    wsb = pbgpu.solve_workspace_bytes(g.nx, g.ny, g.nz, "f32_refine64")
    ws = torch.empty(wsb, dtype=torch.uint8, device=dev)
    x = torch.empty((g.nz, g.ny, g.nx), dtype=torch.float64, device=dev)

    def step():
        t0 = time.perf_counter()
        sysm = pbgpu.setup(g, xyz, rad, chg, prob.eps_in, prob.eps_out, prob.kappa_d2, device=dev)
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        _, info = pbgpu.solve(sysm, tol=1e-9, precision="f32_refine64", inner_tol=1e-4,
                              workspace=ws, out=x)
        t2 = time.perf_counter()
        e = pbgpu.energy(g, xyz, chg, x)
        t3 = time.perf_counter()
        return sysm, info, e, (t1 - t0, t2 - t1, t3 - t2)

    print(f"bench: {prob.name} n={n} natoms={prob.mol.natoms} warmup={args.warmup} steps={args.steps}",
          file=sys.stderr, flush=True)
    if args.calibrate_copy:
        # 512 MiB read + 512 MiB written, three times: the runtime's copy, and
        # the library's own streaming kernel with cached and with nontemporal
        # accesses (the same 16-byte vector loads and stores as the fused pass)
        src = torch.ones(128 << 20, dtype=torch.float32, device=dev)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        pbgpu.stream_copy(src, dst, False)
        pbgpu.stream_copy(src, dst, True)
        torch.cuda.synchronize()
        del src, dst
    # untimed: pick the fused kernel's tiling for this grid shape
    if args.tuning:
        tv = [int(v) for v in args.tuning.split(",")]
        pbgpu.set_tuning(g.nx, g.ny, g.nz, "f32", *tv[:5], streaming=tv[5] if len(tv) > 5 else -1,
                         segments=tv[6] if len(tv) > 6 else 0)
        tuning = dict(pbgpu.get_tuning(g.nx, g.ny, g.nz, "f32"), us_per_iter=None, candidates=0)
    else:
        sys0 = pbgpu.setup(g, xyz, rad, chg, prob.eps_in, prob.eps_out, prob.kappa_d2, device=dev)
        tuning = pbgpu.autotune(sys0, precision="f32", iters_per_trial=20, workspace=ws)
        del sys0
    print(f"bench: tuning {tuning}", file=sys.stderr, flush=True)
    scheme = tuning["scheme"] % 2   # (257^3 does not fit the resident form)
    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    infos, phases = [], []
    t0 = time.perf_counter()
    for _ in range(args.steps):
        sysm, info, e, ph = step()
        infos.append(info)
        phases.append(ph)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    print(f"bench: timed {args.steps} steps in {wall:.3f} s", file=sys.stderr, flush=True)

    iters = sum(i["iters"] for i in infos)
    launches = sum(i["kernel_launches"] for i in infos)
    coded_launches = sum(i["coded_launches"] for i in infos)
    coded = coded_launches == launches and launches > 0
    fbytes = form_bytes(scheme, coded)
    ksec = sum(i["kernel_seconds"] for i in infos)
    total_bytes = launch_bytes(n, iters, launches)
    value = total_bytes / wall / 1e9
    achieved = total_bytes / ksec / 1e9
    traffic = measured_traffic()
    ceiling = copy_ceiling(torch, dev)   # untimed, after the timed steps
    nt_ceiling = stream_ceiling(pbgpu, torch, dev, nontemporal=True)
    cached_ceiling = stream_ceiling(pbgpu, torch, dev, nontemporal=False)
    form_achieved = float(n) * (fbytes * iters + INIT_BYTES * launches) / ksec / 1e9
    roofline = {"bound": "hbm", "achieved": round(achieved, 1), "peak": PEAK_GBS, "unit": "GB/s",
                "frac": round(achieved / PEAK_GBS, 4),
                "basis": f"{ITER_BYTES} B/unknown/iteration: the floor of any schedule that stores the operator as "
                         f"four FP32 arrays (x, r, p read and written, four coefficient arrays read once), "
                         f"whichever pass form runs",
                "form_achieved": round(form_achieved, 1),
                "form_frac": round(form_achieved / PEAK_GBS, 4),
                "traffic": None if traffic is None else round(traffic, 0),
                "kernel": f"k_jpcg_fused<float, {tuning['block']}, {tuning['groups']}, {scheme}, false, "
                          f"{'true' if tuning.get('streaming') else 'false'}, {'true' if coded else 'false'}> "
                          f"(persistent, one launch per inner solve; algorithmic {ITER_BYTES} B/unknown/iteration "
                          f"with the four operator arrays at 4 B each, this pass form moves {fbytes} B"
                          f"{' reading the operator as one 4-byte code word' if coded else ''})",
                "form_bytes_per_unknown_iter": fbytes,
                "form_gbs": round(float(n) * fbytes * iters / ksec / 1e9, 1),
                "bytes_per_launch": round(total_bytes / launches, 0),
                "avg_launch_ms": round(1e3 * ksec / launches, 4),
                "copy_ceiling_gbs": ceiling,
                "stream_ceiling_nt_gbs": nt_ceiling,
                "stream_ceiling_cached_gbs": cached_ceiling}
    if traffic is not None:   # counted HBM bytes per launch over the live launch time
        roofline["traffic_gbs"] = round(traffic / (ksec / launches) / 1e9, 1)
        roofline["traffic_frac"] = round(roofline["traffic_gbs"] / PEAK_GBS, 4)
        roofline["traffic_vs_stream_ceiling"] = round(roofline["traffic_gbs"] / max(nt_ceiling, cached_ceiling), 4)

    forms = {}
    if not args.no_forms:
        print("bench: config 1 (129^3 stencil vs DIA)", file=sys.stderr, flush=True)
        forms["c1_129_stencil_vs_dia"] = bench_c1(pbgpu, torch, synth, dev)
        print(f"bench: {forms['c1_129_stencil_vs_dia']}", file=sys.stderr, flush=True)
        print("bench: small grids, fused single-reduction vs DIA", file=sys.stderr, flush=True)
        forms["small_grids_fused_vs_dia"] = bench_small(pbgpu, torch, synth, dev)
        print(f"bench: {forms['small_grids_fused_vs_dia']}", file=sys.stderr, flush=True)
        print("bench: multigrid-preconditioned CG (config 2)", file=sys.stderr, flush=True)
        forms["c2_multigrid_vs_jacobi"] = bench_mg(pbgpu, torch, synth, dev)
        print(f"bench: {forms['c2_multigrid_vs_jacobi']}", file=sys.stderr, flush=True)
        print("bench: solvation energy (config 2 molecule)", file=sys.stderr, flush=True)
        forms["f1_solvation"] = bench_solvation(pbgpu, torch, synth, dev)
        print(f"bench: {forms['f1_solvation']}", file=sys.stderr, flush=True)
        print("bench: periodic boundary (config 2 molecule)", file=sys.stderr, flush=True)
        forms["f2_periodic_257"] = bench_periodic(pbgpu, torch, synth, dev)
        print(f"bench: {forms['f2_periodic_257']}", file=sys.stderr, flush=True)
        print("bench: 257x257x33 slab", file=sys.stderr, flush=True)
        forms["slab_257x257x33"] = bench_slab(pbgpu, torch, synth, dev)
        print(f"bench: {forms['slab_257x257x33']}", file=sys.stderr, flush=True)
        print("bench: batched form (config 3)", file=sys.stderr, flush=True)
        forms["batched"] = bench_batched(pbgpu, torch, synth, dev)
        print(f"bench: {forms['batched']}", file=sys.stderr, flush=True)
        print("bench: served form (config 4)", file=sys.stderr, flush=True)
        forms["served"] = bench_serving(pbgpu, torch, synth, dev)
        print(f"bench: {forms['served']}", file=sys.stderr, flush=True)

    cpu = None
    if not args.no_cpu_baseline:
        print("bench: timing the CPU oracle sample", file=sys.stderr, flush=True)
        cpu = cpu_baseline(prob)

    # accuracy of the last step, checked by the oracle's own FP64 operator
    from oracle import fdpb
    s = fdpb.System(h=g.h, eps_x=sysm.eps_x.cpu().numpy(), eps_y=sysm.eps_y.cpu().numpy(),
                    eps_z=sysm.eps_z.cpu().numpy(), kappa2=sysm.kappa2.cpu().numpy(),
                    b=sysm.rhs.cpu().numpy())
    xs = x.cpu().numpy()
    relres_oracle = fdpb.true_relres(s, xs)
    e_oracle = fdpb.energy(g.nx, g.ny, g.nz, g.h, g.origin, prob.mol.xyz, prob.mol.charge, xs)

    last = infos[-1]
    gold = oracle_golden_errors(x, e)
    out = {
        "metric": METRIC, "value": round(value, 1), "unit": "GB/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(1e3 * wall / args.steps, 3),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32+f64", "data": "synthetic",
        "config": {"workload": "257^3 grid (16,974,593 unknowns), h=0.5 A, 20,000-atom seeded "
                               "random-walk globule (R=51.7 A); setup + FP32 JPCG inner 1e-4 inside "
                               "FP64 refinement to 1e-9 + energy",
                   "grid": [g.nx, g.ny, g.nz], "natoms": prob.mol.natoms, "tol": 1e-9,
                   "inner_tol": 1e-4,
                   "value_basis": f"effective GB/s: {ITER_BYTES} B/unknown/iteration of the fused launches (the "
                                  f"four-array floor) over the wall time of the timed steps; the pass form that "
                                  f"runs moves {fbytes} B (roofline.form_achieved), counted HBM traffic in "
                                  f"roofline.traffic_gbs"},
        "roofline": roofline,
        "cpu_baseline": cpu,
        "detail": {
            "iters_per_step": iters / args.steps, "outer_per_step": last["outer_iters"],
            "launches_per_step": launches / args.steps,
            "setup_ms": round(1e3 * sum(p[0] for p in phases) / len(phases), 3),
            "solve_ms": round(1e3 * sum(p[1] for p in phases) / len(phases), 3),
            "energy_ms": round(1e3 * sum(p[2] for p in phases) / len(phases), 3),
            "jpcg_kernel_ms_per_step": round(1e3 * ksec / args.steps, 3),
            "jpcg_iters_per_s": round(iters / ksec, 1),
            "jpcg_iter_us": round(1e6 * ksec / iters, 2),
            "pass_form": scheme, "coded_coefficients": coded, "coded_launches_per_step": coded_launches / args.steps,
            "pass_form_bytes_per_unknown_iter": fbytes,
            "pass_form_gbs": round(float(n) * fbytes * iters / ksec / 1e9, 1),
            "relres_true_gpu": last["relres_true"], "relres_true_oracle": relres_oracle,
            "energy_kcal": e, "energy_oracle_of_gpu_phi": e_oracle,
            "vs_oracle_solution": gold,
            "solves_per_s": round(args.steps / wall, 3),
            "tuning": tuning,
        },
        "forms": forms,
    }
    print(json.dumps(out), flush=True)
    # release every device object before the interpreter exits, so that no
    # HIP call runs from exit handlers (profilers tear down before those)
    del sysm, ws, x, xyz, rad, chg
    teardown(torch)


def teardown(torch):
    import gc
    gc.collect()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


if __name__ == "__main__":
    main()
