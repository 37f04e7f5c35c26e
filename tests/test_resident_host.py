"""Host parts of the resident form, their source text compiled with g++. No GPU involved."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1704_02745_amd", "csrc")


def extract(src, name):
    i = src.index(name)
    i = src.rfind("\n", 0, i) + 1
    return src[i:src.index("\n}\n", i) + 3]


def compile_and_run(tmp_path, text, stdin=""):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    (tmp_path / "t.cpp").write_text(text)
    r = subprocess.run(["g++", "-std=c++17", "-O1", str(tmp_path / "t.cpp"), "-o", str(tmp_path / "t")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(tmp_path / "t")], input=stdin, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    return r.stdout


def test_first_wait_covers_the_problems_before(tmp_path):
    """A workgroup's wait in a problem's first barrier is longer than the passes of every problem of the
    launch take at their iteration limits, and stays a positive number of ticks."""
    src = open(os.path.join(CSRC, "resident_impl.hpp")).read()
    cases = [(1, 300 * 7.0), (256, 256 * 1290 * 16.0), (2, 2 * 2_000_000 * 15.0), (3, 3 * 1e9 * 16.0),
             (4096, 4096 * 2147483647 * 20.0)]
    out = compile_and_run(tmp_path, "#include <cstdio>\n" + extract(src, "long long first_wait_ticks(") + r"""
int main() {
    int n;
    double us;
    while (std::scanf("%d %lf", &n, &us) == 2) std::printf("%lld\n", first_wait_ticks(2000000000LL, n, us, 100.0));
}
""", "\n".join(f"{n} {us!r}" for n, us in cases))
    got = [int(v) for v in out.split()]
    assert len(got) == len(cases)
    for (n, us), t in zip(cases, got):
        assert t >= min(2_000_000_000 * (n + 1) + us * 100.0, 3.9e18) and t <= 2 ** 62


# ---- the bricks that resident_plan chooses, on a device of 256 compute units

PLAN_DRIVER = r"""
#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <vector>
#define __host__
#define __device__
struct Layout { int nx, ny, nz; int64_t plane, sp, npad, n; };
struct ResPlan { int bs, nz, tx, ty, nxt, nyt, nzc, grid; size_t lds; const void* fn; double us; };
struct ResVariant { int bs, nz; const void* fn[2]; };
constexpr int kCodedTableSize = 256;
#include "plan.inc"
template <typename T> std::vector<ResVariant> variants();
#define PB_RES_VARIANT(T, BS, NZ) ResVariant { BS, NZ, {nullptr, nullptr} }
#define PB_RES_COMPACT(NZ) ResVariant { 512, NZ, {nullptr, nullptr} }
template <> std::vector<ResVariant> variants<float>() { return {F32_LIST}; }
template <> std::vector<ResVariant> variants<double>() { return {F64_LIST}; }
template <typename T> ResPlan plan(int nx, int ny, int nz, int per) {
    Layout L{nx, ny, nz};
    L.plane = (int64_t)nx * ny;
    L.sp = (L.plane + 63) / 64 * 64;
    L.npad = L.sp * nz;
    ResPlan best{};
    for (int compact = 0; compact < (sizeof(T) == 4 ? 2 : 1) && best.grid == 0; ++compact) {
        double best_cost = 1e300;
        for (const ResVariant& v : variants<T>())
            if (compact == (v.nz >= kCompactFrom))
                resident_search<T>(L, per, v.bs, v.nz, compact, 256, 5 * L.npad / 2, nullptr,
                                   [](double us, int) { return us; }, best_cost, best);
    }
    return best;
}
int main() {
    int nx, ny, nz, per, wide;
    while (std::scanf("%d %d %d %d %d", &nx, &ny, &nz, &per, &wide) == 5) {
        const ResPlan p = wide ? plan<double>(nx, ny, nz, per) : plan<float>(nx, ny, nz, per);
        std::printf("%d %d %d\n", p.bs, p.nz, p.grid);
    }
}
"""


def _listed(name):
    src = open(os.path.join(CSRC, name)).read()
    body = src[src.index("v = {") + 5:]
    return body[:body.index("};")]


def plans(tmp_path, cases):
    dev = open(os.path.join(CSRC, "resident_device.hpp")).read()
    impl = open(os.path.join(CSRC, "resident_impl.hpp")).read()

    def line(name):
        i = dev.index(name)
        return dev[i:dev.index("\n", i) + 1]

    i = dev.index("template <typename T>\n__host__ __device__ constexpr bool lower_in_lds")
    j = dev.index("\n", dev.index("lower_in_lds(int bs, int nzb)")) + 1
    text = (line("constexpr int kMaxResidentGroups") + line("constexpr int kSlotGroup =") +
            extract(dev, "constexpr int slot_groups(") + line("__host__ __device__ constexpr int face_len(") +
            dev[i:j] + "template <typename T>\n" + extract(dev, "constexpr bool x_in_memory(") +
            "template <typename T>\n" + extract(dev, "constexpr size_t resident_lds_bytes(") +
            line("constexpr int kCompactFrom") + extract(impl, "double resident_pass_us(") +
            "template <typename T, typename Cost>\n" + extract(impl, "void resident_search("))
    (tmp_path / "plan.inc").write_text(text)
    driver = PLAN_DRIVER.replace("F32_LIST", _listed("resident_f32.hip")).replace("F64_LIST",
                                                                                 _listed("resident_f64.hip"))
    out = compile_and_run(tmp_path, driver, "\n".join(
        f"{d[0]} {d[1]} {d[2]} {int(b == 'periodic')} {int(p == 'f64')}" for d, b, p in cases))
    return [tuple(int(v) for v in r.split()) for r in out.strip().split("\n")]


def test_planes_shapes_reach_every_kernel(tmp_path):
    """The shapes of test_gpu_resident_planes.py (and of test_gpu_resident.py) run every number of planes
    that the single solves' kernels have, free and periodic, in both precisions."""
    import re

    import test_gpu_resident as base
    import test_gpu_resident_planes as more
    sizes = [m.args[1] for m in base.test_resident_sizes.pytestmark if m.args[0] == "dims"][0]
    cases = [(d, b, "f32") for d in sizes for b in ("free", "periodic")]
    cases += [(d, b, p) for d in base.SHAPES for b in ("free", "periodic") for p in ("f32", "f64")]
    cases += [(d, b, p) for p, d in more.SHAPES for b in ("free", "periodic")]
    got = plans(tmp_path, cases)
    # (7 x 5 x 3 periodic streams: the faces of its bricks do not fit the arrays they lie in)
    reached = {(b, p, bs, nz) for (d, b, p), (bs, nz, g) in zip(cases, got) if g > 0}
    for prec, name in (("f32", "resident_f32.hip"), ("f64", "resident_f64.hip")):
        text = _listed(name)
        kernels = {(int(a), int(b)) for a, b in re.findall(r"PB_RES_VARIANT\(\w+, (\d+), (\d+)\)", text)}
        kernels |= {(512, int(a)) for a in re.findall(r"PB_RES_COMPACT\((\d+)\)", text)}
        for b in ("free", "periodic"):
            missing = kernels - {(bs, nz) for bb, pp, bs, nz in reached if (bb, pp) == (b, prec)}
            assert not missing, (prec, b, missing)
