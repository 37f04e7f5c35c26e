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
