"""The resident form of the fused solve (whole iteration state in registers and
LDS) against the oracle and the streaming form.

A solve takes it by default where the grid's bricks fit the device; a tiling
recorded with set_tuning asks for the streaming form. Both run the same
iteration with the same operations per node and differ by the order of their
FP64 sums alone, so the FP64 potentials of one iteration count agree to FP64
rounding amplified over the iterations (1e-11 of max |phi|), the FP32 ones to
the bars of every FP32 solve (1e-5), and the iteration counts within max(2, 2%).

Shapes: one brick; bricks whose last one along an axis is narrower; a last
chunk of one plane; one brick along x, along y, along z; grids that fill more
than 200 workgroups; the widest that fit.
"""
import numpy as np
import pytest
import torch

from oracle import fdpb, pcg, periodic

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SHAPES = [(7, 5, 3), (16, 16, 4), (17, 31, 33), (130, 3, 9), (3, 130, 9), (9, 3, 130), (48, 41, 37), (61, 53, 47),
          (96, 7, 90)]


@pytest.fixture(scope="module")
def pb():
    import paper_1704_02745_amd as m
    return m


def rand_arrays(nx, ny, nz, seed, wrap):
    rng = np.random.default_rng(seed)
    a = {"eps_x": rng.uniform(1, 80, (nz, ny, nx + 1)), "eps_y": rng.uniform(1, 80, (nz, ny + 1, nx)),
         "eps_z": rng.uniform(1, 80, (nz + 1, ny, nx)), "kappa2": rng.uniform(0, 2, (nz, ny, nx)),
         "b": rng.standard_normal((nz, ny, nx))}
    if wrap:
        a["eps_x"][:, :, -1] = a["eps_x"][:, :, 0]
        a["eps_y"][:, -1] = a["eps_y"][:, 0]
        a["eps_z"][-1] = a["eps_z"][0]
    return a


def to_system(pb, dims, a, boundary):
    t = lambda v: torch.as_tensor(np.ascontiguousarray(v), dtype=torch.float64, device=DEV)
    return pb.System(pb.make_grid(*dims, 0.5, (0.0, 0.0, 0.0), boundary), t(a["eps_x"]), t(a["eps_y"]), t(a["eps_z"]),
                     t(a["kappa2"]), t(a["b"]))


@pytest.mark.parametrize("boundary", ["free", "periodic"])
@pytest.mark.parametrize("dims", SHAPES)
def test_resident_against_oracle(pb, dims, boundary):
    a = rand_arrays(*dims, seed=sum(dims), wrap=boundary == "periodic")
    sysm = to_system(pb, dims, a, boundary)
    if boundary == "free":
        o = pcg.jpcg(fdpb.System(h=0.5, **a), 1e-8, maxiter=5000)
        exact = pcg.jpcg(fdpb.System(h=0.5, **a), 1e-13, maxiter=5000).x
    else:
        ps = fdpb.System(h=0.5, **a)
        o = periodic.jpcg(ps, 1e-8, maxiter=5000)
        exact = periodic.jpcg(ps, 1e-13, maxiter=5000).x
    scale = np.abs(exact).max()
    for prec, tol, bound in (("f64", 1e-8, 1e-7), ("f32", 1e-6, 1e-5), ("f32_refine64", 1e-10, 1e-9)):
        print(f"resident {dims} {boundary} {prec}", flush=True)
        x, info = pb.solve(sysm, tol=tol, precision=prec, maxiter=5000)
        assert info["status"] == pb.PB_OK
        assert np.abs(x.cpu().numpy() - exact).max() <= bound * scale, prec
        if prec == "f64":
            assert abs(info["iters"] - o.iters) <= max(2, 0.02 * o.iters)
            # from a guess: the same solution, and no iteration from the solution itself
            x0 = torch.as_tensor(0.9 * exact, device=DEV)
            xw, iw = pb.solve(sysm, tol=tol, precision=prec, maxiter=5000, x0=x0)
            assert iw["iters"] < info["iters"] and np.abs(xw.cpu().numpy() - exact).max() <= bound * scale
            xs, is_ = pb.solve(sysm, tol=tol, precision=prec, maxiter=5000, x0=torch.as_tensor(exact, device=DEV))
            assert is_["iters"] == 0 and torch.equal(xs.cpu(), torch.as_tensor(exact))


@pytest.mark.parametrize("prec,bound", [("f64", 1e-11), ("f32", 1e-5)])
def test_resident_against_streaming(pb, prec, bound):
    """The same iterations in both forms; two runs of the resident one are
    bitwise equal; a limit of iterations stops both at the same iterate."""
    dims = (57, 50, 43)
    a = rand_arrays(*dims, seed=5, wrap=False)
    sysm = to_system(pb, dims, a, "free")
    x1, i1 = pb.solve(sysm, tol=1e-6, precision=prec)
    x2, i2 = pb.solve(sysm, tol=1e-6, precision=prec)
    xl, il = pb.solve(sysm, tol=1e-6, precision=prec, maxiter=7, check=False)
    zero, iz = pb.solve(to_system(pb, dims, dict(a, b=np.zeros_like(a["b"])), "free"), tol=1e-6, precision=prec)
    assert torch.equal(x1, x2) and i1["iters"] == i2["iters"]
    assert iz["iters"] == 0 and float(zero.abs().max()) == 0.0
    c = pb.tiling_candidates(*dims, prec)[0]
    try:
        pb.set_tuning(*dims, prec, c["block"], c["groups"], c["zchunk"], c["grid"], c["scheme"], c["streaming"],
                      c["segments"])
        x0, i0 = pb.solve(sysm, tol=1e-6, precision=prec)
        xm, im = pb.solve(sysm, tol=1e-6, precision=prec, maxiter=7, check=False)
    finally:
        pb.autotune(sysm, precision=prec, iters_per_trial=3)
    assert abs(i1["iters"] - i0["iters"]) <= max(2, 0.02 * i0["iters"])
    assert float((x1 - x0).abs().max()) <= bound * float(x0.abs().max())
    assert il["status"] == im["status"] == pb.PB_NOT_CONVERGED and il["iters"] == im["iters"] == 7
    assert float((xl - xm).abs().max()) <= bound * float(xm.abs().max())
