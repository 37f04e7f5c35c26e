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


def molecule_system(pb, dims, natoms, seed, boundary="free"):
    import synth
    p = synth.small_problem(*dims, natoms, seed=seed, precision="f32")
    return pb.setup(p.grid, p.mol.xyz, p.mol.radius, p.mol.charge, p.eps_in, p.eps_out, p.kappa_d2, device=DEV,
                    boundary=boundary)


def streaming(pb, sysm, **kw):
    """The solve in the streaming form, the shape's choice of form left as it was."""
    dims = sysm.dims
    if sysm.grid.boundary:
        pb.set_periodic_pass(1)
        try:
            return pb.solve(sysm, **kw)
        finally:
            pb.set_periodic_pass(-1)
    c = [c for c in pb.tiling_candidates(*dims, "f32") if c["scheme"] == 1][0]
    pb.set_tuning(*dims, "f32", c["block"], c["groups"], c["zchunk"], c["grid"], c["scheme"], c["streaming"],
                  c["segments"])
    try:
        return pb.solve(sysm, **kw)
    finally:
        pb.autotune(sysm, precision="f32", iters_per_trial=2)


# every number of planes per brick of the FP32 kernels, full (2 to 19) and compact (24 to 43), is the
# default of some of these
@pytest.mark.parametrize("dims", [(33, 29, 31), (45, 41, 47), (65, 57, 61), (81, 77, 83), (97, 105, 89),
                                  (117, 117, 113), (133, 129, 133), (139, 141, 137), (153, 150, 155), (169, 171, 165)])
@pytest.mark.parametrize("boundary", ["free", "periodic"])
def test_resident_sizes(pb, dims, boundary):
    sysm = molecule_system(pb, dims, max(20, int(1e-3 * dims[0] ** 3) // 8), sum(dims), boundary)
    print(f"resident sizes {dims} {boundary}", flush=True)
    x1, i1 = pb.solve(sysm, tol=1e-6, precision="f32")
    xw, iw = pb.solve(sysm, tol=1e-6, precision="f32", x0=0.9 * x1)
    xr, ir = pb.solve(sysm, tol=1e-9, precision="f32_refine64")
    x0, i0 = streaming(pb, sysm, tol=1e-6, precision="f32")
    scale = float(x0.abs().max())
    assert i1["status"] == iw["status"] == ir["status"] == pb.PB_OK
    assert abs(i1["iters"] - i0["iters"]) <= max(2, 0.02 * i0["iters"]) and iw["iters"] < i1["iters"]
    assert float((x1 - x0).abs().max()) <= 1e-5 * scale
    assert float((xw - x0).abs().max()) <= 1e-5 * scale
    assert float((xr - x0).abs().max()) <= 1e-5 * scale and ir["relres_true"] < 1e-9


def test_batch_of_every_form(pb):
    """Full and compact resident problems and one that only streams, in one batch:
    each bitwise as alone; recorded, a compact problem whose operator stops
    fitting the dictionary runs uncoded and the others as before."""
    shapes = [(139, 141, 137), (49, 45, 41), (96, 97, 95), (201, 193, 189)]
    systems = [molecule_system(pb, s, 200, 900 + i) for i, s in enumerate(shapes)]
    xs, infos = pb.solve_batch(systems, tol=1e-6, precision="f32")
    assert all(i["status"] == pb.PB_OK and i["coded_launches"] == 1 for i in infos), infos
    for k, s in enumerate(systems):
        x, i = pb.solve_batch([s], tol=1e-6, precision="f32")
        assert torch.equal(x[0], xs[k]) and i[0]["iters"] == infos[k]["iters"], k
        y, _ = pb.solve(s, tol=1e-6, precision="f32")
        assert float((y - xs[k]).abs().max()) <= 1e-5 * float(y.abs().max()), k
    g = pb.BatchGraph(systems, tol=1e-6, precision="f32")
    try:
        for _ in range(3):
            g.launch()
            i1 = g.results()
            assert [i["coded_launches"] for i in i1] == [1] * 4
            assert all(torch.equal(g.outs[j], xs[j]) for j in range(4))
            torch.zeros(1 << 20, device=DEV).add_(1.0)
        saved = systems[0].eps_x.clone()
        systems[0].eps_x.copy_(torch.as_tensor(np.random.default_rng(5).uniform(1, 80, tuple(saved.shape)), device=DEV))
        g.launch()
        i2 = g.results()
        assert [i["coded_launches"] for i in i2] == [0, 1, 1, 1] and all(i["status"] == pb.PB_OK for i in i2)
        xd, _ = pb.solve_batch(systems, tol=1e-6, precision="f32")
        assert torch.equal(g.outs[0], xd[0]) and all(torch.equal(g.outs[j], xs[j]) for j in range(1, 4))
        systems[0].eps_x.copy_(saved)
        g.launch()
        g.results()
        assert all(torch.equal(g.outs[j], xs[j]) for j in range(4))
    finally:
        g.close()


@pytest.mark.parametrize("chunk", [1, 7, 100000])
def test_served_chunks(pb, chunk):
    """Served requests of the full and the compact form and one in passes, warm starts among them,
    stopped and resumed after `chunk` iterations (or a few times as many): each bitwise the batch of
    that request alone, which runs through in one launch."""
    shapes = [(45, 41, 47), (97, 89, 93), (139, 141, 137), (141, 131, 149)]
    systems = [molecule_system(pb, s, 150, 700 + i) for i, s in enumerate(shapes)]
    if chunk > 1:
        systems.append(molecule_system(pb, (201, 193, 189), 200, 711))
    want = [pb.solve_batch([s], tol=1e-5, precision="f32")[0][0] for s in systems]
    guess = [0.9 * w if k % 2 else None for k, w in enumerate(want)]
    batch = [pb.solve_batch([s], tol=1e-5, precision="f32", x0s=[g] if g is not None else None)
             for s, g in zip(systems, guess)]
    srv = pb.Server(sum(pb.Server.request_bytes(s) for s in systems) + (64 << 20), max_slots=8, device=DEV)
    try:
        ids = {srv.submit(s, tol=1e-5, precision="f32", x0=g): k for k, (s, g) in enumerate(zip(systems, guess))}
        out = {}
        for _ in range(5000):
            for rid, info in srv.step(chunk=chunk):
                out[ids[rid]] = (srv.outputs[rid].clone(), info)
            if len(out) == len(systems):
                break
    finally:
        srv.close()
    assert len(out) == len(systems)
    for k, (x, info) in out.items():
        xb, ib = batch[k]
        assert info["status"] == pb.PB_OK, k
        if shapes[k:k + 1]:   # (the pass form's tiles differ between server and batch)
            assert info["iters"] == ib[0]["iters"] and torch.equal(x, xb[0]), k
        else:
            assert float((x - xb[0]).abs().max()) <= 1e-5 * float(x.abs().max()), k
