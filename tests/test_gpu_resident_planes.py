"""The resident kernels by planes per brick: single solves of every number of planes that
test_gpu_resident.py does not reach (test_resident_host.py checks on the host that together they reach
all), and the batch's and server's kernels with a last brick of one plane and of one plane less than a
whole one.

The streaming form runs the same iteration and differs by the order of the FP64 sums alone: after the
same 40 iterations, 1e-11 of max |phi| in FP64 and 1e-5 in FP32, the bars of test_gpu_resident.py."""
import pytest
import torch

import synth
from test_gpu_tuning_forms import form

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
BOUND = {"f64": 1e-11, "f32": 1e-5}
SHAPES = [("f64", (65, 63, 61)), ("f64", (73, 75, 71)), ("f64", (85, 81, 83)), ("f64", (97, 105, 89)),
          ("f64", (77, 79, 81)), ("f64", (101, 99, 97)), ("f32", (99, 101, 97)), ("f32", (107, 105, 109))]


@pytest.fixture(scope="module")
def pb():
    import paper_1704_02745_amd as m
    return m


def molecule_system(pb, dims, boundary="free", natoms=120):
    p = synth.small_problem(*dims, natoms, seed=sum(dims), precision="f32")
    return pb.setup(p.grid, p.mol.xyz, p.mol.radius, p.mol.charge, p.eps_in, p.eps_out, p.kappa_d2, device=DEV,
                    boundary=boundary)


def streaming(pb, sysm, prec, **kw):
    """The solve in the streaming form; what was recorded for the shape stays recorded."""
    dims = sysm.dims
    if sysm.grid.boundary:
        pb.set_periodic_pass(1)
        try:
            assert form(pb, sysm, precision=prec, **kw) == "fused"
            return pb.solve(sysm, precision=prec, **kw)
        finally:
            pb.set_periodic_pass(-1)
    was = pb.get_tuning(*dims, prec)
    c = [c for c in pb.tiling_candidates(*dims, prec) if c["scheme"] == 1][0]
    try:
        pb.set_tuning(*dims, prec, c["block"], c["groups"], c["zchunk"], c["grid"], c["scheme"], c["streaming"],
                      c["segments"])
        assert form(pb, sysm, precision=prec, **kw) == "fused"
        return pb.solve(sysm, precision=prec, **kw)
    finally:
        pb.set_tuning(*dims, prec, was["block"], was["groups"], was["zchunk"], was["grid"], was["scheme"],
                      was["streaming"], was["segments"])


@pytest.mark.parametrize("boundary", ["free", "periodic"])
@pytest.mark.parametrize("prec,dims", SHAPES)
def test_planes(pb, prec, dims, boundary):
    s = molecule_system(pb, dims, boundary)
    kw = dict(tol=1e-300, maxiter=40, check=False)
    print(f"planes {prec} {dims} {boundary}", flush=True)
    assert form(pb, s, precision=prec, **kw) == "resident"
    x1, i1 = pb.solve(s, precision=prec, **kw)
    x0, i0 = streaming(pb, s, prec, **kw)
    scale = float(x0.abs().max())
    assert i1["iters"] == i0["iters"] == 40
    assert float((x1 - x0).abs().max()) <= BOUND[prec] * scale
    guess = 0.7 * x0
    w1, j1 = pb.solve(s, precision=prec, x0=guess, **kw)
    w0, j0 = streaming(pb, s, prec, x0=guess, **kw)
    assert j1["iters"] == j0["iters"] == 40
    assert float((w1 - w0).abs().max()) <= BOUND[prec] * scale
    y, i = pb.solve(s, precision=prec, tol=1e-6)
    assert i["status"] == pb.PB_OK and i["relres_true"] <= 1e-5


# planes of the batch's and server's kernels: 19 (FP32, full), 43 (FP32, compact), 8 (FP64)
@pytest.mark.parametrize("prec,dims", [("f32", (40, 37, 20)), ("f32", (40, 37, 37)), ("f32", (150, 160, 130)),
                                       ("f32", (150, 160, 128)), ("f64", (40, 37, 33)), ("f64", (40, 37, 39))])
def test_partial_last_brick(pb, prec, dims):
    s = molecule_system(pb, dims)
    other = molecule_system(pb, (33, 31, 29))
    kw = dict(tol=1e-300, maxiter=40, check=False)
    print(f"last brick {prec} {dims}", flush=True)
    x0, _ = streaming(pb, s, prec, **kw)
    xs, infos = pb.solve_batch([other, s], precision=prec, **kw)
    assert infos[1]["iters"] == 40
    assert float((xs[1] - x0).abs().max()) <= BOUND[prec] * float(x0.abs().max())
    # the bricks of the last chunk hold the same potential as the others do: no plane is left out
    assert float((xs[1] - x0)[-1].abs().max()) <= BOUND[prec] * float(x0.abs().max()) and float(xs[1][-1].abs().max()) > 0
    if prec == "f64":
        return
    full, i = pb.solve_batch([s], precision=prec, tol=1e-5)
    srv = pb.Server(sum(pb.Server.request_bytes(v) for v in (s, other)) + (16 << 20), max_slots=4, device=DEV)
    try:
        ids = [srv.submit(other, tol=1e-4, precision="f32"), srv.submit(s, tol=1e-5, precision="f32")]
        out = {}
        for _ in range(2000):
            for rid, info in srv.step(chunk=3):
                out[rid] = (srv.outputs[rid].clone(), info)
            if len(out) == 2:
                break
    finally:
        srv.close()
    assert torch.equal(out[ids[1]][0], full[0]) and out[ids[1]][1]["iters"] == i[0]["iters"]
