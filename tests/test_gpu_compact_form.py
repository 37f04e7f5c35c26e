"""The compact resident form (FP32 grids of about 134 to 171 nodes an edge): its results do not depend
on pb_set_coded_coefficients, bit for bit, in a solve, a batch, a recorded batch and the server; and an
operator that does not fit a dictionary is put to the dictionary once per solve."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
DIMS = (139, 141, 137)


@pytest.fixture(scope="module")
def pb():
    import paper_1704_02745_amd as m
    m.set_coded_coefficients(True)
    yield m
    m.set_coded_coefficients(True)


def molecule_system(pb, boundary="free"):
    p = synth.small_problem(*DIMS, 200, seed=31, precision="f32")
    return pb.setup(p.grid, p.mol.xyz, p.mol.radius, p.mol.charge, p.eps_in, p.eps_out, p.kappa_d2, device=DEV,
                    boundary=boundary)


def graph_run(pb, s):
    g = pb.BatchGraph([s], tol=1e-6, precision="f32")
    try:
        g.launch()
        i = g.results()[0]
        return g.outs[0].clone(), i
    finally:
        g.close()


def serve(pb, s):
    srv = pb.Server(pb.Server.request_bytes(s) + (16 << 20), max_slots=2, device=DEV)
    try:
        rid = srv.submit(s, tol=1e-6, precision="f32")
        for _ in range(1000):
            for done, info in srv.step(chunk=64):
                assert done == rid
                return srv.outputs[rid].clone(), info
    finally:
        srv.close()


WAYS = {"solve": lambda pb, s: pb.solve(s, tol=1e-6, precision="f32"),
        "refine": lambda pb, s: pb.solve(s, tol=1e-9, precision="f32_refine64"),
        "batch": lambda pb, s: tuple(v[0] for v in pb.solve_batch([s], tol=1e-6, precision="f32")),
        "graph": graph_run, "server": serve}


@pytest.mark.parametrize("way,boundary", [("solve", "free"), ("solve", "periodic"), ("refine", "free"),
                                          ("batch", "free"), ("graph", "free"), ("server", "free")])
def test_independent_of_the_coded_setting(pb, way, boundary):
    s = molecule_system(pb, boundary)
    x1, i1 = WAYS[way](pb, s)
    pb.set_coded_coefficients(False)
    try:
        x0, i0 = WAYS[way](pb, s)
    finally:
        pb.set_coded_coefficients(True)
    assert i1["status"] == i0["status"] == pb.PB_OK
    assert torch.equal(x1, x0) and i1["iters"] == i0["iters"]


def test_unfit_operator_meets_the_dictionary_once(pb):
    s = molecule_system(pb)
    rng = np.random.default_rng(3)
    for a in (s.eps_x, s.eps_y, s.eps_z):
        a.copy_(torch.as_tensor(rng.uniform(1, 80, tuple(a.shape)), device=DEV))
    torch.cuda.synchronize()
    act = torch.profiler.ProfilerActivity
    with torch.profiler.profile(activities=[act.CPU, act.CUDA]) as prof:
        x, info = pb.solve(s, tol=1e-5, precision="f32")
        torch.cuda.synchronize()
    names = [e.name for e in prof.events()]
    solves = [n for n in names if "jpcg" in n]
    if not solves:
        pytest.skip("the profiler recorded no kernels of the library")
    assert info["coded_launches"] == 0 and len(solves) == 1, solves
    assert sum("k_dict_insert" in n for n in names) == 1
