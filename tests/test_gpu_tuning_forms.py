"""Which form a solve runs in after a tiling was recorded for its shape, told by the names of the
kernels it launches."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def pb():
    import paper_1704_02745_amd as m
    return m


def molecule_system(pb, dims, natoms, seed, boundary="free"):
    p = synth.small_problem(*dims, natoms, seed=seed, precision="f32")
    return pb.setup(p.grid, p.mol.xyz, p.mol.radius, p.mol.charge, p.eps_in, p.eps_out, p.kappa_d2, device=DEV,
                    boundary=boundary)


def form(pb, sysm, **kw):
    """The solver kernel of a solve: resident or fused (streaming)."""
    act = torch.profiler.ProfilerActivity
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[act.CPU, act.CUDA]) as prof:
        pb.solve(sysm, **kw)
        torch.cuda.synchronize()
    names = {n for e in prof.events() for n in ("resident", "fused") if "k_jpcg_" + n in e.name}
    if not names:
        pytest.skip("the profiler recorded no kernels of the library")
    assert len(names) == 1, names
    return names.pop()


def test_verdict_is_of_the_boundary_it_was_timed_on(pb):
    """A free system of 137 x 139 x 141 whose operator has no code words streams, and so says the
    autotuner; a periodic molecule on that shape, which it did not time, runs resident as before."""
    dims = (137, 139, 141)
    free = molecule_system(pb, dims, 50, 1)
    rng = np.random.default_rng(2)
    for a in (free.eps_x, free.eps_y, free.eps_z):
        a.copy_(torch.as_tensor(rng.uniform(1, 80, tuple(a.shape)), device=DEV))
    box = molecule_system(pb, dims, 50, 3, "periodic")
    kw = dict(tol=1e-4, precision="f32")
    assert form(pb, box, **kw) == "resident" and form(pb, free, **kw) == "fused"
    pb.autotune(free, precision="f32", iters_per_trial=3)
    assert form(pb, free, **kw) == "fused" and form(pb, box, **kw) == "resident"


# 257^3-class grids stream; the others run resident, full or compact, whatever the autotuner found
@pytest.mark.parametrize("dims,prec", [((65, 57, 61), "f32"), ((141, 139, 137), "f32"), ((61, 53, 47), "f64"),
                                       ((201, 193, 189), "f32")])
def test_saved_tuning_restores_the_form(pb, dims, prec, tmp_path):
    sysm = molecule_system(pb, dims, 100, 5)
    kw = dict(tol=1e-4, precision=prec)
    best = pb.autotune(sysm, precision=prec, iters_per_trial=20)
    tuned = form(pb, sysm, **kw)
    assert (best["scheme"] >= 2) == (tuned == "resident")
    entry = dict(best, nx=dims[0], ny=dims[1], nz=dims[2], precision=prec)
    pb.save_tuning(tmp_path / "tuning.json", [entry])
    # from another record for the shape back to the saved one
    c = pb.tiling_candidates(*dims, prec)[0]
    pb.set_tuning(*dims, prec, c["block"], c["groups"], c["zchunk"], c["grid"], c["scheme"], c["streaming"], c["segments"])
    assert form(pb, sysm, **kw) == "fused" and pb.get_tuning(*dims, prec)["scheme"] == c["scheme"]
    assert pb.load_tuning(tmp_path / "tuning.json") == 1
    got = pb.get_tuning(*dims, prec)
    assert form(pb, sysm, **kw) == tuned and all(got[k] == best[k] for k in got)


@pytest.mark.parametrize("dims,prec,resident", [((45, 41, 47), "f32", True), ((133, 141, 149), "f32", True),
                                                ((41, 45, 37), "f64", True), ((191, 193, 189), "f32", False),
                                                ((129, 127, 131), "f64", False)])
def test_default_tuning_is_what_runs(pb, dims, prec, resident):
    """pb_get_tuning of a shape nothing was recorded for names the form that runs, and recording what it
    returned changes nothing; the resident form is refused where the grid does not fit it."""
    sysm = molecule_system(pb, dims, 60, 6)
    t = pb.get_tuning(*dims, prec)
    kw = dict(tol=1e-3, precision=prec)
    want = "resident" if resident else "fused"
    assert (t["scheme"] >= 2) == resident and form(pb, sysm, **kw) == want
    args = (t["block"], t["groups"], t["zchunk"], t["grid"])
    pb.set_tuning(*dims, prec, *args, t["scheme"], t["streaming"], t["segments"])
    assert form(pb, sysm, **kw) == want and pb.get_tuning(*dims, prec) == t
    if not resident:
        with pytest.raises(pb.PBError):
            pb.set_tuning(*dims, prec, *args, t["scheme"] + 2, t["streaming"], t["segments"])
