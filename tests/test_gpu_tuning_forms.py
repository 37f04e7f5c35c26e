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
