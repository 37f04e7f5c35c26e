"""A system that pb_solve refuses costs its preparation and not a solve: the resident form, whose
flags are read back after it, does nothing on it."""
import time

import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def pb():
    import paper_1704_02745_amd as m
    return m


@pytest.mark.parametrize("prec,dims", [("f32", (129, 127, 125)), ("f64", (97, 93, 95))])
def test_refused_before_the_solve(pb, prec, dims):
    """One node of slightly negative kappa^2 leaves the operator definite, so a solve of it would run through
    its 200 iterations and more; the preparation takes a tenth of that, half is allowed."""
    p = synth.small_problem(*dims, 100, seed=3, precision="f32")
    s = pb.setup(p.grid, p.mol.xyz, p.mol.radius, p.mol.charge, p.eps_in, p.eps_out, p.kappa_d2, device=DEV)

    def timed():
        best = 1e9
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            try:
                pb.solve(s, tol=1e-6, precision=prec)
                status = pb.PB_OK
            except pb.PBError as e:
                status = e.status
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        return best, status

    good, status = timed()
    assert status == pb.PB_OK
    for field, value, want in (("kappa2", -1e-6, pb.PB_ERR_ARG), ("eps_x", -1e-9, pb.PB_ERR_ARG),
                               ("rhs", float("nan"), pb.PB_ERR_NONFINITE)):
        a = getattr(s, field)
        old = a[1, 2, 3].item()
        a[1, 2, 3] = value
        bad, status = timed()
        print(f"{prec} {field}: refused in {bad * 1e6:.0f} us, a solve takes {good * 1e6:.0f}", flush=True)
        assert status == want and bad <= 0.5 * good, field
        a[1, 2, 3] = old
    assert timed()[1] == pb.PB_OK
