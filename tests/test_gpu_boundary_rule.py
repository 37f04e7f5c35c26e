"""Which boundary sum a molecule gets, told by the names of the kernels: interpolated where its terms are
many and some face has tiles of at most a quarter of it."""
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def pb():
    import paper_1704_02745_amd as m
    return m


# 78 x 78 nodes hold 1.49 times the points of four tiles, 79 x 78 are 1.504 times; 131 nodes are two tiles
@pytest.mark.parametrize("dims,natoms,kd2,interpolated", [
    ((41, 41, 41), 10500, 0.0159051, False), ((65, 65, 65), 4200, 0.0159051, False), ((65, 65, 65), 4200, 0.0, False),
    ((78, 78, 78), 2900, 0.0159051, False), ((78, 78, 78), 2900, 0.0, False), ((79, 78, 78), 2900, 0.0159051, True),
    ((79, 78, 78), 2900, 0.0, True), ((97, 97, 97), 1600, 0.0159051, False), ((97, 97, 97), 1900, 0.0159051, True),
    ((130, 75, 75), 4000, 0.0159051, True), ((131, 75, 75), 4000, 0.0159051, False),
    ((131, 131, 60), 3500, 0.0159051, True), ((131, 131, 131), 1100, 0.0159051, True),
    ((156, 156, 156), 750, 0.0159051, True), ((156, 156, 156), 750, 0.0, True)])
def test_rule(pb, dims, natoms, kd2, interpolated):
    gen = torch.Generator().manual_seed(1)
    half = torch.tensor([0.25 * (d - 1) for d in dims], dtype=torch.float64)
    xyz = (1.4 * torch.rand(natoms, 3, generator=gen, dtype=torch.float64) - 0.7) * half
    q = torch.rand(natoms, generator=gen, dtype=torch.float64) - 0.5
    rad = torch.full((natoms,), 0.2, dtype=torch.float64)
    g = pb.make_grid(*dims, 0.5, [-float(v) for v in half])
    act = torch.profiler.ProfilerActivity
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[act.CPU, act.CUDA]) as prof:
        pb.setup(g, xyz, rad, q, 1.0, 80.0, kd2, device=DEV)
        torch.cuda.synchronize()
    names = {n for e in prof.events() for n in ("k_dh_faces", "k_dh_points") if n in e.name}
    if not names:
        pytest.skip("the profiler recorded no kernels of the library")
    assert names == {"k_dh_points" if interpolated else "k_dh_faces"}
