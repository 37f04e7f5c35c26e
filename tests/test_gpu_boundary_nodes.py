"""Interpolated boundary sums node by node: each ghost value against the direct FP64 sum, relative to
the sum of its own terms' magnitudes, so that the weak ends of a tile count like its strong ones. Atoms
fill a ball, or lie together at one place, where the largest tiles just take them.

Tolerance: an atom is interpolated to 3.1e-15 of its largest value on a tile. At the least distance,
(1.5 + 0.1 kappa w) w from the tile's middle lines with kappa w at most 4.5, its value falls over the
tile's diagonal by at most exp(kappa (d2 - d1)) d2 / d1 with d1 = 1.95 w and d2 = (1.95^2 + 8)^(1/2) w:
exp(4.5 * 1.49) * 1.76 = 1,430, so 4.4e-12 of the node's own value."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
H, EPS_OUT = 0.5, 80.0


@pytest.fixture(scope="module")
def pb():
    import paper_1704_02745_amd as m
    return m


@pytest.mark.parametrize("dims,kd2,natoms,centre,spread,positive", [
    ((257, 257, 257), 0.0159051, 1500, (0.0, 0.0, 0.0), 40.0, False),
    ((257, 257, 257), 0.0159051, 1500, (0.0, 25.0, 25.0), 0.5, True),
    ((257, 257, 257), 0.0195, 1500, (3.0, 0.0, 0.0), 0.5, True),
    ((258, 300, 258), 0.0195, 1500, (20.0, 10.0, 0.0), 0.5, False),
    ((193, 177, 161), 0.0159051, 3000, (0.0, 0.0, 0.0), 25.0, True)])
def test_nodes(pb, dims, kd2, natoms, centre, spread, positive):
    gen = torch.Generator().manual_seed(5)
    u = torch.randn(natoms, 3, generator=gen, dtype=torch.float64)
    u = u / u.norm(dim=1, keepdim=True) * torch.rand(natoms, 1, generator=gen, dtype=torch.float64) ** (1 / 3)
    xyz = (torch.tensor(centre, dtype=torch.float64) + spread * u).to(DEV)
    q = (torch.rand(natoms, generator=gen, dtype=torch.float64) - (0.0 if positive else 0.5)).to(DEV)
    org = [-0.5 * H * (d - 1) for d in dims]
    s = pb.setup(pb.make_grid(*dims, H, org), xyz, torch.full((natoms,), 0.1, dtype=torch.float64, device=DEV), q, 1.0,
                 EPS_OUT, kd2)
    kd = math.sqrt(kd2)
    axes = [org[d] + H * torch.arange(dims[d], dtype=torch.float64, device=DEV) for d in range(3)]
    edges = (s.eps_x, s.eps_y, s.eps_z)
    worst = 0.0
    for axis in range(3):
        for side in (0, 1):
            at = [slice(1, -1)] * 3   # no edges of the box: one face's value in each node
            at[axis] = slice(0, 1) if side == 0 else slice(dims[axis] - 1, dims[axis])
            a = [axes[d][at[d]] for d in range(3)]
            a[axis] = torch.tensor([org[axis] + H * (dims[axis] if side else -1)], dtype=torch.float64, device=DEV)
            pts = torch.stack(torch.meshgrid(a[2], a[1], a[0], indexing="ij"), -1).reshape(-1, 3).flip(1)
            phi, mag = torch.empty(len(pts), dtype=torch.float64, device=DEV), torch.empty(
                len(pts), dtype=torch.float64, device=DEV)
            step = 30_000_000 // natoms
            for lo in range(0, len(pts), step):
                d = ((pts[lo:lo + step, None, :] - xyz[None]) ** 2).sum(-1).sqrt()
                t = torch.exp(-kd * d) / d * q
                phi[lo:lo + step], mag[lo:lo + step] = t.sum(1), t.abs().sum(1)
            e = list(at)
            e[axis] = slice(0, 1) if side == 0 else slice(dims[axis], dims[axis] + 1)
            scale = edges[axis][e[2], e[1], e[0]].reshape(-1) / (H * H) / EPS_OUT
            got = s.rhs[at[2], at[1], at[0]].reshape(-1)
            worst = max(worst, float(((got - scale * phi).abs() / (scale * mag)).max()))
    print(f"boundary nodes {dims} kappa^2 {kd2}: worst {worst:.2e}", flush=True)
    assert worst <= 4.4e-12
