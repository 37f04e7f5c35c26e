"""Debye-Hueckel values at the faces where the sum is interpolated: the right-hand side of
the nodes inside each face against the oracle's direct sum, reference behaviour
b = 4 pi q / h^3 + eps / h^2 * phi_DH(ghost).

Tolerance, relative to the largest right-hand side of the faces: each atom is exact or
interpolated to 3.1e-15 of its own largest value on a tile, and 2,000 to 4,000 terms are
added in FP64 in another order than the oracle's (a random walk of 64 roundings of 1.1e-16,
about 7e-15, for terms of both signs whose sum of magnitudes is up to some ten times the
largest result): 2e-13.
"""

import numpy as np
import pytest

from oracle import fdpb

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pb():
    import paper_1704_02745_amd as m
    return m


# 130 nodes are one tile of the first level, 131 are two; kappa 0.16 leaves the first level out
# (kappa w above 4.5), kappa 1 both; 261 x 131 x 66 has faces of different tile counts; in the last
# two the atoms reach to within a node of the faces
@pytest.mark.parametrize("dims,natoms,kappa,reach",
                         [((130, 130, 130), 1500, 0.0, 0.7), ((131, 131, 131), 1500, 0.1261, 0.7),
                          ((130, 129, 131), 1500, 0.16, 0.7), ((130, 130, 131), 1200, 1.0, 0.7),
                          ((261, 131, 66), 4000, 0.1261, 0.7), ((129, 140, 133), 1500, 0.1261, 0.985)])
def test_faces_against_oracle(pb, dims, natoms, kappa, reach):
    rng = np.random.default_rng(11)
    h, e_out = 0.5, 78.54
    nx, ny, nz = dims
    half = 0.5 * h * (np.asarray(dims) - 1)
    origin = tuple(-half)
    xyz = reach * half * rng.uniform(-1.0, 1.0, (natoms, 3))
    radius = np.full(natoms, 0.2)
    charge = rng.uniform(-1.0, 1.0, natoms)
    grid = pb.make_grid(nx, ny, nz, h, origin)
    s = pb.setup(grid, xyz, radius, charge, 2.0, e_out, kappa * kappa, device="cuda:0", want_q=True)
    b = s.rhs.cpu().numpy()
    q = s.qgrid.cpu().numpy()
    eps = {0: s.eps_x.cpu().numpy(), 1: s.eps_y.cpu().numpy(), 2: s.eps_z.cpu().numpy()}
    axes = [origin[a] + h * np.arange(dims[a]) for a in range(3)]
    err, top = 0.0, 0.0
    for axis in range(3):
        for side in (0, 1):
            inner = [slice(1, -1)] * 3                       # i, j, k
            inner[axis] = slice(0, 1) if side == 0 else slice(dims[axis] - 1, dims[axis])
            at = [axes[a][inner[a]] for a in range(3)]
            at[axis] = np.array([origin[axis] + h * (-1.0 if side == 0 else float(dims[axis]))])
            pts = np.stack(np.meshgrid(*at, indexing="ij"), -1).reshape(-1, 3)
            phi = np.concatenate([fdpb.dh_potential(c, xyz, charge, e_out, kappa * kappa)
                                  for c in np.array_split(pts, max(1, len(pts) // 2048))])
            phi = phi.reshape([len(a) for a in at]).transpose(2, 1, 0)
            edge = [slice(1, -1)] * 3
            edge[axis] = slice(0, 1) if side == 0 else slice(dims[axis], dims[axis] + 1)
            e = eps[axis][edge[2], edge[1], edge[0]]
            node = (inner[2], inner[1], inner[0])
            want = fdpb.FOUR_PI * q[node] / h ** 3 + e / (h * h) * phi
            err = max(err, np.abs(b[node] - want).max())
            top = max(top, np.abs(e / (h * h) * phi).max())
    assert err <= 2e-13 * top, (err, top)
