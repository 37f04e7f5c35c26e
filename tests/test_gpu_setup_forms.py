"""The setup's one-launch form for small molecules and its separate launches, on either side of
the rule (256 atoms, 2048 charge keys), against the oracle: mask, edges, salt term and
charges exactly; the right-hand side to 1e-12 of its largest value (FP64 sums in another order
than the oracle's, each term to a few roundings)."""
import numpy as np
import pytest

import synth
from oracle import fdpb, periodic

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pb():
    import paper_1704_02745_amd as m
    return m


@pytest.mark.parametrize("natoms", [0, 1, 2, 50, 256, 257])
@pytest.mark.parametrize("boundary", ["free", "periodic"])
def test_setup_forms(pb, natoms, boundary):
    rng = np.random.default_rng(natoms + 1)
    nx, ny, nz, h = 31, 27, 22, 0.5
    origin = np.array([-7.3, -6.1, -5.2])
    size = h * (np.array([nx, ny, nz]) - 1)
    # half of the atoms within two nodes of one another: runs of many keys per node
    xyz = origin + rng.uniform(0.1, 0.9, (natoms, 3)) * size
    xyz[natoms // 2:] = origin + 0.5 * size + rng.uniform(-1, 1, (natoms - natoms // 2, 3)) * h
    rad, q = rng.uniform(0.3, 1.6, natoms), rng.uniform(-0.8, 0.8, natoms)
    args = (nx, ny, nz, h, origin, xyz, rad, q, 2.0, 80.0, 0.0159051)
    ref, parts = (periodic if boundary == "periodic" else fdpb).assemble(*args, with_parts=True)
    g = synth.Grid(nx, ny, nz, h, origin)
    for kw in (dict(want_q=True, want_mask=True), {}):
        s = pb.setup(g, xyz, rad, q, *args[-3:], device="cuda:0", boundary=boundary, **kw)
        for a, b in ((s.eps_x, ref.eps_x), (s.eps_y, ref.eps_y), (s.eps_z, ref.eps_z), (s.kappa2, ref.kappa2)):
            assert np.array_equal(a.cpu().numpy(), b)
        if kw:
            assert np.array_equal(s.qgrid.cpu().numpy(), parts["qgrid"])
            mask = periodic.padded_mask(parts["mask"]) if boundary == "periodic" else parts["mask"]
            assert np.array_equal(s.mask.cpu().numpy(), mask)
        b = s.rhs.cpu().numpy()
        assert np.abs(b - ref.b).max() <= 1e-12 * max(np.abs(ref.b).max(), 1e-300)
