"""The FP32 V-cycle's marching and bottom kernels (PB_OP_MG) at the edges of their tiles and
chunks, against the FP64 hierarchy (separate kernels, checked against the oracle).

x after one iteration is alpha_0 M b. Tolerance, relative to the largest |x|: the cycle is a
chain of some 60 damped sweeps over the levels, each adding a few roundings of 6e-8 to
values that the smoothing and the transfers do not amplify, and alpha is a quotient of sums in
FP64: 60 * 3 * 6e-8 = 1.1e-5.
"""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pb():
    import paper_1704_02745_amd as m
    return m


# tiles of 256 threads own 12 x 10 (down), 12 x 12 (up) and 14 x 14 columns, those of 1024 (from
# 2^20 nodes on) 28 x 26, 28 x 28 and 30 x 30: whole tiles, one column more, odd and even sizes in
# each direction; two levels only; bottoms of one and two levels, with and without room for them
@pytest.mark.parametrize("dims", [(60, 60, 60), (61, 61, 31), (85, 71, 29), (24, 22, 20), (14, 13, 12), (12, 11, 10),
                                  (140, 9, 7), (7, 100, 45), (113, 105, 91), (112, 104, 96), (141, 91, 83),
                                  (8, 301, 440)])
def test_one_vcycle_fp32(pb, dims):
    prob = synth.small_problem(*dims, 60, seed=4)
    sm = pb.setup(prob.grid, prob.mol.xyz, prob.mol.radius, prob.mol.charge, prob.eps_in, prob.eps_out, prob.kappa_d2,
                  device="cuda:0")
    kw = dict(tol=1e-300, op="mg", maxiter=1, check=False)
    ref, _ = pb.solve(sm, precision="f64", **kw)
    x, _ = pb.solve(sm, precision="f32", **kw)
    try:
        pb.set_coded_coefficients(False)
        x0, _ = pb.solve(sm, precision="f32", **kw)
    finally:
        pb.set_coded_coefficients(True)
    assert torch.equal(x, x0)
    assert float((x - ref).abs().max()) <= 1.1e-5 * float(ref.abs().max())
