"""The 40-byte pass's deferred x step: with beta >= kDeferBeta a pass leaves x alone and the next adds
both steps, the direction before its own rebuilt as (p - r/d) / beta. The FP32 recurrence of both ways
of summing x on the same r and p, on the host: the rounding error of x against its sum in 64 bits is no
larger than with every step added by itself.

Tolerance: 2% of a root mean square over 18,000 to 90,000 nodes, whose sampling error is about
1/sqrt(2n) = 0.5% for independent roundings and larger for neighbours' that go together. No GPU involved."""
import os
import re

import numpy as np
import pytest

import synth
from oracle import fdpb

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
f32, f64 = np.float32, np.float64


def defer_beta():
    src = open(os.path.join(ROOT, "paper_1704_02745_amd", "csrc", "jpcg.hip")).read()
    assert "beta >= T(kDeferBeta)" in src
    return float(re.search(r"constexpr double kDeferBeta = ([0-9.]+);", src).group(1))


def fma(a, b, c):
    return (f64(a) * b.astype(f64) + c).astype(f32)


@pytest.mark.parametrize("dims,natoms,seed", [((33, 33, 33), 50, 1), ((29, 24, 27), 20, 4), ((49, 45, 41), 150, 2)])
def test_deferred_step_rounds_x_no_worse(dims, natoms, seed):
    s = fdpb.assemble_problem(synth.small_problem(*dims, natoms, seed=seed, precision="f32"))
    h2, ex, ey, ez = s.h ** 2, s.eps_x, s.eps_y, s.eps_z
    D = ((ex[:, :, :-1] + ex[:, :, 1:] + ey[:, :-1] + ey[:, 1:] + ez[:-1] + ez[1:]) / h2 + s.kappa2).astype(f32)
    X, Y, Z = ((e / h2).astype(f32) for e in (ex[:, :, 1:-1], ey[:, 1:-1], ez[1:-1]))
    inv = f32(1) / D

    def apply(p):
        q = D * p
        q[:, :, :-1] -= X * p[:, :, 1:]
        q[:, :, 1:] -= X * p[:, :, :-1]
        q[:, :-1] -= Y * p[:, 1:]
        q[:, 1:] -= Y * p[:, :-1]
        q[:-1] -= Z * p[1:]
        q[1:] -= Z * p[:-1]
        return q

    def dot(a, b):
        return float((a.astype(f64) * b).sum())

    limit = defer_beta()
    r = s.b.astype(f32)
    p = r * inv
    rz = dot(r, p)
    exact = np.zeros(r.shape)
    each, deferred = np.zeros_like(r), np.zeros_like(r)
    pending, before, skipped = 0.0, 0.0, 0
    for k in range(1, 81):
        q = apply(p)
        alpha = rz / dot(p, q)
        rn = fma(f32(-alpha), q, r)
        zn = rn * inv
        new = dot(rn, zn)
        beta = new / rz
        exact += f64(f32(alpha)) * p.astype(f64)
        each = fma(f32(alpha), p, each)
        if pending != 0.0:
            deferred = fma(f32(alpha), p, deferred)
            deferred = fma(f32(pending / before), p - r * inv, deferred)
            pending = 0.0
        elif f32(beta) >= f32(limit):
            pending, before, skipped = alpha, beta, skipped + 1
        else:
            deferred = fma(f32(alpha), p, deferred)
        if k in (5, 10, 20, 40, 80):
            x = fma(f32(pending), p, deferred) if pending != 0.0 else deferred
            assert np.linalg.norm(x - exact) <= 1.02 * np.linalg.norm(each - exact), k
        p, r, rz = fma(f32(beta), p, zn), rn, new
    assert skipped >= 10
