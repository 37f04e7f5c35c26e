"""The streaming kernels of the batch and the server, on shapes that no resident form takes: more
nodes than the bricks of the device hold (FP64 from 1.05 million, FP32 without code words from 2.5 and
with them from 5.64 million), or more planes (2,048, 4,864, 11,008). Against the oracle, alone against
in a mix, recorded against direct, and served in chunks of any length."""
import numpy as np
import pytest
import torch

import synth
from oracle import fdpb, pcg

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def pb():
    import paper_1704_02745_amd as m
    return m


def arrays(dims, seed, salt, few):
    """Random edges (few: one dielectric and three salt values, which fit a dictionary)."""
    nx, ny, nz = dims
    rng = np.random.default_rng(seed)
    edge = (lambda *s: np.full(s, 4.0)) if few else (lambda *s: rng.uniform(1, 80, s))
    k2 = rng.choice(np.array([salt, 1.5 * salt, 2.0 * salt]), (nz, ny, nx)) if few else rng.uniform(0, salt, (nz, ny, nx))
    return dict(eps_x=edge(nz, ny, nx + 1), eps_y=edge(nz, ny + 1, nx), eps_z=edge(nz + 1, ny, nx), kappa2=k2,
                b=rng.standard_normal((nz, ny, nx)))


def to_system(pb, dims, a):
    t = lambda v: torch.as_tensor(np.ascontiguousarray(v), dtype=torch.float64, device=DEV)
    return pb.System(pb.make_grid(*dims, 0.5, (0.0, 0.0, 0.0)), t(a["eps_x"]), t(a["eps_y"]), t(a["eps_z"]),
                     t(a["kappa2"]), t(a["b"]))


# the widest rows the batch takes (512 in FP32, 256 in FP64), with many values and with few; and thin
# columns, whose tiles are mostly padding
CASES = {"f32": [((512, 72, 70), 2000.0, False), ((512, 90, 130), 300.0, True), ((2, 3, 5000), 40.0, False)],
         "f64": [((256, 66, 66), 2000.0, False), ((3, 3, 2100), 40.0, False), ((113, 111, 109), 300.0, True)]}


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_streaming_batch(pb, prec):
    # against the oracle's FP64 iterate of the same number: the bars of every solve against it (1e-5 in
    # FP32, 1e-12 in FP64)
    tol, bound = (1e-6, 1e-5) if prec == "f32" else (1e-9, 1e-12)
    systems, refs = [], []
    for k, (dims, salt, few) in enumerate(CASES[prec]):
        a = arrays(dims, 40 + k, salt, few)
        refs.append(fdpb.System(h=0.5, **a))
        systems.append(to_system(pb, dims, a))
    xs, infos = pb.solve_batch(systems, tol=tol, precision=prec)
    for x, i, ref in zip(xs, infos, refs):
        o = pcg.jpcg(ref, tol, maxiter=5000)
        print(f"streaming batch {prec} {x.shape}: {i['iters']} iterations, oracle {o.iters}", flush=True)
        assert i["status"] == pb.PB_OK and i["coded_launches"] == 0
        assert abs(i["iters"] - o.iters) <= max(2, 0.02 * o.iters)
        same = o.x if i["iters"] == o.iters else pcg.jpcg(ref, 1e-300, maxiter=i["iters"]).x
        assert np.abs(x.cpu().numpy() - same).max() <= bound * np.abs(same).max()
    for k, s in enumerate(systems):
        x, i = pb.solve_batch([s], tol=tol, precision=prec)
        assert i[0]["coded_launches"] == (1 if prec == "f32" and CASES[prec][k][2] else 0)
        assert torch.equal(x[0], xs[k]) and i[0]["iters"] == infos[k]["iters"], k
    # another z-chunk: other tiles, the same problem, and alone as in a mix
    z0 = pb.get_batch_zchunk()
    try:
        pb.set_batch_zchunk(7)
        xz, iz = pb.solve_batch(systems, tol=tol, precision=prec)
        for k, s in enumerate(systems):
            x, i = pb.solve_batch([s], tol=tol, precision=prec)
            assert torch.equal(x[0], xz[k]) and i[0]["iters"] == iz[k]["iters"], k
            assert abs(iz[k]["iters"] - infos[k]["iters"]) <= 1
            if iz[k]["iters"] == infos[k]["iters"]:
                assert float((xz[k] - xs[k]).abs().max()) <= bound * float(xs[k].abs().max())
    finally:
        pb.set_batch_zchunk(z0)
    warm = [0.9 * x for x in xs]
    xw, iw = pb.solve_batch(systems, tol=tol, precision=prec, x0s=warm)
    for i, j in zip(iw, infos):
        assert i["iters"] <= j["iters"] and i["relres_true"] <= 10 * tol
    g = pb.BatchGraph(systems, tol=tol, precision=prec)
    try:
        for _ in range(3):
            g.launch()
            ig = g.results()
            assert [i["coded_launches"] for i in ig] == [1 if prec == "f32" and c[2] else 0 for c in CASES[prec]]
            assert all(torch.equal(a, b) for a, b in zip(g.outs, xs))
            torch.zeros(1 << 20, device=DEV).add_(1.0)
    finally:
        g.close()


def serve(pb, requests, chunk):
    srv = pb.Server(sum(pb.Server.request_bytes(s) for s, _, _ in requests) + (64 << 20), max_slots=8, device=DEV)
    try:
        ids = {srv.submit(s, tol=tol, precision=prec): k for k, (s, tol, prec) in enumerate(requests)}
        out = {}
        for _ in range(5000):
            for rid, info in srv.step(chunk=chunk):
                assert info["status"] == pb.PB_OK
                out[ids[rid]] = (srv.outputs[rid].clone(), info["iters"])
            if len(out) == len(requests):
                return out
    finally:
        srv.close()
    raise AssertionError("requests left over")


@pytest.mark.parametrize("coded", [True, False])
def test_served_streaming_resumes_bitwise(pb, coded):
    """A molecule of 201 x 193 x 189, whose passes leave x to the next one (its betas reach 0.9), alone (every
    running request has code words) and beside one that has none: the same bits whatever the chunks, a
    pending step of x kept across each stop, and the batch's result to 1e-5."""
    p = synth.small_problem(201, 193, 189, 200, seed=711, precision="f32")
    mol = pb.setup(p.grid, p.mol.xyz, p.mol.radius, p.mol.charge, p.eps_in, p.eps_out, p.kappa_d2, device=DEV)
    requests = [(mol, 1e-4, "f32"), (mol, 1e-5, "f32_refine64")]
    if not coded:
        requests.append((to_system(pb, (150, 140, 130), arrays((150, 140, 130), 3, 2.0, False)), 1e-4, "f32"))
    whole = serve(pb, requests, 100000)
    xb, ib = pb.solve_batch([mol], tol=1e-4, precision="f32")
    assert abs(whole[0][1] - ib[0]["iters"]) <= max(2, 0.02 * ib[0]["iters"])
    assert float((whole[0][0] - xb[0]).abs().max()) <= 1e-3 * float(xb[0].abs().max())
    for chunk in (1, 7, 32):
        got = serve(pb, requests, chunk)
        for k in got:
            assert got[k][1] == whole[k][1] and torch.equal(got[k][0], whole[k][0]), (chunk, k)
