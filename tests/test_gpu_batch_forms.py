"""Batches that mix problems of the compact resident form (139 x 141 x 137 and 153 x 150 x 155 in FP32)
with problems that have no code words: one below the size that holds a dictionary (15 x 13 x 14) and
one whose operator has more values than a dictionary (random edges). A problem's form follows from its
own shape and operator, so its result is bitwise that of the problem alone, direct and recorded; and
the recorded batch's streaming launch shares its workgroups among the problems that stream in it."""
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


def molecule_system(pb, dims, natoms, seed):
    p = synth.small_problem(*dims, natoms, seed=seed, precision="f32")
    return pb.setup(p.grid, p.mol.xyz, p.mol.radius, p.mol.charge, p.eps_in, p.eps_out, p.kappa_d2, device=DEV)


def random_system(pb, dims, seed):
    s = molecule_system(pb, dims, 20, seed)
    rng = np.random.default_rng(seed)
    for a in (s.eps_x, s.eps_y, s.eps_z):
        a.copy_(torch.as_tensor(rng.uniform(1, 80, tuple(a.shape)), device=DEV))
    return s


@pytest.fixture(scope="module")
def compact(pb):
    s = molecule_system(pb, (139, 141, 137), 200, 31)
    x, i = pb.solve_batch([s], tol=1e-6, precision="f32")
    assert i[0]["status"] == pb.PB_OK and i[0]["coded_launches"] == 1
    return s, x[0], i[0]["iters"]


@pytest.mark.parametrize("other", ["small", "random", "random_compact", "larger"])
def test_compact_problem_in_any_mix(pb, compact, other):
    s, x1, iters = compact
    o = {"small": lambda: molecule_system(pb, (15, 13, 14), 4, 7), "random": lambda: random_system(pb, (49, 45, 41), 8),
         "random_compact": lambda: random_system(pb, (141, 131, 149), 9),
         "larger": lambda: molecule_system(pb, (201, 193, 189), 200, 10)}[other]()
    codes = 1 if other == "larger" else 0
    alone, ia = pb.solve_batch([o], tol=1e-6, precision="f32")
    xs, infos = pb.solve_batch([o, s], tol=1e-6, precision="f32")
    assert [i["status"] for i in infos] == [pb.PB_OK] * 2
    assert [i["coded_launches"] for i in infos] == [codes, 1]
    assert torch.equal(xs[1], x1) and infos[1]["iters"] == iters
    assert torch.equal(xs[0], alone[0]) and infos[0]["iters"] == ia[0]["iters"]
    g = pb.BatchGraph([o, s], tol=1e-6, precision="f32")
    try:
        for _ in range(3):
            g.launch()
            ig = g.results()
            assert [i["coded_launches"] for i in ig] == [codes, 1] and [i["status"] for i in ig] == [pb.PB_OK] * 2
            assert torch.equal(g.outs[1], x1) and torch.equal(g.outs[0], alone[0])
            torch.zeros(1 << 20, device=DEV).add_(1.0)
    finally:
        g.close()


def test_recorded_mix_takes_no_longer(pb):
    """Ten compact problems and one that streams: recorded, the latter has the whole streaming launch, as
    in the direct batch, and the two take the same device time (1.25: the spread of two timings)."""
    systems = [molecule_system(pb, (153, 150, 155), 200, 50 + k) for k in range(10)]
    systems.append(molecule_system(pb, (201, 193, 189), 200, 60))
    direct, recorded = [], []
    g = pb.BatchGraph(systems, tol=1e-6, precision="f32")
    try:
        for _ in range(3):
            direct.append(pb.solve_batch(systems, tol=1e-6, precision="f32")[1][0]["kernel_seconds"])
            g.launch()
            recorded.append(g.results()[0]["kernel_seconds"])
    finally:
        g.close()
    print(f"direct {min(direct)*1e3:.2f} ms, recorded {min(recorded)*1e3:.2f} ms", flush=True)
    assert min(recorded) <= 1.25 * min(direct)


def test_autotune_times_what_streams(pb):
    """Of a batch with one problem that streams, that one is timed, as it is alone (1.3: two timings); what
    the whole batch is refused for stays refused."""
    big = molecule_system(pb, (201, 193, 189), 200, 60)
    systems = [molecule_system(pb, (117, 113, 121), 100, 70 + k) for k in range(12)] + [big]
    z0 = pb.get_batch_zchunk()
    try:
        alone = min(pb.batch_autotune([big], precision="f32", iters_per_trial=20)["seconds"] for _ in range(2))
        mixed = min(pb.batch_autotune(systems, precision="f32", iters_per_trial=20)["seconds"] for _ in range(2))
        print(f"autotune: alone {alone*1e3:.2f} ms, in the batch {mixed*1e3:.2f} ms", flush=True)
        assert mixed <= 1.3 * alone
        small = molecule_system(pb, (9, 8, 7), 2, 1)
        with pytest.raises(pb.PBError):
            pb.batch_autotune([small] * 5000 + [big], precision="f32", iters_per_trial=1)
    finally:
        pb.set_batch_zchunk(z0)
