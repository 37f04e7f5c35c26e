"""What a solve server keeps of its arena for itself."""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def pb():
    import paper_1704_02745_amd as m
    return m


@pytest.mark.parametrize("slots", [1, 256, 4096])
def test_reserve_per_slot(pb, slots):
    """One kernel argument record (240 bytes), an offset (4), a digest (32) and a record (64) per slot, each
    array rounded up to 256 bytes: the rest of the arena is for requests."""
    srv = pb.Server(64 << 20, max_slots=slots, device=DEV)
    try:
        assert srv.stats()["arena_used"] <= 340 * slots + 4 * 256
    finally:
        srv.close()


def test_requests_and_reserve_fill_the_arena(pb):
    """An arena of exactly the requests and that reserve holds them all at once."""
    systems = []
    for k, dims in enumerate([(45, 41, 47), (97, 89, 93), (139, 141, 137), (33, 29, 31)]):
        p = synth.small_problem(*dims, 60, seed=300 + k, precision="f32")
        systems.append(pb.setup(p.grid, p.mol.xyz, p.mol.radius, p.mol.charge, p.eps_in, p.eps_out, p.kappa_d2,
                                device=DEV))
    want = [pb.solve_batch([s], tol=1e-5, precision="f32")[0][0] for s in systems]
    arena = sum(pb.Server.request_bytes(s) for s in systems) + 340 * len(systems) + 4 * 256
    srv = pb.Server(arena, max_slots=len(systems), device=DEV)
    try:
        ids = {srv.submit(s, tol=1e-5, precision="f32"): k for k, s in enumerate(systems)}
        out = {}
        for step in range(1000):
            for rid, info in srv.step(chunk=16):
                assert info["status"] == pb.PB_OK
                out[ids[rid]] = srv.outputs[rid].clone()
            if step == 0:
                assert srv.stats()["pending"] == 0
            if len(out) == len(systems):
                break
    finally:
        srv.close()
    assert all(torch.equal(out[k], want[k]) for k in range(len(systems)))
