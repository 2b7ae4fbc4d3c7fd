"""The register-resident kernel's sweeps run three planes between barriers without a
branch between them, so a tile that ends inside such a group also computes the
group's planes past its end and must leave no trace there; tiles of 32 planes
have an instance of their own. Against the streaming kernel of the same
iteration (cg_variant 1), which rounds alike: the same bits."""
import pytest
import torch

from paper_2603_11045_amd import Solver
from paper_2603_11045_amd import workloads as wl

pytestmark = pytest.mark.gpu

# (nx, ny, nz, planes per tile): groups that a tile fills, misses by one and two planes,
# the last tile thinner than the others, tiles of one plane and of 32, ragged columns
CASES = [
    (64, 16, 9, 3), (64, 16, 10, 10), (70, 13, 11, 11), (40, 9, 7, 1), (64, 8, 5, 2), (96, 24, 40, 17),
    (64, 16, 33, 32), (64, 16, 63, 32), (64, 16, 31, 31), (64, 16, 32, 32), (130, 20, 64, 32),
]


def run(nx, ny, nz, tile_z, variant):
    w = wl.small_problem(nx, ny, nz, 4, seed=nx + nz, dt=2.0, precision="f32", rtol=1e-6)
    gs = wl.random_surface_weights(4, ny, nx, seed=3)
    s = Solver(nx, ny, nz, h=(0.9, 1.1, 0.7), rtol=1e-6, max_iter=3000, cg_variant=variant, tile_z=tile_z)
    s.set_barrier_timeout(5.0)               # a lost reduction would end the call, not hang it
    S = s.forward(torch.from_numpy(w.alpha).cuda().float(), torch.from_numpy(w.q_xy).cuda().float(), w.q_t, w.dt, 4)
    G, dq, dT0 = s.adjoint_vjp(torch.from_numpy(gs).cuda().float())
    out = (S, G, dq, dT0), (s.step_iters("forward"), s.step_iters("adjoint")), s.stats()["resident"]
    s.close()
    return out


@pytest.mark.parametrize("nx,ny,nz,tile_z", CASES)
def test_resident_sweeps_match_streaming(nx, ny, nz, tile_z):
    print("resident sweep", nx, ny, nz, tile_z, flush=True)
    a, it_a, res = run(nx, ny, nz, tile_z, 2)
    b, it_b, res_b = run(nx, ny, nz, tile_z, 1)
    assert res == 1 and res_b == 0
    assert all((x == y).all() for x, y in zip(it_a, it_b))
    for x, y in zip(a, b):
        assert torch.equal(x, y)
