"""The temporally blocked fixed-K kernels beyond one tile shape: every height of
the interior tiles, deep columns, ragged and wrapping tiles, a last phase
shorter than the others, and more steps than one launch takes. Against the
streaming kernel (forced by an explicit tile depth): the deep kernels round as
its sweep does (the same bits); the shallow ones sum the face terms in another
order, within the bound of the oracle comparison of one such solve (1e-5)."""
import numpy as np
import pytest
import torch

from paper_2603_11045_amd import Solver
from paper_2603_11045_amd import workloads as wl

pytestmark = pytest.mark.gpu

# (nx, ny, nz, rows of the interior tiles)
CASES = [
    (50, 9, 7, 2), (120, 110, 5, 4), (200, 200, 3, 8),       # nz <= 16
    (75, 50, 24, 2), (5, 7, 17, 2), (120, 110, 20, 4),       # nz <= 24
    (30, 31, 32, 2), (121, 109, 27, 4),                      # nz <= 32
]


@pytest.mark.parametrize("case", CASES, ids=["x".join(map(str, c[:3])) for c in CASES])
@pytest.mark.parametrize("periodic,robin", [(False, 0.0), (True, 0.5)])
def test_blocked_matches_streaming(case, periodic, robin):
    nx, ny, nz, rows = case
    nsteps, K = 14, 7
    print("blocked", case, periodic, robin, flush=True)
    w = wl.small_problem(nx, ny, nz, nsteps, seed=nx + nz, dt=0.4, precision="f32")
    g = torch.from_numpy(wl.random_surface_weights(nsteps, ny, nx, seed=5, dtype=np.float32)).cuda()
    outs = []
    for tz in (0, 4):
        s = Solver(nx, ny, nz, h=(0.9, 1.1, 0.5), periodic=periodic, robin=robin, jacobi_k=K, tile_z=tz)
        s.set_barrier_timeout(5.0)           # a lost phase tag would end the call, not hang it
        S = s.forward(torch.from_numpy(w.alpha).cuda(), torch.from_numpy(w.q_xy).cuda(), w.q_t, w.dt, nsteps)
        st = s.stats()
        assert st["jacobi_blocked"] == (1 if tz == 0 else 0)
        if tz == 0:
            assert st["tile_y"] == rows and st["launches_fwd"] == 2
        assert st["fwd_iters"] == K * nsteps
        res = st["worst_rel_res"]
        G, dq, dT0 = s.adjoint_vjp(g)
        outs.append(([S, dq, dT0, G], res))
        s.close()
    (a, ra), (b, rb) = outs
    assert abs(ra - rb) <= 1e-5 * rb
    for x, y in zip(a, b):
        if nz > 16:
            assert torch.equal(x, y)
        else:
            assert float((x - y).norm() / y.norm()) <= 1e-5
