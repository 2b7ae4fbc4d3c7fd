"""One context that changes its grid and comes back after a full round of 256 launch
numbers: words that the first grid left in the slots and halo banks then carry
the tags that its new launches wait for, unless they were cleared in between.
Bit for bit against a fresh context."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2603_11045_amd import _lib
from paper_2603_11045_amd import workloads as wl

pytestmark = pytest.mark.gpu

BIG, SMALL = (96, 64, 16), (48, 40, 4)


class Context:
    def __init__(self):
        self.lib = _lib.load()
        self.ctx = ctypes.c_void_p()
        assert self.lib.nh_create(ctypes.byref(self.ctx), torch.cuda.current_device(),
                                  ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
        assert self.lib.nh_set_barrier_timeout(self.ctx, 5.0) == 0

    def grid(self, shape, jacobi_k=0):
        assert self.lib.nh_set_grid(self.ctx, *shape, 1.0, 1.0, 1.0) == 0
        assert self.lib.nh_set_jacobi_sweeps(self.ctx, jacobi_k) == 0

    def forward(self, w):
        a, q = torch.from_numpy(w.alpha).cuda(), torch.from_numpy(w.q_xy).cuda()
        qt = np.ascontiguousarray(w.q_t[:w.nsteps], dtype=np.float64)
        out = torch.empty(w.nsteps, w.ny, w.nx, device="cuda")
        code = self.lib.nh_forward(self.ctx, a.data_ptr(), q.data_ptr(), qt.ctypes.data_as(ctypes.POINTER(ctypes.c_double)),
                                   w.dt, w.nsteps, out.data_ptr())
        assert code == 0, _lib.last_error(self.ctx)
        torch.cuda.synchronize()
        return out

    def close(self):
        self.lib.nh_destroy(self.ctx)


@pytest.mark.parametrize("jacobi_k", [0, 9], ids=["cg", "fixed-k"])
def test_a_grid_used_again_a_round_later(jacobi_k):
    problem = lambda shape, n, seed: wl.small_problem(*shape, n, seed=seed, dt=2.0, precision="f32", rtol=1e-6)
    c, fresh = Context(), Context()
    try:
        fresh.grid(BIG, jacobi_k)
        c.grid(BIG, jacobi_k)
        c.forward(problem(BIG, 13, 1))       # twelve steps and a launch of one
        c.grid(SMALL)
        for n in [12] * 20 + [3]:            # 243 numbers on another grid
            c.forward(problem(SMALL, n, 2))
        c.grid(BIG, jacobi_k)
        for k in range(16):                  # the same numbers again, modulo 256, one step a launch
            print("tag round", jacobi_k, k, flush=True)
            w = problem(BIG, 1, 10 + k)
            assert torch.equal(c.forward(w), fresh.forward(w)), k
    finally:
        c.close()
        fresh.close()
