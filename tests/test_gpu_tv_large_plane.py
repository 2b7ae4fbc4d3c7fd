"""The regulariser on an x-y plane of more than 2^31 cells: element offsets within a
plane are 64-bit. All cells equal but for a patch across the wrap of the y axis
(the last rows hold the offsets beyond 2^31), so the gradient is the FP64
oracle's on the patch alone and zero elsewhere, and the value the patch's plus
eps for every other cell.

Tolerances as for the small grids: 1e-5 (FP32) and 1e-12 (FP64) of the norm."""
import numpy as np
import pytest
import torch

from oracle import tv as orc_tv
from paper_2603_11045_amd.solver import Solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_plane_beyond_32_bit_offsets(precision):
    nx, ny = 46342, 46343
    assert nx * ny > 1 << 31
    print("tv large plane", precision, flush=True)
    h, eps, weight = (0.2, 0.3, 0.1), 1e-3, 0.7
    t = torch.float32 if precision == "f32" else torch.float64
    # 16 rows (the first 8 and the last 8 of the plane) x 64 columns, equal values around the patch
    rows = np.r_[0:8, ny - 8:ny]
    p = np.full((1, 16, 64), 0.5)
    rng = np.random.default_rng(5)
    p[0, :4, :48] = rng.uniform(0.1, 1.0, size=(4, 48))
    p[0, 10:, :48] = rng.uniform(0.1, 1.0, size=(6, 48))
    p = p.astype(np.float32).astype(np.float64)
    a = torch.full((1, ny, nx), 0.5, dtype=t, device="cuda")
    at = torch.from_numpy(rows).cuda()
    a[0, at, :64] = torch.from_numpy(p[0]).cuda().to(t)
    s = Solver(nx, ny, 1, h=h, precision=precision)
    v, g = s.tv(a, eps=eps, weight=weight)
    s.close()
    g_o = weight * orc_tv.tv_grad(p, h, eps)[0]
    v_o = weight * (orc_tv.tv_value(p, h, eps) + h[0] * h[1] * h[2] * eps * (nx * ny - p.size))
    # the column before the patch's first is the plane's last (the oracle's small ring: its 64th)
    cols = torch.from_numpy(np.r_[0:63, nx - 1]).cuda()
    got = g[0][at[:, None], cols[None, :]].cpu().numpy()
    tol = 1e-12 if precision == "f64" else 1e-5
    assert np.linalg.norm(got - g_o) <= tol * np.linalg.norm(g_o)
    g[0][at[:, None], cols[None, :]] = 0
    assert int(torch.count_nonzero(g)) == 0
    assert abs(v - v_o) <= tol * abs(v_o)
