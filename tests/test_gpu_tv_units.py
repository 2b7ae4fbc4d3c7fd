"""How the regulariser's kernel cuts a grid into waves: columns of 16, 32 and 64
lanes with rows folded into the rest, four rows per lane, one plane or several
per unit. At the edges of each, value and gradient against the FP64 oracle.

Tolerances: the value and the gradient are sums of at most four terms per cell,
each a few roundings of 6e-8 (FP32) or 1.1e-16 (FP64) off, taken relative to
the norm; the FP32 inputs are exact on both sides: 1e-5 and 1e-12 leave room
for cancellation in a cell's sum."""
import numpy as np
import pytest
import torch

from oracle import tv as orc_tv
from paper_2603_11045_amd.solver import Solver

pytestmark = pytest.mark.gpu

# (nz, ny, nx)
SHAPES = [
    (3, 2, 16), (5, 15, 16), (4, 17, 17), (6, 9, 32), (7, 8, 33), (2, 5, 64), (3, 4, 65), (40, 33, 31), (5, 1, 200),
    (1, 65, 2), (17, 260, 256), (64, 200, 130),     # the last two: units of several planes, with a remainder in z or not
]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_tv_units_match_oracle(shape, precision):
    print("tv units", shape, precision, flush=True)
    nz, ny, nx = shape
    h, eps, weight = (0.2, 0.3, 0.1), 1e-3, 0.7
    t = torch.float32 if precision == "f32" else torch.float64
    a = np.random.default_rng(sum(shape)).uniform(0.1, 1.0, size=shape)
    a = a.astype(np.float32).astype(np.float64) if precision == "f32" else a
    s = Solver(nx, ny, nz, h=h, precision=precision)
    v, g = s.tv(torch.from_numpy(a).cuda().to(t), eps=eps, weight=weight)
    s.close()
    v_o, g_o = weight * orc_tv.tv_value(a, h, eps), weight * orc_tv.tv_grad(a, h, eps)
    tol = 1e-12 if precision == "f64" else 1e-5
    assert abs(v - v_o) <= tol * abs(v_o)
    assert np.linalg.norm(g.cpu().numpy() - g_o) <= tol * np.linalg.norm(g_o)
    assert np.abs(g.cpu().numpy() - g_o).max() <= 100 * tol * np.abs(g_o).max()
