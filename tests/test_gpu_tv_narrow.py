"""The regulariser on small, narrow and thin grids: a thread per cell, and beyond that
lanes of 1 to 64 columns with rows folded into the rest, one row or four per
lane. Value and gradient against the FP64 oracle.

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
    (1, 1, 1), (5000, 1, 1), (9, 8, 8), (300, 3, 3), (5, 1, 64), (4000, 100, 1),     # a thread per cell: few columns,
    (20, 128, 128),                                                                  # and the largest of the others
    (300, 1200, 1), (300, 600, 2), (300, 400, 3), (300, 220, 5), (128, 200, 13), (128, 100, 30), (100, 50, 70),
    (64, 2, 5000), (4000, 1, 101),                                                   # one row per lane
    (300, 1000, 4), (260, 1001, 7), (257, 300, 15), (64, 3, 5000), (1000, 50, 70),   # four rows per lane
]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("added", [False, True])
def test_tv_narrow_grids_match_oracle(shape, precision, added):
    print("tv narrow", shape, precision, flush=True)
    nz, ny, nx = shape
    h, eps, weight = (0.2, 0.3, 0.1), 1e-3, 0.7
    t = torch.float32 if precision == "f32" else torch.float64
    rng = np.random.default_rng(sum(shape))
    a = rng.uniform(0.1, 1.0, size=shape)
    a = a.astype(np.float32).astype(np.float64) if precision == "f32" else a
    g0 = rng.standard_normal(shape) if added else np.zeros(shape)
    s = Solver(nx, ny, nz, h=h, precision=precision)
    v, g = s.tv(torch.from_numpy(a).cuda().to(t), eps=eps, weight=weight,
                grad=torch.from_numpy(g0.copy()).cuda() if added else None)
    s.close()
    v_o, g_o = weight * orc_tv.tv_value(a, h, eps), g0 + weight * orc_tv.tv_grad(a, h, eps)
    tol = 1e-12 if precision == "f64" else 1e-5
    assert abs(v - v_o) <= tol * abs(v_o)
    assert np.linalg.norm(g.cpu().numpy() - g_o) <= tol * np.linalg.norm(g_o) + 1e-300
