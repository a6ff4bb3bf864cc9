"""The current deposit's two targets (a block's LDS box, the grid itself) and the box's way back to the
grid, at sizes where their indices can go wrong: charge continuity, div E - rho unchanged from a field
of zero, with rho from the GPU's own positions.

Tolerance: a node's change is a sum of at most some hundred terms per step, each with a few roundings
relative to the density, and weights off by 2^-53 of a coordinate of up to 330 cells: below 1e-11 of
the largest density over 4 steps.
"""
import numpy as np
import pytest

from paper_1311_5551_amd import workloads as W
from paper_1311_5551_amd.sim import Run, Tables

from test_gpu_feedback import _div, _rho, _workload

pytestmark = pytest.mark.gpu


# boxes: narrow and tall, wider than a block, one cell, the whole of a small periodic grid; and chunks
# spread over more nodes than a box holds (the grid itself)
@pytest.mark.parametrize("n,x0,x1,y0,y1", [(700, 3, 5, 2, 300), (1500, 1, 330, 40, 42), (130, 7.2, 7.8, 9.1, 9.9),
                                           (1025, 0, 1, 0, 1), (5000, 0, 336, 0, 304), (1, 335.9, 336, 303.9, 304)])
def test_charge_is_conserved(oracle_tables, n, x0, x1, y0, y1):
    nx, ny, dx, dy, dt = 336, 304, 0.3, 0.25, 0.1
    F = np.zeros((9, ny, nx))
    w = _workload(n, nx, ny, dx, dy, dt, 1e-4, F, n_steps=4, spread=2.0, flags=W.FLAG_PROPAGATE)
    rng = np.random.default_rng(n)
    w.electrons["x"], w.electrons["y"] = rng.uniform(x0, x1, n) * dx, rng.uniform(y0, y1, n) * dy
    r = Run(w, Tables.from_arrays(oracle_tables))
    e = r.species(0, "electron")
    rho0 = _rho(-1e-4, e["x"], e["y"], nx, ny, dx, dy)
    for _ in range(4):
        r.step(1)
    F1, e = r.fields(0), r.species(0, "electron")
    rho1 = _rho(-1e-4, e["x"], e["y"], nx, ny, dx, dy)
    change = _div(F1[0], F1[1], dx, dy) - (rho1 - rho0)
    scale = np.abs(rho0).max()
    r.close()
    assert np.abs(rho1 - rho0).max() > 1e-3 * scale  # the charge moved
    assert np.abs(change).max() <= 1e-11 * scale
