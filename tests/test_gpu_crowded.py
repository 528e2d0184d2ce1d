"""Cells holding more particles than a collision group, which the workgroup
collides one after the other: against the FP64 oracle.

A tight cluster of particles at rest stays in one cell: particles of one
velocity keep one velocity under the collision's rotation, so the cluster moves
as a whole."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


def _rm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1608_04904_amd as rm
    return rm


def _pile(s, first, count, at, spread=1e-3, seed=1):
    """Particles [first, first + count) of state s at rest around `at`."""
    rng = np.random.default_rng(seed)
    sl = slice(first, first + count)
    s["x"][:, sl] = np.asarray(at, dtype=float)[:, None] + spread * rng.random((3, count))
    s["v"][:, sl] = 0.0


@pytest.mark.parametrize("L,rho,count,n0,tuning", [
    ((6, 5, 8), 6, 150, 200, None),                       # beyond a wave's 128 slots
    ((6, 5, 8), 6, 80, 120, dict(collide_ppt=1)),         # beyond 64
    ((6, 5, 8), 6, 350, 400, dict(collide_block=512)),
    ((6, 5, 8), 6, 300, 300, None),                       # with the cell's others: full, no virtual particles
    ((5, 6, 7), 40, 600, 1000, None),                     # workgroup form, beyond its 512
])
@pytest.mark.parametrize("layer", [0, 1])
def test_oversized_cell_cut_by_a_plate(L, rho, count, n0, tuning, layer):
    """A cell of the first or last layer with fewer particles than
    wall_density holds virtual ones, however many real ones it has, and counts
    for no temperature.  (The virtual momentum is a Box-Muller draw: 1e-12.)"""
    rm = _rm()
    print(f"[crowded] plates L={L} count={count} n0={n0} layer={layer} {tuning}", flush=True)
    p = W.base_params(L=L, rho=rho, dt=0.002, n_md=2)
    p["walls"], p["wall_density"], p["accel"] = 1, n0, (0.01, 0.0, 0.0)
    s = W.random_state(p, 61)
    _pile(s, 10, count, (2.3, 2.6, 0.004 if layer == 0 else L[2] - 0.006))
    g = rm.System(p, 8)
    if tuning:
        g.set_tuning(**tuning)
    g.set_state(s)
    o = oracle.Oracle(p, 8, init=False)
    o.set_state(s)
    for _ in range(2):
        g.step(2, 1)
        o.run(2, 1)
    a, b = g.get_state(), o.get_state()
    assert np.array_equal(a["id"], b["id"])
    assert np.abs(a["v"] - b["v"]).max() <= 1e-12 * max(np.abs(b["v"]).max(), 1.0)
    assert np.abs(a["x"] - b["x"]).max() <= 1e-12 * max(L)
    ga, oa = g.observables(), o.observables()
    assert ga["n_cells_T"] == oa["n_cells_T"]
    assert ga["temperature"] == pytest.approx(oa["temperature"], rel=1e-11)
    g.close()
