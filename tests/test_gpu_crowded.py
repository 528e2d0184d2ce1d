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


def _crowd(rule="srd", precision=64, accel=None, colloid=True, bulk=0.3, counts=(65, 100, 128, 129, 200, 700)):
    p = W.base_params(L=(12, 13, 14), rho=5, dt=0.002, n_md=3, rule=rule, precision=precision)
    p["bulk_rate"] = bulk
    if accel:
        p["accel"] = accel
    elif colloid:
        W.add_colloid(p, (6.0, 6.5, 7.0), sigma=2.0, eps_B=0.5, catalytic=1)
    s = W.random_state(p, 62, species_B_fraction=0.5, float32=precision == 32)
    k = 11
    # around the colloid's cut-off, within its list reach and beyond it
    for i, c in enumerate(counts):
        _pile(s, k, c, (8.1 + 0.01 * i, 6.5 + 1.1 * (i - 2.5), 7.3 + 1.2 * (i % 2)), seed=70 + i)
        k += c + 7
    # (the core of the colloid stays free of particles)
    d = s["x"] - np.array([6.0, 6.5, 7.0])[:, None]
    assert accel or not colloid or (d * d).sum(axis=0).min() > 1.0
    return p, s


@pytest.mark.parametrize("tuning", [None, dict(collide_ppt=1), dict(collide_block=512),
                                    dict(collide_block=512, collide_ppt=1, collide_cells=8)])
@pytest.mark.parametrize("kind", ["colloid", "accelerated"])
def test_oversized_cells_bitwise(kind, tuning):
    """Reaction, its energy, list membership and catalysis of oversized cells."""
    rm = _rm()
    p, s = _crowd(accel=(0.3, -0.1, 0.2) if kind == "accelerated" else None)
    print(f"[crowded] {kind} N={p['n_solvent']} {tuning}", flush=True)
    g = rm.System(p, 9)
    if tuning:
        g.set_tuning(**tuning)
    g.set_state(s)
    o = oracle.Oracle(p, 9, init=False)
    o.set_state(s)
    for k in range(3):
        g.step(3, 1)
        o.run(3, 1)
        a, b = g.get_state(), o.get_state()
        for f in ("id", "state", "x", "v", "X", "V"):
            assert np.array_equal(np.asarray(a[f]), np.asarray(b[f])), (f, k)
    ga, oa = g.observables(raise_on_flags=False), o.observables()
    for f in ("n_B", "n_bulk_flips", "n_cat_flips", "n_candidates", "n_cells_T", "flags"):
        assert ga[f] == oa[f], f
    assert ga["n_bulk_flips"] > 0
    assert ga["temperature"] == pytest.approx(oa["temperature"], rel=1e-12)
    assert ga["e_rxn"] == pytest.approx(oa["e_rxn"], rel=1e-9, abs=1e-9)
    g.close()


@pytest.mark.parametrize("tuning", [None, dict(collide_ppt=1)])
def test_oversized_cells_thermostat(tuning):
    """(Box-Muller draws: 1e-12 after one interval.)"""
    rm = _rm()
    p, s = _crowd(rule="at", colloid=False)
    print(f"[crowded] thermostat N={p['n_solvent']} {tuning}", flush=True)
    g = rm.System(p, 9)
    if tuning:
        g.set_tuning(**tuning)
    g.set_state(s)
    o = oracle.Oracle(p, 9, init=False)
    o.set_state(s)
    g.step(3, 1)
    o.run(3, 1)
    a, b = g.get_state(), o.get_state()
    assert np.array_equal(a["id"], b["id"]) and np.array_equal(a["state"], b["state"])
    assert np.abs(a["v"] - b["v"]).max() <= 1e-12
    assert np.abs(a["x"] - b["x"]).max() <= 1e-12
    ga, oa = g.observables(), o.observables()
    assert ga["n_cells_T"] == oa["n_cells_T"] and ga["n_bulk_flips"] == oa["n_bulk_flips"]
    assert ga["temperature"] == pytest.approx(oa["temperature"], rel=1e-12)
    g.close()


def _interval_us(rm, p, state, n_md):
    import time
    import torch
    s = rm.System(p, 3)
    s.set_state(state)
    s.step(n_md, 2)
    best = 1e9
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        s.step(n_md, 5)
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t) / 5 * 1e6)
    s.close()
    return best


@pytest.mark.parametrize("rule", ["srd", "at"])
def test_cells_beyond_a_run_cost_by_their_particles(rule):
    """512 cells of 200 particles, which do not fit a wave's run, beside 512
    cells of 100, which do: at most four times the time (twice the particles,
    four times the comparisons for their order)."""
    rm = _rm()
    t = {}
    for k in (100, 200):
        p = W.base_params(L=(32, 32, 32), rho=1, dt=0.01, n_md=5, rule=rule, kT=1e-12)
        n = p["n_solvent"] = 512 * k
        g = np.stack(np.meshgrid(*[np.arange(8) * 4 + 0.77] * 3, indexing="ij"), 0).reshape(3, -1)
        s = W.random_state(p, 63)
        s["x"] = np.repeat(g, k, axis=1) + 1e-3 * np.random.default_rng(1).random((3, n))
        s["v"][:] = 0.0
        t[k] = _interval_us(rm, p, s, 5)
    print(f"[crowded] {rule}: {t}", flush=True)
    assert t[200] <= 4.0 * t[100]
