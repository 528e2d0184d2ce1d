"""Boxes with many more cells than particles, whose per-cell work is not a few
particle workgroups' to do."""
import time

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


def _box(L, n, **kw):
    p = W.base_params(L=L, rho=1, dt=0.02, n_md=6, **kw)
    p["n_solvent"] = n
    return p


@pytest.mark.parametrize("L,n", [
    ((16, 16, 16), 1), ((16, 16, 16), 100), ((16, 16, 16), 1024), ((16, 16, 16), 1025), ((17, 16, 16), 100), ((64, 64, 64), 1000),
    ((33, 9, 65), 500), ((33, 9, 65), 5000), ((40, 40, 40), 2 * 1024 + 1),
])
@pytest.mark.parametrize("kind", ["bulk", "hilbert", "colloid", "colloids", "accelerated", "serial"])
def test_sparse_boxes_bitwise(L, n, kind):
    rm = _rm()
    p = _box(L, n)
    p["bulk_rate"] = 2.0
    if kind == "hilbert":
        p["cell_order"] = "hilbert"
    if kind in ("colloid", "serial"):
        W.add_colloid(p, (5.0, 4.5, 6.0), sigma=1.5, eps_B=0.5, catalytic=1)
    if kind == "colloids":
        for k in range(3):
            W.add_colloid(p, (2.5 + 4.0 * k, 4.5, 6.0), sigma=1.2, catalytic=k % 2)
    if kind == "accelerated":
        p["accel"] = (0.1, 0.0, -0.2)
    print(f"[sparse] L={L} n={n} {kind}", flush=True)
    s = W.random_state(p, 5, species_B_fraction=0.5)
    # pairs, so that cells collide
    s["x"][:, 1::2] = np.clip(s["x"][:, :2 * (n // 2):2] + 0.05, 0.0, np.array(L)[:, None] - 0.01)
    if p["colloids"]:
        for c in p["colloids"]:
            d = s["x"] - np.array(c["x"])[:, None]
            near = (d * d).sum(axis=0) < 0.9 * c["sigma"] ** 2
            s["x"][:, near] = 0.25
    g = rm.System(p, 11)
    if kind == "serial":
        g.set_tuning(chain_serial=1)
    g.set_state(s)
    o = oracle.Oracle(p, 11, init=False)
    o.set_state(s)
    for k in range(3):
        g.step(6, 1)
        o.run(6, 1)
        a, b = g.get_state(), o.get_state()
        for f in ("id", "state", "x", "v", "X", "V"):
            assert np.array_equal(np.asarray(a[f]), np.asarray(b[f])), (f, k)
    assert g.observables()["n_candidates"] == o.observables()["n_candidates"]
    g.close()


def test_sparse_thermostat_and_plates():
    rm = _rm()
    for kind in ("at", "plates"):
        p = _box((40, 40, 40), 1500)
        if kind == "at":
            p["rule"] = "at"
        else:
            p["walls"], p["wall_density"], p["accel"] = 1, 3, (0.1, 0.0, 0.0)
        s = W.random_state(p, 6)
        s["x"][:, 1::2] = np.clip(s["x"][:, ::2] + 0.05, 0.0, 39.99)
        g = rm.System(p, 11)
        g.set_state(s)
        o = oracle.Oracle(p, 11, init=False)
        o.set_state(s)
        g.step(6, 1)
        o.run(6, 1)
        a, b = g.get_state(), o.get_state()
        assert np.array_equal(a["id"], b["id"])
        assert np.abs(a["v"] - b["v"]).max() <= 1e-12 and np.abs(a["x"] - b["x"]).max() <= 1e-12
        g.close()


def test_sparse_and_dense_slots_of_one_batch():
    rm = _rm()
    ps = [_box((40, 40, 40), 900), W.dimer_system(L=14, rho=5, n_md=6, seed=3, bulk_rate=0.05),
          _box((16, 16, 16), 20), _box((20, 20, 20), 40000)]
    b = rm.Batch(4, 64)
    for k, p in enumerate(ps):
        b.set_slot(k, p, 31 + k, 6)
    b.step(3)
    for k, p in enumerate(ps):
        g = rm.System(p, 31 + k)
        g.step(6, 3)
        x, y = b.get_state(k), g.get_state()
        for f in ("id", "state", "x", "v", "X", "V"):
            assert np.array_equal(np.asarray(x[f]), np.asarray(y[f])), (k, f)
        g.close()
    b.close()


def _interval_us(rm, p):
    import torch
    s = rm.System(p, 3)
    s.step(p["n_md"], 2)
    best = 1e9
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        s.step(p["n_md"], 5)
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t) / 5 * 1e6)
    s.close()
    return best


@pytest.mark.parametrize("L", [64, 128])
@pytest.mark.parametrize("colloid", [False, True])
def test_fewer_particles_never_take_longer(L, colloid):
    """The same box with 0.2 particles per cell and with a thousand in all."""
    rm = _rm()
    t = {}
    for n in (L ** 3 // 5, 1000):
        p = _box((L, L, L), n)
        if colloid:
            W.add_colloid(p, (20.0, 21.0, 22.0), sigma=3.0, catalytic=1)
        t[n] = _interval_us(rm, p)
    print(f"[sparse] {L}^3 colloid={colloid}: {t}", flush=True)
    assert t[1000] <= 1.25 * t[L ** 3 // 5]
