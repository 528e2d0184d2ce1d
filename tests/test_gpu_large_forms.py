"""Forms of the launch that only the number of particles chooses, each over
several intervals at the smallest sizes that take it, against the FP64 oracle."""
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


def _both(p, n_md, n_coll, tuning=None, exact=True, change=None):
    rm = _rm()
    print(f"[large] L={p['L']} N={p['n_solvent']} {tuning}", flush=True)
    g = rm.System(p, 9)
    if tuning:
        g.set_tuning(**tuning)
    s = g.get_state()
    if change:
        change(s)
        g.set_state(s)
    o = oracle.Oracle(p, 9, init=False)
    o.set_state(s)
    for k in range(n_coll):
        g.step(n_md, 1)
        o.run(n_md, 1)
    a, b = g.get_state(), o.get_state()
    for f in ("id", "state"):
        assert np.array_equal(a[f], b[f]), f
    for f in ("x", "v", "X", "V"):
        if exact:
            assert np.array_equal(a[f], np.asarray(b[f]).reshape(a[f].shape)), f
        else:
            assert np.abs(a[f] - np.asarray(b[f]).reshape(a[f].shape)).max(initial=0.0) <= 1e-12, f
    ga, oa = g.observables(), o.observables()
    for f in ("n_B", "n_bulk_flips", "n_cat_flips", "n_candidates", "n_cells_T", "flags"):
        assert ga[f] == oa[f], f
    assert ga["temperature"] == pytest.approx(oa["temperature"], rel=1e-11)
    assert ga["e_rxn"] == pytest.approx(oa["e_rxn"], rel=1e-9, abs=1e-9)
    g.close()


@pytest.mark.parametrize("n", [1 << 20, (1 << 20) + 1])
def test_list_closed_by_many_workgroups(n):
    """Up to 1024 chunks the first workgroup that closes an interval does the
    bookkeeping, beyond them the last to arrive; the list that each writes is used
    by the next interval and its counters are found zero again."""
    p = W.base_params(L=(48, 48, 46), rho=10, dt=0.01, n_md=4)
    p["n_solvent"] = n
    p["bulk_rate"] = 0.2
    W.add_colloid(p, (20.0, 21.0, 22.0), sigma=3.0, eps_B=0.5, catalytic=1)
    _both(p, 4, 4)


# one wave per tile: from 2^23 particles
BIG = (96, 96, 92)


def _pile(s, at, count, seed):
    rng = np.random.default_rng(seed)
    k = rng.permutation(s["x"].shape[1])[:count]
    s["x"][:, k] = np.asarray(at)[:, None] + 1e-3 * rng.random((3, count))
    s["v"][:, k] = 0.0


@pytest.mark.parametrize("kind", ["dimer", "accelerated", "plates", "thermostat"])
@pytest.mark.parametrize("ppt", [1, 2])
def test_collision_of_one_wave_per_tile(kind, ppt):
    p = W.base_params(L=BIG, rho=10, dt=0.004, n_md=2, rule="at" if kind == "thermostat" else "srd")
    p["bulk_rate"] = 0.5
    if kind == "dimer":
        W.add_dimer(p, (40.0, 41.0, 42.0), (0.6, 0.0, 0.8))
    if kind == "accelerated":
        p["accel"] = (0.2, -0.1, 0.3)
    if kind == "plates":
        p["walls"], p["wall_density"], p["accel"] = 1, 250, (0.1, 0.0, 0.0)

    def change(s):
        rng = np.random.default_rng(4)
        s["state"][:] = rng.random(s["state"].size) < 0.5
        # oversized cells, the last in the lowest layer, one beside the dimer
        for i, c in enumerate([66, 90, 127, 140, 300, 900]):
            _pile(s, (46.3 + 0.01 * i if i == 0 else 10.6 + 7.2 * i, 41.3, 44.7 if i == 0 else 0.003), c, 80 + i)
    exact = kind in ("dimer", "accelerated")
    _both(p, 2, 2 if exact else 1, dict(collide_ppt=ppt), exact, change)
