"""What the particles' and cells' values are to the last bit and sign, whatever
form the launch takes."""
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


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("place", ["solvent", "colloid", "serial"])
@pytest.mark.parametrize("way", [-1.0, 1.0])
def test_a_coordinate_that_lands_on_zero_is_plus_zero(precision, place, way):
    """Four drifts of 1/8 take 0.5 to exactly zero, or to the upper face; nothing
    else leaves the box."""
    rm = _rm()
    p = W.base_params(L=(12, 12, 12), rho=6, dt=0.125, n_md=4, precision=precision)
    if place != "solvent":
        # (no force: a step this long would throw the solvent out of the box)
        W.add_colloid(p, (6.0, 6.0, 6.0), sigma=1.0, eps_A=0.0, eps_B=0.0)
    s = W.random_state(p, 17, float32=True)
    away = np.abs(s["x"] - 6.0).max(axis=0) > 4.0
    s["v"][:, away] = 0.0
    s["v"][:, ~away] = np.clip(s["v"][:, ~away], -3.0, 3.0)
    for d in range(3):
        k = np.flatnonzero(away)[d::3]
        s["x"][d, k], s["v"][d, k] = (0.5 if way < 0 else 11.5), way
    print(f"[bits] zero FP{precision} {place} {way}", flush=True)
    g = rm.System(p, 3)
    if place == "serial":
        g.set_tuning(chain_serial=1)
    g.set_state(s)
    g.step(4, 1)
    x = g.get_state()["x"]
    assert (x == 0.0).sum() > 100
    assert not np.signbit(x).any(), f"{int(np.signbit(x).sum())} coordinates are -0.0"
    if precision == 64:
        o = oracle.Oracle(p, 3, init=False)
        o.set_state(s)
        o.run(4, 1)
        assert x.tobytes() == np.asarray(o.get_state()["x"]).tobytes()
    g.close()


def test_observables_of_a_slot_do_not_depend_on_the_others():
    """A slot alone and beside one of 8.7 million particles, which takes
    another form of the collision: the same bits."""
    rm = _rm()
    p = W.dimer_system(L=20, rho=10, n_md=4, seed=3, bulk_rate=0.5)
    big = W.base_params(L=(96, 95, 96), rho=10, dt=0.01, n_md=4)
    s = W.random_state(p, 9, species_B_fraction=0.5)
    out = []
    for beside in (False, True):
        b = rm.Batch(2, 64)
        b.set_slot(0, p, 21, 4)
        b.set_state(0, s)
        if beside:
            b.set_slot(1, big, 22, 4)
        print(f"[bits] beside={beside}", flush=True)
        seen = []
        for _ in range(3):
            b.step(1)
            seen.append(b.observables(0))
        out.append(seen)
        b.close()
    for a, c in zip(*out):
        assert a == c, [(k, a[k], c[k]) for k in a if a[k] != c[k]]
    assert out[0][-1]["n_bulk_flips"] > 10 and out[0][-1]["e_rxn"] != 0.0


def test_waits_given_up_leave_finite_positions():
    """Three colloids take the exchange with a master workgroup; with a wait
    budget of 1 us its waits expire, and the workgroups then go on with the last
    positions they have."""
    rm = _rm()
    p = W.base_params(L=(40, 24, 24), rho=10, dt=0.01, n_md=10)
    for k in range(3):
        W.add_colloid(p, (7.0 + 13.0 * k, 12.0, 12.0), sigma=4.0)
    s = W.random_state(p, 12)
    g = rm.System(p, 3)
    g.set_tuning(barrier_budget_us=1, use_graph=0)
    g.set_state(s)
    print("[bits] waits given up", flush=True)
    g.step(10, 1)
    o = g.observables(raise_on_flags=False)
    assert o["flags"] & 32
    a = g.get_state()
    assert np.isfinite(a["x"]).all() and np.isfinite(a["v"]).all()
    assert o["flags"] & 4 == 0
    g.close()
