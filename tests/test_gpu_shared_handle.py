"""Reads of one handle from several host threads, and observations of every
size: the partial sums that pass through pinned host memory, those that are
copied from the workspace, and the allocation-free ones are the same."""
import ctypes as C
import threading

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _rm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1608_04904_amd as rm
    return rm


def _solvent(L, precision=64, **kw):
    return W.base_params(L=L, rho=10, dt=0.01, n_md=3, precision=precision, **kw)


def _in_threads(fs):
    err = []

    def run(f):
        try:
            f()
        except BaseException as e:            # noqa: BLE001 (reported below)
            err.append(e)
    ts = [threading.Thread(target=run, args=(f,)) for f in fs]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    if err:
        raise err[0]


def test_slots_of_a_batch_observed_by_two_threads():
    rm = _rm()
    b = rm.Batch(2, 64)
    for k, L in enumerate([(20, 20, 20), (23, 20, 20)]):
        b.set_slot(k, _solvent(L), 5 + k, 3)
    b.step(1)
    want = [b.observables(k) for k in range(2)]
    assert want[0] != want[1]
    wrong = []

    def read(k):
        for _ in range(400):
            if b.observables(k) != want[k]:
                wrong.append(k)
    print("[shared] two slots, two threads", flush=True)
    _in_threads([lambda: read(0), lambda: read(1)])
    assert not wrong, f"{len(wrong)} of 800 observations were not their slot's"
    b.close()


@pytest.mark.parametrize("L,precision", [((20, 20, 20), 64), ((20, 20, 20), 32), ((38, 38, 37), 32)])
def test_state_read_by_several_threads(L, precision):
    """Each thread with host buffers of its own (an FP32 state of more than 2^19
    particles is exchanged in two passes)."""
    rm = _rm()
    p = _solvent(L, precision)
    g = rm.System(p, 7)
    g.step(3, 1)
    want = g.get_state()
    from paper_1608_04904_amd import _StateBuffers, _capi
    wrong = []

    def read():
        buf = _StateBuffers(p["n_solvent"], 0)
        for _ in range(30):
            h = buf.host_state()
            assert _capi.lib().rmp_get_state(g.h, C.byref(h)) == _capi.OK
            for f in ("x", "v", "id", "state"):
                if not np.array_equal(getattr(buf, f)[..., ::499], want[f][..., ::499]):
                    wrong.append(f)
                    getattr(buf, f)[:] = 0
    print(f"[shared] state of {p['n_solvent']} particles, FP{precision}, six threads", flush=True)
    _in_threads([read] * 6)
    assert not wrong, wrong
    g.close()


@pytest.mark.parametrize("fields", [("x",), ("v",), ("id",), ("state",), ("x", "state"), ()])
@pytest.mark.parametrize("L,precision", [((9, 8, 7), 64), ((9, 8, 7), 32), ((40, 40, 40), 32)])
def test_reading_some_fields(L, precision, fields):
    rm = _rm()
    p = _solvent(L, precision)
    g = rm.System(p, 7)
    g.step(3, 1)
    want = g.get_state()
    from paper_1608_04904_amd import _StateBuffers, _capi
    buf = _StateBuffers(p["n_solvent"], 0)
    buf.x[:] = buf.v[:] = -1.0
    buf.id[:] = 7
    buf.state[:] = 9
    h = buf.host_state()
    for f in ("x", "v", "id", "state"):
        if f not in fields:
            setattr(h, f, None)
    assert _capi.lib().rmp_get_state(g.h, C.byref(h)) == _capi.OK
    for f, untouched in (("x", -1.0), ("v", -1.0), ("id", 7), ("state", 9)):
        got = getattr(buf, f)
        assert np.array_equal(got, want[f]) if f in fields else (got == untouched).all(), f
    g.close()


# up to 1, and 1024 and 1025, and 3072 chunks of 1024 particles
@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n", [1, 1024, 1025, 1 << 20, (1 << 20) + 1, 3 << 20])
def test_every_way_of_an_observation_agrees(n, precision):
    rm = _rm()
    p = _solvent((64, 64, 64), precision)
    p["n_solvent"] = n
    g = rm.System(p, 3)
    g.step(3, 1)
    print(f"[shared] observations of {n} particles FP{precision}", flush=True)
    first = g.observables()
    assert all(g.observables() == first for _ in range(10))
    assert first == g.observables_noalloc()
    g.step(3, 1)
    assert g.observables() == g.observables_noalloc() != first
    g.close()


def test_slots_of_different_size_observed_in_turn():
    rm = _rm()
    b = rm.Batch(3, 64)
    sizes = [2000, (1 << 20) + 5000, 300_000]
    alone = []
    for k, n in enumerate(sizes):
        p = _solvent((48, 48, 48))
        p["n_solvent"] = n
        b.set_slot(k, p, 9 + k, 3)
        g = rm.System(p, 9 + k)
        g.step(3, 2)
        alone.append(g.observables())
        g.close()
    b.step(2)
    for _ in range(4):
        for k in (0, 1, 2, 1, 0):
            assert b.observables(k) == alone[k], k
    b.close()


def _us(f, reps=15):
    import time
    ts = []
    for _ in range(reps):
        t = time.perf_counter()
        f()
        ts.append(time.perf_counter() - t)
    return 1e6 * sorted(ts)[reps // 2]


def test_observation_time_does_not_jump_with_the_size():
    """48^3 cells of 10 particles (1080 chunks) beside 47^3 (1014)."""
    rm = _rm()
    t = {}
    for L in (47, 48):
        g = rm.System(_solvent((L, L, L)), 3)
        g.step(3, 1)
        for _ in range(12):
            g.observables()
        t[L] = _us(g.observables)
        g.close()
    print(f"[shared] observation us {t}", flush=True)
    assert t[48] <= 1.6 * t[47]


def test_small_fp32_read_of_ids_copies_ids_alone():
    rm = _rm()
    from paper_1608_04904_amd import _StateBuffers, _capi
    p = _solvent((36, 36, 36), 32)
    g = rm.System(p, 3)
    g.step(3, 1)
    buf = _StateBuffers(p["n_solvent"], 0)
    t = {}
    for name in ("all", "ids"):
        h = buf.host_state()
        if name == "ids":
            h.x = h.v = None
        t[name] = _us(lambda: _capi.lib().rmp_get_state(g.h, C.byref(h)))
    print(f"[shared] FP32 read us {t}", flush=True)
    assert t["ids"] <= 0.5 * t["all"]
    g.close()
