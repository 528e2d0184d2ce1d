"""The record layout's kernels at the edges of their ranges, bit for bit
against the FP64 oracle: streaming with coordinates that leave the box several
times in an interval, start on its faces or do not move; tiles with fewer
particles than cells, more cells than a run holds, cells beyond a wave's slots
and the density at which the collision changes form; every workgroup and
register shape of the streaming, and its three places (in the MD chain's
launch, before it, beside it)."""
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


def _same(p, state, n_md, n_coll, tuning=None):
    rm = _rm()
    print(f"[records] L={p['L']} N={p['n_solvent']} n_md={n_md} tuning={tuning}", flush=True)
    g = rm.System(p, 11)
    if tuning:
        g.set_tuning(**tuning)
    g.set_state(state)
    o = oracle.Oracle(p, 11, init=False)
    o.set_state(state)
    for k in range(n_coll):
        g.step(n_md, 1)
        o.run(n_md, 1)
        a, b = g.get_state(), o.get_state()
        for f in ("id", "state", "x", "v", "X", "V"):
            assert np.array_equal(np.asarray(a[f]), np.asarray(b[f])), (f, k)
    g.close()


@pytest.mark.parametrize("L,rho", [
    ((5, 6, 7), 40),      # workgroup form
    ((4, 4, 4), 32),      # the last density of the wave form
    ((4, 4, 4), 33),      # the first of the workgroup form
    ((33, 9, 5), 0.3),    # runs bounded by their cells
    ((65, 3, 3), 2),
    ((3, 5, 67), 5),
    ((16, 16, 16), 3),    # the largest grid that the permutation scans itself
    ((17, 16, 16), 3),
])
def test_densities_and_ragged_boxes(L, rho):
    p = W.base_params(L=L, rho=rho, dt=0.02, n_md=6)
    p["bulk_rate"] = 0.02
    _same(p, W.random_state(p, 5, species_B_fraction=0.4), 6, 3)


@pytest.mark.parametrize("n_md", [1, 9, 10, 11, 25])
def test_many_wraps_and_faces(n_md):
    p = W.base_params(L=(6, 8, 5), rho=6, dt=0.05, n_md=n_md)
    s = W.random_state(p, 9)
    x, v = np.array(s["x"]), np.array(s["v"])
    L = np.array(p["L"], dtype=float)
    v[:, ::7] = np.clip(40.0 * v[:, ::7], -40.0, 40.0)   # leaves the box every few steps
    v[:, 1::7] = 0.0
    v[:, 2::7] *= -0.0
    x[0, 3::7] = 0.0
    x[1, 4::7] = np.nextafter(L[1], 0.0)
    x[:, 5::7] = np.nextafter(0.0, 1.0)
    v[:, 5::7] = -np.abs(v[:, 5::7])
    s["x"], s["v"] = x, v
    _same(p, s, n_md, 3)


@pytest.mark.parametrize("tuning", [
    None,                                           # streaming in the chain's launch
    dict(chain_serial=1, stream_block=64, stream_ppt=1),
    dict(chain_serial=1, stream_block=128, stream_ppt=2),
    dict(chain_serial=1, stream_block=256, stream_ppt=4),
    dict(collide_ppt=1, collide_cells=8),
    dict(collide_block=512, collide_cells=64),
    dict(chain_block=512),
])
def test_streaming_places_and_shapes(tuning):
    p = W.base_params(L=(14, 13, 15), rho=7, dt=0.01, n_md=12)
    W.add_colloid(p, (4.0, 5.0, 6.0), sigma=1.5, catalytic=1)
    p["bulk_rate"] = 0.01
    p["n_solvent"] -= 37
    _same(p, W.random_state(p, 3, species_B_fraction=0.2), 12, 3, tuning)


@pytest.mark.parametrize("shift", [(0, 0, 0), (1, -1, 0), (-1, 1, 1), (2, -2, 5)])
@pytest.mark.parametrize("nc", [1, 2, 3])
def test_colloid_images_within_and_beyond_a_box_length(nc, shift):
    """Unwrapped colloid positions in every range of the periodic image, up to
    the faces, for every variant of the chain by colloid count."""
    p = W.base_params(L=(15, 14, 16), rho=4, dt=0.01, n_md=8)
    L = np.array(p["L"], dtype=float)
    for k, x in enumerate([(0.0, 3.0, 4.0), (7.5, np.nextafter(L[1], 0.0), 8.0), (11.0, 7.0, 13.0)][:nc]):
        W.add_colloid(p, x, sigma=1.2 + 0.1 * k, catalytic=k % 2)
    s = W.random_state(p, 21 + nc)
    s["X"] = np.asarray(s["X"]) + np.array(shift) * L
    _same(p, s, 8, 3)
