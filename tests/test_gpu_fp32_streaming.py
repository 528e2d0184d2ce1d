"""FP32 streaming bit for bit: the drifts of one interval evaluated here in
numpy, each fused multiply-add rounded once to float (the oracle is FP64).  The
collision that follows changes velocities and order, not positions, so the
particles are compared by id."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

F = np.float32


def _rm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1608_04904_amd as rm
    return rm


def fma32(a, b, c):
    """fma of floats: the product is exact in double; the sum is rounded to odd
    (53 bits, two more than twice 24 are not needed), then once to float."""
    p = np.asarray(a, dtype=np.float64) * np.asarray(b, dtype=np.float64)
    c = np.asarray(c, dtype=np.float64)
    s = p + c
    t = s - p
    err = (p - (s - t)) + (c - t)
    even = (s.view(np.int64) & 1) == 0
    s = np.where((err > 0) & even, np.nextafter(s, np.inf), s)
    s = np.where((err < 0) & even, np.nextafter(s, -np.inf), s)
    return s.astype(F)


def wrap(x, L):
    L = F(L)
    up = x >= L
    dn = x < 0
    y = np.where(dn, x + L, x)
    y = np.where(dn & (y >= L), y - L, y)
    return np.where(up, x - L, y).astype(F)


def test_fma32_rounds_once():
    """Products that fall just beside the middle of two floats."""
    a, b = F(1 + 2 ** -12), F(1 + 2 ** -12)           # 1 + 2^-11 + 2^-24: a tie
    assert fma32(a, b, F(0)) == F(1 + 2 ** -11)
    assert fma32(a, b, F(2 ** -60)) == F(1 + 2 ** -11 + 2 ** -23)
    assert fma32(a, b, F(-2 ** -60)) == F(1 + 2 ** -11)


def _streamed(p, s):
    x, v = s["x"].astype(F), s["v"].astype(F)
    dt, hdt = F(p["dt"]), F(0.5 * p["dt"])
    g = [F(a) for a in p.get("accel", (0, 0, 0))]
    flow = any(a != 0 for a in g)
    for _ in range(p["n_md"]):
        for d in range(3):
            if flow:
                v[d] = fma32(hdt, g[d], v[d])
            x[d] = wrap(fma32(dt, v[d], x[d]), p["L"][d])
            if flow:
                v[d] = fma32(hdt, g[d], v[d])
    return x


@pytest.mark.parametrize("n_md", [1, 9, 10, 11, 25])
@pytest.mark.parametrize("kind,tuning", [
    ("solvent", {}), ("solvent", dict(stream_block=64, stream_ppt=4)),
    ("colloid", {}), ("colloid", dict(chain_serial=1, stream_ppt=1)), ("colloid", dict(chain_block=512)),
    ("accelerated", {}), ("accelerated", dict(stream_block=128)), ("accelerated", dict(stream_block=64)),
])
def test_fp32_drifts_bitwise(kind, tuning, n_md):
    rm = _rm()
    p = W.base_params(L=(7, 9, 6) if kind != "colloid" else (12, 13, 11), rho=8, dt=0.04, n_md=n_md, precision=32)
    if kind == "accelerated":
        p["accel"] = (0.3, -0.7, 1.1)
    if kind == "colloid":
        # (no force: the list's members then drift as the others do)
        W.add_colloid(p, (6.0, 6.0, 5.0), sigma=1.0, eps_A=0.0, eps_B=0.0)
    s = W.random_state(p, 31, float32=True)
    x, v = s["x"], s["v"]
    L = np.array(p["L"], dtype=float)
    far = np.flatnonzero(np.abs(x - np.array([6.0, 6.0, 5.0])[:, None]).max(axis=0) > 3.0)
    v[:, far[::7]] = np.clip(30.0 * v[:, far[::7]], -30.0, 30.0).astype(F)      # leaves the box every few steps
    v[:, far[1::7]] = 0.0
    x[0, far[2::7]] = 0.0
    x[1, far[3::7]] = np.nextafter(F(L[1]), F(0))
    x[:, far[4::7]] = np.nextafter(F(0), F(1))
    v[:, far[4::7]] = -np.abs(v[:, far[4::7]])
    print(f"[fp32] {kind} n_md={n_md} {tuning}", flush=True)
    g = rm.System(p, 3)
    if tuning:
        g.set_tuning(**tuning)
    g.set_state(s)
    g.step(n_md, 1)
    a = g.get_state()
    want = np.empty((3, p["n_solvent"]), dtype=F)
    want[:, s["id"]] = _streamed(p, s)
    got = a["x"].astype(F)
    bad = (got != want[:, a["id"]]).any(axis=0)
    assert not bad.any(), (int(bad.sum()), got[:, bad][:, :3], want[:, a["id"]][:, bad][:, :3])
    g.close()
