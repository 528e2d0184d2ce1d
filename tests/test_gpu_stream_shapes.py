"""Every workgroup size and number of particles per thread of the streaming
kernel: the same bits as the default, and about the same time."""
import time

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


def _params(kind, precision):
    p = W.base_params(L=(13, 11, 17), rho=7, dt=0.02, n_md=7, precision=precision)
    p["bulk_rate"] = 0.1
    if kind == "accelerated":
        p["accel"] = (0.1, 0.2, -0.1)
    if kind == "colloid":
        W.add_colloid(p, (6.0, 5.0, 8.0), sigma=1.5, eps_B=0.5, catalytic=1)
    return p


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("kind", ["solvent", "colloid", "accelerated"])
def test_streaming_shapes_same_bits(kind, precision):
    rm = _rm()
    p = _params(kind, precision)
    want = None
    for block in (256, 128, 64):
        for ppt in (2, 1, 4):
            g = rm.System(p, 5)
            g.set_tuning(chain_serial=1, stream_block=block, stream_ppt=ppt)
            print(f"[shapes] {kind} FP{precision} block={block} ppt={ppt}", flush=True)
            g.step(7, 3)
            s = g.get_state()
            want = want or s
            for f in ("id", "state", "x", "v", "X", "V"):
                assert s[f].tobytes() == want[f].tobytes(), (f, block, ppt)
            g.close()


def test_small_workgroups_keep_the_device_full():
    rm = _rm()
    import torch
    p = W.base_params(L=(64, 64, 64), rho=10, dt=0.01, n_md=20)
    t = {}
    for block, ppt in ((256, 2), (64, 1), (64, 2), (128, 2)):
        g = rm.System(p, 5)
        g.set_tuning(stream_block=block, stream_ppt=ppt, use_graph=1)
        g.step(20, 3)
        best = 1e9
        for _ in range(5):
            torch.cuda.synchronize()
            a = time.perf_counter()
            g.step(20, 10)
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - a) / 10 * 1e6)
        t[block, ppt] = best
        g.close()
    print(f"[shapes] interval us {t}", flush=True)
    assert max(t.values()) <= 1.2 * t[256, 2]
