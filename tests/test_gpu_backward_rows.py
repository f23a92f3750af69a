"""The matrix-core blend backward at the edges of its blocks: chunks of 1 to
17 rows (blocks of 1, 4 and 8), lists of partial groups of eight entries, a
batch boundary (more than 256 entries in a tile), entries that wrap around the
azimuth circle (a coarse full-circle grid with Gaussians close to the view),
clamped weights, power and amplitude gradients.  Gradients against the FP64
oracle's reverse mode within the suite's 1e-4 of each tensor's largest entry:
FP32 sums of at most a few thousand terms err by some 1e-6 of it."""
import math

import numpy as np
import pytest

from oracle import oracle as O
from paper_2605_24290_amd import scenes as S

from .parity import gpu, needs_gpu, renderer_for

pytestmark = [gpu, needs_gpu]

GRID = S.Grid(36, 72, -math.pi / 2, math.pi / 36)
TOL = 1e-4


def _case(K, N, mode, use_mlp, near, seed):
    wl = S.make_workload("c1" if use_mlp else "c0", K=K, N=N, grid=GRID, seed=seed, use_mlp=use_mlp)
    sc = wl.scene
    rng = np.random.default_rng(seed)
    if near:
        # some Gaussians within a metre of the first view: their boxes span the
        # azimuth circle; some nearly opaque ones: their weights reach the clamp
        c = wl.tx[0] if mode == "tx" else wl.rx[0]
        d = rng.normal(size=(near, 3))
        d /= np.linalg.norm(d, axis=1, keepdims=True)
        sc.means[:near] = (c + d * rng.uniform(0.3, 0.9, size=(near, 1))).astype(np.float32)
        sc.logits[near:2 * near] = 6.0
    return wl, rng


@pytest.mark.parametrize("mode,N,K,use_mlp,near", [
    ("rx", 3, 7, False, 0), ("rx", 2, 900, True, 12), ("tx", 1, 300, True, 8), ("tx", 2, 300, False, 8),
    ("tx", 3, 1100, True, 12), ("tx", 5, 500, True, 8), ("tx", 8, 260, False, 8), ("tx", 9, 700, True, 8),
    ("tx", 17, 400, True, 8)])
def test_gradients(mode, N, K, use_mlp, near):
    import torch
    from paper_2605_24290_amd import rxgs
    wl, rng = _case(K, N, mode, use_mlp, near, 400 + K + N)
    dC = rng.normal(size=(N, 2, GRID.H, GRID.W)).astype(np.float32)
    dP = (0.1 * rng.normal(size=N)).astype(np.float32)
    r = renderer_for(wl)
    saved = rxgs.Saved(r)
    C, P, _ = r.render(wl.rx, tx=wl.tx, mode=mode, saved=saved)
    g = r.backward(saved, C, torch.as_tensor(dC, device="cuda"), torch.as_tensor(dP, device="cuda"))
    cen, rv = O.views_for(mode, wl.tx, wl.rx)
    ora = O.render(wl.scene, GRID, cen, wl.rx, rv, mlp=wl.mlp)
    # (a pixel whose decision lies within the FP32 evaluation's reach of its
    # threshold is given no weight in the loss, on both sides)
    sure = (ora["margin"] >= 1e-4)[:, None]
    assert sure.mean() > 0.97
    dC = np.where(sure, dC, np.float32(0.0))
    dP0 = np.zeros_like(dP)
    g = r.backward(saved, C, torch.as_tensor(dC, device="cuda"), torch.as_tensor(dP0, device="cuda"))
    want = O.backward(wl.scene, GRID, cen, wl.rx, rv, dC, dP0, mlp=wl.mlp)
    for k, v in g.items():
        a, b = v.cpu().numpy().ravel().astype(np.float64), want[k].ravel()
        assert np.abs(a - b).max() <= TOL * np.abs(b).max(), (k, np.abs(a - b).max() / np.abs(b).max())
    saved.close()
    r.close()


@pytest.mark.parametrize("mode,N", [("rx", 2), ("tx", 6)])
def test_power_and_amplitude_paths_are_linear(mode, N):
    """dL/dC, dL/dpower and dL/damplitude enter one pixel gradient: the sum of
    their separate backwards is the joint one."""
    import torch
    from paper_2605_24290_amd import rxgs
    wl, rng = _case(600, N, mode, True, 8, 77)
    r = renderer_for(wl)
    saved = rxgs.Saved(r)
    C, P, _ = r.render(wl.rx, tx=wl.tx, mode=mode, saved=saved)
    t = lambda *s: torch.as_tensor(rng.normal(size=s).astype(np.float32), device="cuda")
    dC, dP, dA = t(*C.shape), t(N), t(N, GRID.H, GRID.W)
    joint = r.backward(saved, C, dC, dP, dA=dA)
    joint = {k: v.double() for k, v in joint.items()}
    parts = [r.backward(saved, C, dC), r.backward(saved, C, None, dP), r.backward(saved, C, None, None, dA=dA)]
    for k, v in joint.items():
        s = sum(p[k].double() for p in parts)
        assert float((s - v).abs().max()) <= 1e-4 * float(v.abs().max()), k
    saved.close()
    r.close()
